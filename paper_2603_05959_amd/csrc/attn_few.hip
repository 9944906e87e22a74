// Attention over the half-precision cache for launches too small for the 128-query items of attn_bf16.hip: few
// tokens per frame (the camera head's one), few heads, short caches.  Those items are mostly padding or hold a
// tile or two here, and what counts is how fast K and V arrive, how many parts are merged and how many launches
// it takes: one, merges included.  Latency bounds it at the small end (one query of 16 heads over 189 slots: 5.8 us
// of a step's 19), the rate of K and V out of L2 and the vector work per score at the large one (256 queries of 192
// heads over 16640 slots: 330 us, 630 TFLOP/s).
//
// A workgroup takes G groups of 16 queries of one head over one of `splits` ranges of the slots, on
// v_mfma_f32_16x16x32_f16:
//   S^T = K Q^T      A = K rows, B = Q^T; a lane holds one query's scores
//   O^T = V^T P^T    A = V^T, B = P^T straight from the S^T accumulators
// Operands come from memory as they lie there, without LDS and without a barrier in the loop: of a
// 32-slot tile lane (l16, gl) reads 16-byte pieces of K rows l16 and 16 + l16, and of the V rows
// 4 gl + i and 16 + 4 gl + i (i < 4: the slots whose weights its accumulators hold) the elements
// 4 l16 .. +3; eight byte permutes a row quad turn these into V^T operands.  Weight sums are one more product,
// with a row of ones, over the weights as the matrix unit sees them.
//
// Queries enter as bf16 holds them, times a power of two (exact in half unless subnormal); the rest of
// scale * log2(e) is an fp32 factor of the exponent, so the error of rounding a scaled query, the largest of
// attn_bf16.hip, does not arise here.
#include "append_parts.h"
#include "attn_parts.h"
#include <math.h>

namespace ovggt {

typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2;

constexpr float kFewBias = 7.0f;        // weights are stored as 2^7 * p: the middle of the half range
constexpr float kFewLag = 8.0f;         // the reference may lag the running maximum by 2^8: weights stay below 2^15

struct AttnFewParams {
  const char* kv;
  char* meta;
  const uint16_t* q;
  char* out;
  float* recs;
  int layer0, n_total, QB, n_work, splits;
  float q_limit, q_scale;     // queries are clamped to +-q_limit and multiplied by q_scale, a power of two
  float c;                    // scale * log2(e) / q_scale
  const char *k_new, *v_new;  // APPENDS: the frame's rows
};

// APPENDS (1; 2: with the previous frame's moves): the workgroup is the only one of its head, so nobody else reads or writes
// the head's rows, and it appends the frame's before it attends (8 pieces a row, at most 64 rows).  A launch less
// where launches are what a step consists of: one token of 16 heads over 189 slots, step 18.6 -> 15.5 us.
template <int G, bool OUT_F32, int APPENDS>
__global__ void __launch_bounds__(kPartThreads)
attn_few_kernel(Geom g, AttnFewParams p) {
  __shared__ MergeArea<(G > 1 ? 2 : 1)> area;
  // Consecutive workgroups of an XCD walk the query blocks of one range of one head (its L2 holds the rows).
  const int idx = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  if (idx >= p.n_work) return;                                       // whole workgroup
  const int qb = idx % p.QB, rest = idx / p.QB;
  const int sp = rest % p.splits, lh = rest / p.splits;
  const int q0 = qb * G * kPartRows;
  const int li = lh / g.H, h = lh - li * g.H;
  const int lane = threadIdx.x & 63, l16 = lane & 15, gl = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint16_t* kbase = (const uint16_t*)layer_k((char*)p.kv, g, p.layer0 + li) + (size_t)h * g.cap * 64;
  const uint16_t* vbase = (const uint16_t*)layer_v((char*)p.kv, g, p.layer0 + li) + (size_t)h * g.cap * 64;
  const int n_total = p.n_total, nt = (n_total + 31) >> 5;
  const int t0 = (int)((long)nt * sp / p.splits), t1 = (int)((long)nt * (sp + 1) / p.splits);
  if constexpr (APPENDS > 0) {
    static_assert(G * kPartRows * 8 <= kPartThreads, "a thread for every piece");
    const int layer = p.layer0 + li, m = (int)threadIdx.x >> 3;
    const size_t frame = (size_t)li * g.M * g.H * 128;
    if (g.hybrid && h == 0) centroid_to_fp32(g, p.meta, layer, threadIdx.x, kPartThreads);
    if (m < g.M) append_piece<APPENDS == 2>(g, (char*)p.kv, p.meta, layer, p.k_new + frame, p.v_new + frame, h, m, threadIdx.x & 7, p.n_total - g.M);
    __syncthreads();                                   // the rows are stored
  }
  u32x4 kf[2][2];
  u32x2 vf[2][4];
  // rows at or beyond n_total are never read (they may hold anything): the last resident row stands in
  auto load_k = [&](int t) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const uint16_t* kp = kbase + (size_t)min(t * 32 + 16 * b + l16, n_total - 1) * 64 + 8 * gl;
#pragma unroll
      for (int j = 0; j < 2; ++j) kf[b][j] = *(const u32x4*)(kp + 32 * j);
    }
  };
  auto load_v = [&](int t) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        vf[b][i] = *(const u32x2*)(vbase + (size_t)min(t * 32 + 16 * b + 4 * gl + i, n_total - 1) * 64 + 4 * l16);
  };
  if (t0 + wave < t1) { load_k(t0 + wave); load_v(t0 + wave); }

  f16x8 qf[G][2];
#pragma unroll
  for (int q = 0; q < G; ++q) {
    const uint16_t* qp = p.q + (((size_t)li * g.M + min(q0 + q * kPartRows + l16, g.M - 1)) * g.H + h) * 64 + 8 * gl;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const u32x4 w = *(const u32x4*)(qp + 32 * j);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        qf[q][j][2 * e] = (_Float16)(__builtin_amdgcn_fmed3f(__uint_as_float(w[e] << 16), -p.q_limit, p.q_limit) * p.q_scale);
        qf[q][j][2 * e + 1] = (_Float16)(__builtin_amdgcn_fmed3f(__uint_as_float(w[e] & 0xFFFF0000u), -p.q_limit, p.q_limit) * p.q_scale);
      }
    }
  }
  const float c = p.c;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  const _Float16 one = (_Float16)1.0f;
  const f16x8 ones = {one, one, one, one, one, one, one, one};
  f32x4 O[G][4], L[G];
  float m[G];
#pragma unroll
  for (int q = 0; q < G; ++q) {
    m[q] = -3.402823466e38f;
    L[q] = zero;
#pragma unroll
    for (int d = 0; d < 4; ++d) O[q][d] = zero;
  }
  for (int t = t0 + wave; t < t1; t += kPartWaves) {
    const int tn = min(t + kPartWaves, t1 - 1);
    f32x4 S[G][2];
#pragma unroll
    for (int q = 0; q < G; ++q)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        S[q][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, kf[b][0]), qf[q][0], zero, 0, 0, 0);
        S[q][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, kf[b][1]), qf[q][1], S[q][b], 0, 0, 0);
      }
    load_k(tn);                                        // K of the next tile travels during this tile's P V, V during its Q K
    if (t * 32 + 32 > n_total) {                       // absent slots: no weight, and no 0 * inf from the stand-in row
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bool absent = t * 32 + 16 * b + 4 * gl + i >= n_total;
#pragma unroll
          for (int q = 0; q < G; ++q) S[q][b][i] = absent ? -INFINITY : S[q][b][i];
          if (absent) vf[b][i] = u32x2{0u, 0u};
        }
    }
    f16x8 P[G];
#pragma unroll
    for (int q = 0; q < G; ++q) {
      // The reference m (the maximum at some earlier tile, less 7) follows only when it is passed by 2^15, so most
      // tiles rescale nothing and look at no other lane.
      const float mx = fmaxf(fmaxf(fmaxf(S[q][0][0], S[q][0][1]), fmaxf(S[q][0][2], S[q][0][3])),
                             fmaxf(fmaxf(S[q][1][0], S[q][1][1]), fmaxf(S[q][1][2], S[q][1][3]))) * c;
      if (__builtin_amdgcn_ballot_w64(mx > m[q] + (kFewLag + kFewBias)) != 0ull) {
        float x = fmaxf(mx, __shfl_xor(mx, 16, 64));
        x = fmaxf(x, __shfl_xor(x, 32, 64));
        const float mn = fmaxf(m[q], x - kFewBias), a = __builtin_amdgcn_exp2f(m[q] - mn);
        m[q] = mn;
        L[q] *= a;
#pragma unroll
        for (int d = 0; d < 4; ++d) O[q][d] *= a;
      }
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) P[q][4 * b + i] = (_Float16)__builtin_amdgcn_exp2f(fmaf(S[q][b][i], c, -m[q]));
      L[q] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ones, P[q], L[q], 0, 0, 0);
    }
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const uint32_t sel = (d & 1) ? 0x07060302u : 0x05040100u;        // the high or the low halves of two words
      u32x4 w;
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        w[2 * b] = __builtin_amdgcn_perm(vf[b][1][d >> 1], vf[b][0][d >> 1], sel);
        w[2 * b + 1] = __builtin_amdgcn_perm(vf[b][3][d >> 1], vf[b][2][d >> 1], sel);
      }
#pragma unroll
      for (int q = 0; q < G; ++q)
        O[q][d] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, w), P[q], O[q][d], 0, 0, 0);
    }
    load_v(tn);
  }

  float l[G];
#pragma unroll
  for (int q = 0; q < G; ++q) l[q] = L[q][0];          // every row of the product with ones is the sum over the tile
  uint32_t* arrive = (uint32_t*)(layer_meta(p.meta, g, p.layer0 + li) + g.off_arrive) + (size_t)h * p.QB + qb;
  constexpr int rec = part_rec_floats(G);
  const size_t first = (size_t)lh * p.splits * p.QB + qb;              // record of range 0; the ranges are QB apart
  merge_and_write<1>(area, O, m, l, sp, p.splits, arrive, p.recs + first * rec, (size_t)p.QB * rec,
                     [&](int row, int piece, const f32x4& r) {
                       if (q0 + row >= g.M) return;
                       const size_t at = (((size_t)li * g.M + q0 + row) * g.H + h) * 64 + 4 * piece;
                       if constexpr (OUT_F32) {
                         *(f32x4*)((float*)p.out + at) = r;
                       } else {
                         const bf16x4 o = {(__bf16)r[0], (__bf16)r[1], (__bf16)r[2], (__bf16)r[3]};
                         *(bf16x4*)((__bf16*)p.out + at) = o;
                       }
                     });
}

// Ranges of the slots for each block of queries: one more for every CU that would idle, two from where both keep a tile
// for each wave (attention of 1 query of 16 heads over 301 slots: 8.3 us with one, 10.3 with two; over 561 11.1 and 10.9),
// then one for every eight tiles begun (over 801 slots 11.1, with one less 11.4).  Ranges for two workgroups a CU took 21.7
// us instead of 24.7 at 1 query of 2 heads over 2049 slots, but 57 instead of 37 at 128 of 16 over 4224.
static long few_splits(long blocks, int n_total, int cus) {
  const long tiles = (n_total + 31) / 32, most = (tiles + kPartWaves - 1) / kPartWaves;
  if (blocks >= cus || tiles < 2 * kPartWaves) return 1;
  long s = cus / blocks;
  if (s > most) s = most;
  return s > kMaxSplits ? kMaxSplits : s;
}

// What a launch with G groups of 16 queries a workgroup takes beyond the fixed part of the smallest, in us: what the
// larger merge adds, what each round of workgroups after the first adds (first loads and merge of the waves), what the
// merge of ranges adds, and the rate at which 256 CUs take 16 queries past a slot, over the share of the CUs that the
// rounds fill.  Fit over 590 launches of 1 to 2100 queries, 16 to 32 K slots and 1 to 2304 heads, all three G: 5 to 6 %
// rms.  The part per round: 226 queries over 573 slots of 2304 heads are 36 rounds of 13 us with G = 4.
static float few_cost(int G, const Geom& g, int nl, int n_total, int cus) {
  const int at = G == 1 ? 0 : G == 2 ? 1 : 2;
  constexpr float kMerge[3] = {0.f, 1.6f, 5.3f}, kRound[3] = {1.7f, 2.5f, 8.9f}, kRanges[3] = {2.5f, 3.0f, 5.5f};
  constexpr float kRate[3] = {21.0e-6f, 10.9e-6f, 6.1e-6f};
  const long blocks = (long)((g.M + G * kPartRows - 1) / (G * kPartRows)) * g.H * nl, splits = few_splits(blocks, n_total, cus);
  const long wgs = blocks * splits, rounds = (wgs + cus - 1) / cus;
  const float fill = (float)wgs / (float)(rounds * cus), rate = kRate[at] * (256.f / (float)cus);
  return kMerge[at] + kRound[at] * (float)(rounds - 1) + (splits > 1 ? kRanges[at] : 0.f) +
         rate * (float)(blocks * G) * (float)n_total / fill;
}

// More groups read K and V less often, fewer fill the chip with less work and merge sooner.
static int few_groups(const Geom& g, int nl, int n_total, int cus) {
  int best = 1;
  for (int G = 2; G <= 4; G *= 2)
    if (few_cost(G, g, nl, n_total, cus) < few_cost(best, g, nl, n_total, cus)) best = G;
  return best;
}

// Whether a launch comes here or goes to attn_bf16.hip and its merge pass.  That kernel has twice the rate once its
// workgroups hold long runs of tiles, but pays about seven tiles' time to start and finish a run, multiplies
// whole 128-query blocks, and merges one record per run; the estimate follows the way it cuts a launch.
// The margin of a tenth keeps sizes where the two are level on the older path: of the 590 launches 4 are slower than
// there, by up to 4 us.  Step times there and here, 16 heads: 1 query over 4097 slots 47.0 and 25.6 us, 64 over 16448 69
// and 42, 128 over 4224 in 12 layers 196 and 85, 700 over 4796 50 and 55; 1041 queries of 2 heads over 5137 61 and 38.
// Attention alone, short caches of many heads: 104 queries of 384 heads over 608 slots 36 and 42 us, 226 of 2304 over
// 573 177 and 469.
bool attn_few_better(const Geom& g, int nl, int n_total, int n_wgs) {
  // a tile; the ends of a run, in tiles, alone and behind another round's; runs of a workgroup that takes cut items
  constexpr float kTileUs = 1.7f, kRunTiles = 7.f, kRoundTiles = 6.5f, kRuns = 1.25f;
  const long pairs = ((long)g.H * nl + 1) / 2, QB = (g.M + kQueryTile - 1) / kQueryTile, T = (n_total + kSlotTile - 1) / kSlotTile;
  const long wgs = n_wgs, per_xcd = wgs / 8;
  float tiles, recs;      // of the busiest workgroup, run overhead included; of an item, where the merge pass has no table of them
  if (attn_whole_items(g.H * nl, (int)QB, (int)wgs)) {
    const long items = pairs / 8 * QB, left = items % per_xcd;
    tiles = (float)(items / per_xcd) * ((float)T + kRunTiles) + (left ? (float)((left * T + per_xcd - 1) / per_xcd) + kRunTiles : 0.f);
    recs = 0.f;
  } else {
    const bool by_round = pairs > 8 && pairs % 8 == 0 && QB * T >= per_xcd;      // one head pair per XCD and round
    const float chunks = by_round ? (float)per_xcd : (float)wgs / (float)pairs;  // of a head pair
    const float run = fmaxf((float)(QB * T) / chunks, 1.f);
    tiles = by_round ? (float)(pairs / 8) * (run + kRoundTiles) : run + kRunTiles * kRuns;
    recs = fminf(chunks / (float)QB, (float)T);
    const bool table = (by_round || (wgs % pairs == 0 && wgs / pairs <= 64)) && QB <= 16 && recs <= 12.f;
    if (table) recs = 0.f;
  }
  const float there = kTileUs * tiles + 4.f + 0.6f * recs;
  return 1.1f * few_cost(few_groups(g, nl, n_total, n_wgs), g, nl, n_total, n_wgs) < there;
}

AttnSplit attn_few_split(const Geom& g, int nl, int n_total, size_t ws_bytes, int n_wgs) {
  AttnSplit sp;
  const int G = few_groups(g, nl, n_total, n_wgs);
  sp.rows = G * kPartRows;
  const long blocks = (long)((g.M + sp.rows - 1) / sp.rows) * g.H * nl;
  long splits = few_splits(blocks, n_total, n_wgs);
  while (splits > 1 && (size_t)(blocks * splits) * part_rec_floats(G) * sizeof(float) > ws_bytes) --splits;
  sp.ranges = (int)splits;
  sp.work = blocks * splits;
  return sp;
}

bool attn_few_appends(const Geom& g, int nl, int n_total, size_t ws_bytes, int n_wgs) {
  const AttnSplit sp = attn_few_split(g, nl, n_total, ws_bytes, n_wgs);
  return sp.ranges == 1 && g.M <= sp.rows;
}

hipError_t launch_attn_few(const Geom& g, char* kv, char* meta, int layer0, int nl, const void* q, const void* k_new, const void* v_new,
                           int appends, void* out, int n_total, float scale, char* ws, size_t ws_bytes, int n_wgs, bool out_f32,
                           hipStream_t s) {
  AttnFewParams p;
  const AttnSplit sp = attn_few_split(g, nl, n_total, ws_bytes, n_wgs);
  p.kv = kv; p.meta = meta; p.q = (const uint16_t*)q; p.out = (char*)out; p.recs = (float*)ws;
  p.layer0 = layer0; p.n_total = n_total;
  p.QB = (g.M + sp.rows - 1) / sp.rows;
  const float c = fminf(scale * 1.4426950408889634f, 3.402823466e38f);
  p.q_limit = 65504.f / c;
  p.q_scale = ldexpf(1.0f, ilogbf(c));
  p.c = c / p.q_scale;
  p.splits = sp.ranges;
  p.k_new = (const char*)k_new; p.v_new = (const char*)v_new;
  if (appends && (sp.ranges != 1 || g.M > sp.rows)) return hipErrorInvalidValue;     // one workgroup a head
  if (sp.work > 0x7FFFFFF0L) return hipErrorInvalidValue;
  p.n_work = (int)sp.work;
  const dim3 grid((unsigned)((sp.work + 7) / 8 * 8)), block(kPartThreads);
#define OVGGT_FEW_OUT(GG, AP) \
  if (out_f32) hipLaunchKernelGGL((attn_few_kernel<GG, true, AP>), grid, block, 0, s, g, p); \
  else hipLaunchKernelGGL((attn_few_kernel<GG, false, AP>), grid, block, 0, s, g, p)
#define OVGGT_FEW_LAUNCH(GG) \
  if (appends == 0) { OVGGT_FEW_OUT(GG, 0); } else if (appends == 1) { OVGGT_FEW_OUT(GG, 1); } else { OVGGT_FEW_OUT(GG, 2); }
  switch (sp.rows / kPartRows) {
    case 1: OVGGT_FEW_LAUNCH(1); break;
    case 2: OVGGT_FEW_LAUNCH(2); break;
    default: OVGGT_FEW_LAUNCH(4); break;
  }
#undef OVGGT_FEW_OUT
#undef OVGGT_FEW_LAUNCH
  return hipGetLastError();
}

}  // namespace ovggt
