// fp32 attention of the new frame's queries over the resident cache (paper
// Sec. 3.1), for handles whose dtype is f32.
//
// Everything stays in fp32: both products run on v_mfma_f32_16x16x4_f32, the
// softmax between them on the VALU.
//   S^T = K Q^T      A = K rows, B = Q^T; a lane holds one query's scores
//   O^T = V^T P^T    A = V^T, B = P^T straight from the S^T accumulators
// The order in which a contraction index is walked is free, so operands are
// taken from memory the way they lie there: of a 16-slot tile lane (l16, g)
// reads 16-byte pieces of K row l16 (elements 16 j + 4 g .. +3) and of V rows
// 4 g .. 4 g + 3 (elements 4 l16 .. +3), whole 64- and 256-byte runs, and both
// enter the matrix unit from these registers; no operand passes through LDS.
//
// 1041 queries over 5137 slots, 16 heads (22 GFLOP): 39.5 ms as a scalar kernel with
// one workgroup per query, 230 us like this (a step of 253 us less 23 of append and
// selection; 254 under a trace), 95 TFLOP/s; the f32 matrix rate (157 at 2.4 GHz)
// bounds it: the matrix pipes are busy 60 % of the time, and what they wait for is K
// and V out of L2 (11 TB/s: a 16-query block re-reads both).  Blocks of 32 queries
// halve that traffic but fill the chip worse (528 instead of 1056 blocks for 256 CUs)
// and took 10 to 20 % longer over every size from 17 to 1041 queries.
#include "attn_parts.h"
#include <type_traits>

namespace ovggt {

constexpr float kF32Lag = 8.0f;         // the softmax reference may lag the running maximum by 2^8
constexpr int kF32Unit = 4;             // exponents of a wave that starts over, and of the merge, count powers of 2^4
constexpr float kF32Low = 6.0f;         // how far, in these, its reference lies above the maximum
constexpr float kF32Far = 0x1p100f;     // weighted sums up to here stay finite when 8 waves of 16 ranges are merged
constexpr float kF32High = 0x1p24f;     // exponents of the first walk are within 1 of the true ones up to here
constexpr int kF32Rows = kPartRows;     // queries of a workgroup
constexpr int kF32MaxRecs = 4096;       // parts of a split launch (17 MB of workspace at most)

// Workspace of an fp32 handle: one record per part.
size_t attn_f32_ws_bytes(int layer_heads, int tokens_per_frame) {
  const long blocks = (long)((tokens_per_frame + kF32Rows - 1) / kF32Rows) * layer_heads;
  const long recs = blocks * kMaxSplits < kF32MaxRecs ? blocks * kMaxSplits : kF32MaxRecs;
  return (size_t)recs * part_rec_floats(1) * sizeof(float);
}

struct AttnF32Params {
  const char* kv;
  char* meta;
  const float* q;
  float* out;
  float* recs;
  int layer0, n_total, QB, n_work, splits;
  float c, c_unit;            // softmax scale * log2(e), and the same over kF32Unit
};

// A workgroup takes 16 queries of one head over one of `splits` equal ranges of
// the slots; its waves share the 16-slot tiles of the range (wave w: every 8th
// from the w-th) and merge through LDS.  With more than one range, the parts go
// to memory and the workgroup that arrives last for a query block merges them.
__global__ void __launch_bounds__(kPartThreads)
attn_f32_kernel(Geom g, AttnF32Params p) {
  constexpr int W = kPartWaves;
  __shared__ MergeArea<1> area;
  // Consecutive workgroups of an XCD walk the query blocks of one range of one head, whose K and V
  // rows then come from that XCD's L2.
  const unsigned wg = blockIdx.y * gridDim.x + blockIdx.x;
  const int idx = (int)((wg & 7) * (gridDim.x >> 3) * gridDim.y + (wg >> 3));
  if (idx >= p.n_work) return;                                       // whole workgroup
  const int qb = idx % p.QB, rest = idx / p.QB;
  const int sp = rest % p.splits, lh = rest / p.splits;
  const int q0 = qb * kF32Rows;
  const int li = lh / g.H, h = lh - li * g.H;
  const int lane = threadIdx.x & 63, l16 = lane & 15, gl = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const float* kbase = (const float*)layer_k((char*)p.kv, g, p.layer0 + li) + (size_t)h * g.cap * 64;
  const float* vbase = (const float*)layer_v((char*)p.kv, g, p.layer0 + li) + (size_t)h * g.cap * 64;

  f32x4 qf[4];
  {
    const float* qp = p.q + (((size_t)li * g.M + min(q0 + l16, g.M - 1)) * g.H + h) * 64 + 4 * gl;
#pragma unroll
    for (int j = 0; j < 4; ++j) qf[j] = *(const f32x4*)(qp + 16 * j);
  }
  const int n_total = p.n_total, nt = (n_total + 15) >> 4;
  const int t0 = (int)((long)nt * sp / p.splits), t1 = (int)((long)nt * (sp + 1) / p.splits);
  const bool ragged = (n_total & 15) != 0;
  if (nt == 1 && wave > 0) return;                                   // one tile: one wave has it all
  f32x4 O[1][4];
  float m[1], l[1];
  auto walk = [&](auto second) {
    constexpr bool over = decltype(second)::value;
    const float c = over ? p.c_unit : p.c;
    f32x4 kf[4], vf[4];
    m[0] = -3.402823466e38f;
    l[0] = 0.f;
#pragma unroll
    for (int d = 0; d < 4; ++d) O[0][d] = f32x4{0.f, 0.f, 0.f, 0.f};
    // rows at or beyond n_total are never read (they may hold anything): the last resident row stands in
    auto load_k = [&](int t) {
      const float* kp = kbase + (size_t)min(t * 16 + l16, n_total - 1) * 64 + 4 * gl;
#pragma unroll
      for (int j = 0; j < 4; ++j) kf[j] = *(const f32x4*)(kp + 16 * j);
    };
    auto load_v = [&](int t) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        vf[i] = *(const f32x4*)(vbase + (size_t)min(t * 16 + 4 * gl + i, n_total - 1) * 64 + 4 * l16);
    };
    if (t0 + wave < t1) { load_k(t0 + wave); load_v(t0 + wave); }
    for (int t = t0 + wave; t < t1; t += W) {
      const int tn = min(t + W, t1 - 1);
      f32x4 S;
      {
        f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;        // two chains: a product never waits for the one before it
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int j = 0; j < 4; j += 2) {
            s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[j][e], qf[j][e], s0, 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[j + 1][e], qf[j + 1][e], s1, 0, 0, 0);
          }
        S = s0 + s1;
      }
      load_k(tn);                                        // K of the next tile travels during this tile's P V, V during its Q K
      if (ragged && t == nt - 1) {                       // absent slots: no weight, and no 0 * inf from the stand-in row
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bool absent = t * 16 + 4 * gl + i >= n_total;
          S[i] = absent ? -INFINITY : S[i];
          if (absent) vf[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
      }
      // The reference m follows the maximum only when it is passed by 2^8 (weights are fp32: no
      // accuracy is lost), so most tiles rescale nothing and look at no other lane.
      const float mx = fmaxf(fmaxf(S[0], S[1]), fmaxf(S[2], S[3])) * c;
      if (__builtin_amdgcn_ballot_w64(mx > m[0] + (over ? -kF32Low : kF32Lag)) != 0ull) {
        float x = fmaxf(mx, __shfl_xor(mx, 16, 64));
        x = fmaxf(x, __shfl_xor(x, 32, 64));
        const float mn = fmaxf(m[0], over ? x + kF32Low : x), a = __builtin_amdgcn_exp2f((over ? kF32Unit : 1) * (m[0] - mn));
        m[0] = mn;
        l[0] *= a;
#pragma unroll
        for (int d = 0; d < 4; ++d) O[0][d] *= a;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) S[i] = __builtin_amdgcn_exp2f(over ? kF32Unit * (S[i] * c - m[0]) : fmaf(S[i], c, -m[0]));
      l[0] += (S[0] + S[1]) + (S[2] + S[3]);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int d = 0; d < 4; ++d) O[0][d] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[i][d], S[i], O[0][d], 0, 0, 0);
      load_v(tn);
    }
  };
  walk(std::false_type());
  // Where the first walk does not hold, the wave starts over.
  // Scores times c leave the fp32 range where scores times the scale do not, and above 2^24 what a fused exponent
  // leaves of the largest score's rounding is no longer small: exponents in units of 2^4, rounded before the reference
  // is taken off, count every score that is finite once scaled.
  // Sums of weights up to 2^8, or of many weights of 1 that turn out to be small beside another wave's, leave the fp32
  // range where values of V are near its end, although the result, a mean of them, does not: with weights up to
  // 2^-24, 2^17 slots of any value stay below the largest number.
  float size = 0.f;                                      // infinities and NaN stay in it
#pragma unroll
  for (int d = 0; d < 4; ++d)
    size += (fabsf(O[0][d][0]) + fabsf(O[0][d][1])) + (fabsf(O[0][d][2]) + fabsf(O[0][d][3]));
  const bool far = !(size <= kF32Far) || !(fabsf(m[0]) <= kF32High);     // a wave without tiles, too: its m stays the lowest
  if (__builtin_amdgcn_ballot_w64(far) != 0ull) walk(std::true_type());
  else m[0] *= 1.0f / kF32Unit;

  l[0] += __shfl_xor(l[0], 16, 64);
  l[0] += __shfl_xor(l[0], 32, 64);
  if (nt == 1) {                                         // nothing to merge: 2 queries over 10 slots of 1536 heads 13.8 -> 7.9 us
    if (q0 + l16 < g.M) {
      float* o = p.out + (((size_t)li * g.M + q0 + l16) * g.H + h) * 64 + 16 * gl;
#pragma unroll
      for (int i = 0; i < 4; ++i) *(f32x4*)(o + 4 * i) = f32x4{O[0][0][i] / l[0], O[0][1][i] / l[0], O[0][2][i] / l[0], O[0][3][i] / l[0]};
    }
    return;
  }
  uint32_t* arrive = (uint32_t*)(layer_meta(p.meta, g, p.layer0 + li) + g.off_arrive) + (size_t)h * p.QB + qb;
  const size_t first = (size_t)lh * p.splits * p.QB + qb;              // record of range 0; the ranges are QB apart
  merge_and_write<kF32Unit>(area, O, m, l, sp, p.splits, arrive, p.recs + first * part_rec_floats(1), (size_t)p.QB * part_rec_floats(1),
                     [&](int row, int piece, const f32x4& r) {
                       if (q0 + row < g.M) *(f32x4*)(p.out + (((size_t)li * g.M + q0 + row) * g.H + h) * 64 + 4 * piece) = r;
                     });
}

// Ranges per query block.  Fewer blocks than CUs: one range more for every CU that would idle, as long
// as a range keeps 16 tiles, two for each wave (step time, 65 queries of 2 heads over 4161 slots: 60 us
// with 1 range, 33 with 4, 29 with 16; 700 queries of one head over 4796: 68 with 1, 36 with 4, 41 with 6;
// 17 of 8 heads over 1017: 28 with 1, 24 with 4).  More blocks than CUs: ranges smooth the last,
// partly filled round (1056 blocks = 4.1 a CU: 286 us with 1 range, 259 with 2, 250 with 3 and with 16).
static int f32_splits(long blocks, int n_tiles, long max_recs, long cus) {
  long s = 1;
  if (blocks < cus) {
    s = cus / blocks;
    if (s > n_tiles / 16) s = n_tiles / 16;
    if (s > kMaxSplits) s = kMaxSplits;
  } else if (blocks <= kMaxArrive) {
    float best = 0.f;
    for (long k = 1; k <= 4 && n_tiles / k >= 64; ++k) {
      const long rounds = (blocks * k + cus - 1) / cus;
      const float full = (float)(blocks * k) / (float)(rounds * cus);
      if (full > best + 0.02f) { best = full; s = k; }
    }
  }
  while (s > 1 && blocks * s > max_recs) --s;
  return s < 1 ? 1 : (int)s;
}

AttnSplit attn_f32_split(const Geom& g, int nl, int n_total, size_t ws_bytes, int n_wgs) {
  AttnSplit sp;
  sp.rows = kF32Rows;
  const long blocks = (long)((g.M + kF32Rows - 1) / kF32Rows) * g.H * nl;
  sp.ranges = f32_splits(blocks, (n_total + 15) / 16, (long)(ws_bytes / (part_rec_floats(1) * sizeof(float))), n_wgs);
  sp.work = blocks * sp.ranges;
  return sp;
}

// A launch takes less than 2^32 threads along x: beyond 2^22 workgroups (of 512) the grid gets rows.
bool attn_f32_grid(long work, unsigned* x, unsigned* y) {
  constexpr long kMaxX = 1L << 22;
  const long rows = (work + kMaxX - 1) / kMaxX, wide = ((work + rows - 1) / rows + 7) / 8 * 8;      // whole rounds of the 8 XCDs
  if (rows * wide > 0x7FFFFFFFL) return false;
  *x = (unsigned)wide; *y = (unsigned)rows;
  return true;
}

hipError_t launch_attn_f32(const Geom& g, char* kv, char* meta, int layer0, int nl, const void* q, void* out,
                           int n_total, float scale, char* ws, size_t ws_bytes, int n_wgs, hipStream_t s) {
  AttnF32Params p;
  const AttnSplit sp = attn_f32_split(g, nl, n_total, ws_bytes, n_wgs);
  p.kv = kv; p.meta = meta; p.q = (const float*)q; p.out = (float*)out;
  p.recs = (float*)ws;
  p.layer0 = layer0; p.n_total = n_total;
  p.QB = (g.M + kF32Rows - 1) / kF32Rows;
  p.c = scale * 1.4426950408889634f;
  p.c_unit = (scale / kF32Unit) * 1.4426950408889634f;
  p.splits = sp.ranges;
  unsigned gx, gy;
  if (!attn_f32_grid(sp.work, &gx, &gy)) return hipErrorInvalidValue;
  p.n_work = (int)sp.work;
  hipLaunchKernelGGL(attn_f32_kernel, dim3(gx, gy), dim3(kPartThreads), 0, s, g, p);
  return hipGetLastError();
}

}  // namespace ovggt
