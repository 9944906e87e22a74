// The diversity pass (paper Eq. 7's d_i) of one workgroup, for the kernel that does nothing else and for the one that
// merges the attention's parts meanwhile.
#pragma once
#include "ovggt_internal.h"
#include "../../include/ovggt.h"
#include <hip/hip_fp16.h>

namespace ovggt {

constexpr int kDivThreads = 256;
constexpr int kDivWaves = kDivThreads / 64;

__device__ inline void unpack_halfs(const uint4& w, float f[8]) {
  const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const __half2 h = *(const __half2*)&ww[t];
    f[2 * t] = __low2float(h);
    f[2 * t + 1] = __high2float(h);
  }
}

// ---- pass 2: d_i per history slot ----------------------------------------------------------------
// A wave takes 8 consecutive slots.  For every head one load instruction fetches the 8 slots' rows,
// 1 KiB of consecutive memory (the cache is head-major: a slot's key is H rows 2 MB apart, and
// pieces shorter than this made the pass latency- rather than bandwidth-bound): lane l holds the
// 16-byte piece l & 7 of slot l >> 3.  The balanced tree over the concatenated index h*64 + e
// (zero-padded to a power of two) is evaluated as: a pairwise tree over the lane's 8 elements, three
// butterfly steps over the 8 lanes of a slot (quad permutes and the half-row mirror: after each
// step all lanes of a group hold the group's sum, so any lane of the sibling group is a valid
// partner), and a tree over the heads folded in as they arrive (a binary counter of partial sums).
__device__ inline float dpp_f(float v, int ctrl_is) {
  // ctrl_is: 0 quad [1,0,3,2], 1 quad [2,3,0,1], 2 row half mirror
  const int x = __float_as_int(v);
  int y;
  switch (ctrl_is) {
    case 0: y = __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xF, 0xF, false); break;
    case 1: y = __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xF, 0xF, false); break;
    default: y = __builtin_amdgcn_update_dpp(0, x, 0x141, 0xF, 0xF, false); break;
  }
  return __int_as_float(y);
}
__device__ inline float tree8_lanes8(const float (&p)[8]) {
  float v = ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
  v = v + dpp_f(v, 0);
  v = v + dpp_f(v, 1);
  v = v + dpp_f(v, 2);
  return v;
}
constexpr int ilog2(int x) { return x <= 1 ? 0 : 1 + ilog2(x / 2); }

// dot(k, c) and |k|^2 of the 8 slots of a wave; key_of(h, k8) delivers the lane's 8 elements of head h
// (h < H).  cs: the centroid in LDS, H*64 floats.  Every lane of a slot's group returns the slot's sums.
template <int HP, typename KeyOf>
__device__ inline void slot_sums(const float* cs, int piece, int H, KeyOf key_of, float* dot, float* nk) {
#pragma clang fp contract(off)
  constexpr int LV = ilog2(HP);
  float sd[LV + 1], sn[LV + 1];
  float vd = 0.f, vn = 0.f;
#pragma unroll
  for (int h = 0; h < HP; ++h) {
    vd = 0.f; vn = 0.f;                                // heads beyond H are the tree's zero padding
    if (h < H) {
      float k8[8];
      key_of(h, k8);
      const float4 c0 = *(const float4*)(cs + h * 64 + piece * 8), c1 = *(const float4*)(cs + h * 64 + piece * 8 + 4);
      const float cc[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
      float p[8], q[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) { p[i] = k8[i] * cc[i]; q[i] = k8[i] * k8[i]; }
      vd = tree8_lanes8(p);
      vn = tree8_lanes8(q);
    }
#pragma unroll
    for (int lvl = 0; lvl < LV; ++lvl) {
      if ((h >> lvl) & 1) { vd = sd[lvl] + vd; vn = sn[lvl] + vn; }
      else { sd[lvl] = vd; sn[lvl] = vn; break; }
    }
  }
  *dot = vd; *nk = vn;
}

constexpr int kDivHeadBatch = 16;              // head rows of a round requested together (64 registers)

// Workgroup `block` of `blocks` of a layer's pass; cs: HP * 64 floats of LDS.
template <int HP>
__device__ inline void diversity_pass(const Geom& g, char* kv, char* meta, int layer, int block, int blocks, int n_hist, float* cs) {
#pragma clang fp contract(off)
  char* mb = layer_meta(meta, g, layer);
  const uint8_t* flags = (const uint8_t*)(mb + g.off_flags);
  const float* cvec = (const float*)(mb + g.off_cvec);   // the fp32 centroid the frame's append left
  float* dval = (float*)(mb + g.off_dval);
  const char* K = layer_k(kv, g, layer);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sl = lane >> 3, piece = lane & 7;
  const int H = g.H;
  for (int i = threadIdx.x; i < H * 64; i += kDivThreads) cs[i] = cvec[i];
  __syncthreads();

  // |c|^2 by the same tree (the centroid plays the key)
  float nc, unused;
  slot_sums<HP>(cs, piece, H, [&](int h, float (&k8)[8]) {
#pragma unroll
    for (int i = 0; i < 8; ++i) k8[i] = cs[h * 64 + piece * 8 + i];
  }, &nc, &unused);
  const float root_nc = __builtin_sqrtf(nc);

  // minimum and maximum of the d_i this wave writes: the selection normalises with them and reads
  // one pair per wave of this pass instead of every d_i
  float d_lo = __builtin_inff(), d_hi = -__builtin_inff();
  const int stride = blocks * kDivWaves * 8;
  for (int s0 = (block * kDivWaves + wave) * 8; s0 < n_hist; s0 += stride) {
    const int slot = s0 + sl;
    const int sc = min(slot, n_hist - 1);
    const uint8_t fl = flags[sc];
    const char* row0 = K + (size_t)sc * 128 + piece * 16;
    float dot, nk;
    if constexpr (HP <= kDivHeadBatch) {
      // every load is issued (heads beyond H repeat the last one): no branch between the loads, so
      // all of them are in flight before the first wait
      uint4 w[HP];
#pragma unroll
      for (int h = 0; h < HP; ++h) w[h] = *(const uint4*)(row0 + (size_t)min(h, H - 1) * g.cap * 128);
      slot_sums<HP>(cs, piece, H, [&](int h, float (&k8)[8]) { unpack_halfs(w[h], k8); }, &dot, &nk);
    } else {
      slot_sums<HP>(cs, piece, H, [&](int h, float (&k8)[8]) {
        unpack_halfs(*(const uint4*)(row0 + (size_t)h * g.cap * 128), k8);
      }, &dot, &nk);
    }
    if (piece == 0 && slot < n_hist && fl == 0) {
      const float den = __builtin_sqrtf(nk) * root_nc;
      const float cosv = den == 0.f ? 0.f : dot / den;
      const float dv = 1.0f - cosv;
      dval[slot] = dv;
      d_lo = fminf(d_lo, dv); d_hi = fmaxf(d_hi, dv);
    }
  }
  // only the first lane of each slot's eight holds values: three butterfly steps across the slots,
  // one pair per wave (no workgroup barrier: a workgroup lives for a few slot groups only)
#pragma unroll
  for (int off = 8; off < 64; off *= 2) {
    d_lo = fminf(d_lo, __shfl_xor(d_lo, off, 64));
    d_hi = fmaxf(d_hi, __shfl_xor(d_hi, off, 64));
  }
  if (lane == 0) ((float2*)(mb + g.off_dpart))[block * kDivWaves + wave] = make_float2(d_lo, d_hi);
}

}  // namespace ovggt
