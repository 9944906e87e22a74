// The append (paper Eq. 2) of one 16-byte piece of a token's K and V, for the kernel that appends a frame and for the
// attention kernel of the smallest launches, which appends its own head's rows.
#pragma once
#include "ovggt_internal.h"
#include "../../include/ovggt.h"
#include <hip/hip_fp16.h>

namespace ovggt {

// bf16 handles keep K and V as IEEE binary16: both attention products then run
// on the f16 MFMA, P*V with 11-bit softmax weights instead of 8-bit ones and
// Q*K^T with queries that carry the softmax scale at 11 bits.  Values beyond the
// half range saturate (and are reported), values below 2^-14 round to the half
// subnormal grid.
__device__ inline uint32_t bf16pair_to_half(uint32_t w, bool* clipped) {
  float a = __uint_as_float(w << 16), b = __uint_as_float(w & 0xFFFF0000u);
  if (!(fabsf(a) <= 65504.f)) { *clipped = true; a = a != a ? a : copysignf(65504.f, a); }
  if (!(fabsf(b) <= 65504.f)) { *clipped = true; b = b != b ? b : copysignf(65504.f, b); }
  const __half2 h = __floats2half2_rn(a, b);
  return *(const uint32_t*)&h;
}

// Hybrid scoring: the frame's diversity pass wants the centroid in fp32.  The running sum (64-bit
// integers in units of 2^-24, final since the previous frame's update) is rounded integer -> fp64
// -> fp32, each to nearest even, and scaled by 2^-24 exactly.
__device__ inline void centroid_to_fp32(const Geom& g, char* meta, int layer, int first, int step) {
  char* mb = layer_meta(meta, g, layer);
  const long long* csum = (const long long*)(mb + g.off_csum);
  float* cvec = (float*)(mb + g.off_cvec);
  for (int e = first; e < g.H * g.d; e += step) cvec[e] = (float)(double)csum[e] * 5.9604644775390625e-8f;
}

// k_new, v_new: the layer's rows, token-major [M][H][d]; the cache is head-major [H][cap][d].
// MOVES: the compaction that follows the previous frame's selection has not been applied yet
// (n == B).  Its sources are exactly the slots this frame overwrites, so the thread that owns a
// piece of slot B + m first carries the piece it finds there to the slot the selection assigned
// (below B, disjoint from every slot written here), then stores the new one: no other thread
// reads or writes either location.
template <bool MOVES>
__device__ inline void append_piece(const Geom& g, char* kv, char* meta, int layer, const char* k_new, const char* v_new, int h, int m,
                                    int piece, int n) {
  const int row_bytes = g.d * g.esize;             // 128 (bf16) or 256 (f32)
  const size_t src = ((size_t)m * g.H + h) * row_bytes + piece * 16;
  const size_t dst = ((size_t)h * g.cap + (n + m)) * row_bytes + piece * 16;
  uint4 kk = *(const uint4*)(k_new + src);
  uint4 vv = *(const uint4*)(v_new + src);
  char* mb = layer_meta(meta, g, layer);
  if constexpr (MOVES) {
    // the entry that sits in the slot is fetched together with its destination, not after it: one
    // round trip to memory less on the path of every moved piece
    const uint4 ok = *(const uint4*)(layer_k(kv, g, layer) + dst);
    const uint4 ov = *(const uint4*)(layer_v(kv, g, layer) + dst);
    const uint32_t to = ((const uint32_t*)(mb + g.off_mvmap))[m];
    if (to < (uint32_t)g.B) {                        // kNoMove, or anything out of range: nothing to carry
      const size_t mv = ((size_t)h * g.cap + to) * row_bytes + piece * 16;
      uint32_t id = 0; float sc = 0.f; uint8_t fl = 0;
      const bool meta_thread = h == 0 && piece == 0;
      if (meta_thread) {
        id = ((const uint32_t*)(mb + g.off_ids))[n + m];
        sc = ((const float*)(mb + g.off_ss))[n + m];
        fl = ((const uint8_t*)(mb + g.off_flags))[n + m];
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the old contents are in registers before anything is stored
      *(uint4*)(layer_k(kv, g, layer) + mv) = ok;
      *(uint4*)(layer_v(kv, g, layer) + mv) = ov;
      if (meta_thread) {
        ((uint32_t*)(mb + g.off_ids))[to] = id;
        ((float*)(mb + g.off_ss))[to] = sc;
        ((uint8_t*)(mb + g.off_flags))[to] = fl;
      }
    }
  }
  if (g.esize == 2) {
    bool clipped = false;
    kk.x = bf16pair_to_half(kk.x, &clipped); kk.y = bf16pair_to_half(kk.y, &clipped);
    kk.z = bf16pair_to_half(kk.z, &clipped); kk.w = bf16pair_to_half(kk.w, &clipped);
    vv.x = bf16pair_to_half(vv.x, &clipped); vv.y = bf16pair_to_half(vv.y, &clipped);
    vv.z = bf16pair_to_half(vv.z, &clipped); vv.w = bf16pair_to_half(vv.w, &clipped);
    if (clipped) atomicOr(&((Ctrl*)(mb + g.off_ctrl))->status, (uint32_t)OVGGT_STATUS_VRANGE);
  }
  *(uint4*)(layer_k(kv, g, layer) + dst) = kk;
  *(uint4*)(layer_v(kv, g, layer) + dst) = vv;
  if (h == 0 && piece == 0) {
    // ids t*M + i (Eq. 2's arrival order): the frame's first id lives in the control block, where the
    // previous frame's selection left it, so the launch is the same for every frame (graph replay)
    const uint32_t gid0 = ((const Ctrl*)(mb + g.off_ctrl))->gid_next;
    ((uint32_t*)(mb + g.off_ids))[n + m] = gid0 + (uint32_t)m;
    ((float*)(mb + g.off_ss))[n + m] = 0.f;
    ((uint8_t*)(mb + g.off_flags))[n + m] = 0;
  }
}


}  // namespace ovggt
