// What the two attention kernels on 16x16 matrix tiles share: the merge of a workgroup's eight waves,
// and of the parts that several workgroups wrote for one block of queries.
#pragma once
#include "ovggt_internal.h"

namespace ovggt {

typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kPartRows = 16;           // queries of one 16x16 tile
constexpr int kPartWaves = 8;
constexpr int kPartThreads = 64 * kPartWaves;
constexpr int kPartPitch = 68;          // floats per row of the merge area (64 + 4: rows start on different banks)
constexpr int kMaxSplits = 16;          // slot ranges of a block of queries

// A record: the O rows of a part, then their references and weight sums.
constexpr int part_rec_floats(int groups) { return groups * (kPartRows * 64 + 2 * kPartRows); }

// N groups of 16 queries are merged at a time.
template <int N>
struct MergeArea {
  float o[N][kPartWaves][kPartRows][kPartPitch];
  float m[N][kPartWaves][kPartRows], l[N][kPartWaves][kPartRows];
  uint32_t is_last;
};

__device__ inline void store_through(float* p, const f32x4& v) {
  const float2 a = {v[0], v[1]}, b = {v[2], v[3]};
  __hip_atomic_store((unsigned long long*)p, __builtin_bit_cast(unsigned long long, a), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store((unsigned long long*)p + 1, __builtin_bit_cast(unsigned long long, b), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Each of the 8 waves holds, for G groups of 16 queries, unnormalised O^T (lane (l16, gl), accumulator d,
// element i: query l16, output element 16 gl + 4 i + d), the softmax reference m and the weight sum l of
// query l16 (the same in all four gl).  `write(row, piece, o)` receives the normalised elements 4 piece .. +3 of
// query `row` (0 .. 16 G - 1) of the block.  References count powers of 2^UNIT.  With splits > 1 the parts of the block are records at
// recs + s * rec_stride, counted at `arrive` (zero before and after); the last arrival merges them.
template <int UNIT, int G, int N, typename Write>
__device__ inline void merge_and_write(MergeArea<N>& a, const f32x4 (&O)[G][4], const float (&m)[G], const float (&l)[G], int sp,
                                       int splits, uint32_t* arrive, float* recs, size_t rec_stride, Write write) {
  static_assert(G % N == 0 && N <= 2, "32 rows of 16 pieces a pass");
  const int lane = threadIdx.x & 63, l16 = lane & 15, gl = lane >> 4, wave = threadIdx.x >> 6;
  const int row = (int)threadIdx.x >> 4, piece = (int)threadIdx.x & 15;
#pragma unroll
  for (int q0 = 0; q0 < G; q0 += N) {
    if (q0 > 0) __syncthreads();                       // the area is read out
#pragma unroll
    for (int q = 0; q < N; ++q)
      if (gl == 0) { a.m[q][wave][l16] = m[q0 + q]; a.l[q][wave][l16] = l[q0 + q]; }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < N; ++q) {                      // the common reference first, then the rescaled parts
      float mt = a.m[q][0][l16];
#pragma unroll
      for (int w = 1; w < kPartWaves; ++w) mt = fmaxf(mt, a.m[q][w][l16]);
      const float f = __builtin_amdgcn_exp2f(UNIT * (m[q0 + q] - mt));
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const f32x4 o = {O[q0 + q][0][i] * f, O[q0 + q][1][i] * f, O[q0 + q][2][i] * f, O[q0 + q][3][i] * f};
        *(f32x4*)&a.o[q][wave][l16][16 * gl + 4 * i] = o;
      }
    }
    __syncthreads();
    if (row < N * kPartRows) {
      const int q = row / kPartRows, r16 = row & (kPartRows - 1);
      f32x4 o = {0.f, 0.f, 0.f, 0.f};
      float ls = 0.f, mt = a.m[q][0][r16];
#pragma unroll
      for (int w = 1; w < kPartWaves; ++w) mt = fmaxf(mt, a.m[q][w][r16]);
#pragma unroll
      for (int w = 0; w < kPartWaves; ++w) {
        ls += a.l[q][w][r16] * __builtin_amdgcn_exp2f(UNIT * (a.m[q][w][r16] - mt));
        o += *(const f32x4*)&a.o[q][w][r16][4 * piece];
      }
      const int r = q0 * kPartRows + row;
      if (splits == 1) {
        write(r, piece, f32x4{o[0] / ls, o[1] / ls, o[2] / ls, o[3] / ls});
      } else {
        float* rec = recs + (size_t)sp * rec_stride;
        store_through(rec + r * 64 + 4 * piece, o);
        if (piece == 0) {
          __hip_atomic_store(rec + G * kPartRows * 64 + r, mt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(rec + G * kPartRows * 65 + r, ls, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    }
  }
  if (splits == 1) return;
  // Parts are written through to device-coherent memory, so a wave waits for its own stores only;
  // the counter is a relaxed device-scope atomic and the last arrival invalidates its caches.
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    const bool last = __hip_atomic_fetch_add(arrive, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)splits - 1u;
    if (last) {
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      __hip_atomic_store(arrive, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    a.is_last = last ? 1u : 0u;
  }
  __syncthreads();
  if (!a.is_last) return;
#pragma unroll 1
  for (int r = row; r < G * kPartRows; r += kPartThreads / 16) {
    float pm[kMaxSplits], pl[kMaxSplits], mt = -INFINITY, ls = 0.f;
#pragma unroll
    for (int s = 0; s < kMaxSplits; ++s) {             // ranges beyond the last repeat it, with no weight
      const float* rec = recs + (size_t)min(s, splits - 1) * rec_stride + G * kPartRows * 64 + r;
      pm[s] = rec[0];
      pl[s] = rec[G * kPartRows];
    }
#pragma unroll
    for (int s = 0; s < kMaxSplits; ++s) mt = fmaxf(mt, pm[s]);
#pragma unroll
    for (int s = 0; s < kMaxSplits; ++s) {
      pm[s] = s < splits ? __builtin_amdgcn_exp2f(UNIT * (pm[s] - mt)) : 0.f;
      ls += s < splits ? pl[s] * pm[s] : 0.f;
    }
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
    const float* part = recs + r * 64 + 4 * piece;
#pragma unroll
    for (int s0 = 0; s0 < kMaxSplits; s0 += 8) {       // eight parts in flight
      if (s0 >= splits) break;
      f32x4 v[8];
#pragma unroll
      for (int s = 0; s < 8; ++s) v[s] = *(const f32x4*)(part + (size_t)min(s0 + s, splits - 1) * rec_stride);
#pragma unroll
      for (int s = 0; s < 8; ++s)
        if (s0 + s < splits) o += v[s] * pm[s0 + s];
    }
    write(r, piece, f32x4{o[0] / ls, o[1] / ls, o[2] / ls, o[3] / ls});
  }
}

}  // namespace ovggt
