// Cache maintenance kernels: zero fill, append (paper Eq. 2) and the in-place
// hole-fill compaction that follows Eq. 8's selection.  All are pure copies,
// bound by HBM bandwidth; every lane moves 16-byte pieces of 128-byte-or-longer
// contiguous rows.
#include "append_parts.h"

namespace ovggt {

// --------------------------------------------------------------------------
__global__ void __launch_bounds__(256) fill_zero_kernel(uint4* p, size_t n16) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  const uint4 z = {0u, 0u, 0u, 0u};
  for (; i < n16; i += stride) p[i] = z;
}

hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s) {
  const size_t n16 = bytes / 16;        // buffers are sized in multiples of 256 bytes
  if (n16 == 0) return hipSuccess;
  size_t blocks = (n16 + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)blocks), dim3(256), 0, s, (uint4*)p, n16);
  return hipGetLastError();
}

// --------------------------------------------------------------------------
// Timing aid: one wave that returns after `ticks` ticks of the constant-rate wall clock (or after
// a fixed number of polls, whichever comes first, so the kernel ends under all circumstances).
__global__ void __launch_bounds__(64) spin_kernel(unsigned long long ticks) {
  const unsigned long long t0 = wall_clock64();
  for (int i = 0; i < (1 << 22); ++i) {
    if (wall_clock64() - t0 >= ticks) break;
    __builtin_amdgcn_s_sleep(8);
  }
}

hipError_t launch_spin(unsigned long long ticks, hipStream_t s) {
  hipLaunchKernelGGL(spin_kernel, dim3(1), dim3(64), 0, s, ticks);
  return hipGetLastError();
}

// --------------------------------------------------------------------------
// Append.  Input rows are token-major [M][H][d]; the cache is head-major
// [H][cap][d].  One thread per 16-byte piece of K and of V.
template <bool MOVES>
__global__ void __launch_bounds__(256)
append_kernel(Geom g, char* kv, char* meta, int layer0, const char* k_new, const char* v_new, int n) {
  const int layer = layer0 + blockIdx.y;
  if (g.hybrid && blockIdx.x == 0) centroid_to_fp32(g, meta, layer, threadIdx.x, blockDim.x);
  const int row_bytes = g.d * g.esize;             // 128 (bf16) or 256 (f32)
  const int pieces = row_bytes / 16;
  const size_t per_layer_in = (size_t)g.M * g.H * row_bytes;
  const size_t total = (size_t)g.M * g.H * pieces;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int piece = (int)(i % pieces);
  const int h = (int)((i / pieces) % g.H);
  const int m = (int)(i / ((size_t)pieces * g.H));
  append_piece<MOVES>(g, kv, meta, layer, k_new + (size_t)blockIdx.y * per_layer_in, v_new + (size_t)blockIdx.y * per_layer_in, h, m, piece, n);
}

hipError_t launch_append(const Geom& g, char* kv, char* meta, int layer0, int nl,
                         const void* k_new, const void* v_new, int n, bool apply_moves, hipStream_t s) {
  const size_t total = (size_t)g.M * g.H * (g.d * g.esize / 16);
  dim3 grid((unsigned)((total + 255) / 256), (unsigned)nl);
  if (apply_moves && n == g.B)
    hipLaunchKernelGGL(append_kernel<true>, grid, dim3(256), 0, s, g, kv, meta, layer0,
                       (const char*)k_new, (const char*)v_new, n);
  else if (apply_moves)
    return hipErrorInvalidValue;                     // a pending compaction implies a full cache
  else
    hipLaunchKernelGGL(append_kernel<false>, grid, dim3(256), 0, s, g, kv, meta, layer0,
                       (const char*)k_new, (const char*)v_new, n);
  return hipGetLastError();
}

// --------------------------------------------------------------------------
// Compaction.  Workgroup r of a layer moves entry src[r] -> dst[r]: 2*H rows of
// d elements (K and V of every head) plus id, score and flag.  Destinations are
// slots below B, sources slots at or above B, so no ordering between moves is
// needed.  Workgroups beyond the list length exit at once.
__global__ void __launch_bounds__(256)
compact_kernel(Geom g, char* kv, char* meta, int layer0) {
  const int layer = layer0 + blockIdx.y;
  char* mb = layer_meta(meta, g, layer);
  const Ctrl* ctrl = (const Ctrl*)(mb + g.off_ctrl);
  const uint32_t n_moves = ctrl->n_moves;
  const uint32_t r = blockIdx.x;
  if (r >= n_moves) return;
  const uint32_t dst = ((const uint32_t*)(mb + g.off_mvdst))[r];
  const uint32_t src = ((const uint32_t*)(mb + g.off_mvsrc))[r];
  if (dst >= (uint32_t)g.B || src < (uint32_t)g.B || src >= (uint32_t)g.cap) return;   // never out of bounds
  const int row_bytes = g.d * g.esize;
  const int pieces = row_bytes / 16;
  const int total = 2 * g.H * pieces;
  char* kbase = layer_k(kv, g, layer);
  const size_t v_off = (size_t)g.H * g.cap * row_bytes;
  for (int i = threadIdx.x; i < total; i += blockDim.x) {
    const int piece = i % pieces;
    const int h = (i / pieces) % g.H;
    const int isv = i / (pieces * g.H);
    char* base = kbase + (isv ? v_off : 0) + (size_t)h * g.cap * row_bytes + piece * 16;
    *(uint4*)(base + (size_t)dst * row_bytes) = *(const uint4*)(base + (size_t)src * row_bytes);
  }
  if (threadIdx.x == 0) {
    uint32_t* ids = (uint32_t*)(mb + g.off_ids);
    float* ss = (float*)(mb + g.off_ss);
    uint8_t* fl = (uint8_t*)(mb + g.off_flags);
    ids[dst] = ids[src];
    ss[dst] = ss[src];
    fl[dst] = fl[src];
  }
}

// --------------------------------------------------------------------------
// Sec. 3.3: protection granted or withdrawn for resident tokens of one frame.  One thread per
// slot: ids in [gid_lo, gid_lo + M) whose mask byte is set (no mask: all of them) take the flag.
__global__ void __launch_bounds__(256)
set_protect_kernel(Geom g, char* meta, int layer0, int n, uint32_t gid_lo, const uint8_t* mask, int on) {
  char* mb = layer_meta(meta, g, layer0 + blockIdx.y);
  const int slot = blockIdx.x * blockDim.x + threadIdx.x;
  if (slot >= n) return;
  const uint32_t local = ((const uint32_t*)(mb + g.off_ids))[slot] - gid_lo;     // wraps for ids below gid_lo
  if (local >= (uint32_t)g.M) return;
  if (mask && mask[local] == 0) return;
  ((uint8_t*)(mb + g.off_flags))[slot] = on ? 1 : 0;
}

hipError_t launch_set_protect(const Geom& g, char* meta, int layer0, int nl, int n, uint32_t gid_lo,
                              const uint8_t* mask, int on, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  dim3 grid((unsigned)((n + 255) / 256), (unsigned)nl);
  hipLaunchKernelGGL(set_protect_kernel, grid, dim3(256), 0, s, g, meta, layer0, n, gid_lo, mask, on);
  return hipGetLastError();
}

// --------------------------------------------------------------------------
// Checkpoints of bf16 handles.  The host's layout is token-major bf16 [n][H][d], the cache is
// head-major half; conversion and transposition run here, through a staging area in device memory,
// so that K and V cross the bus in whole buffers.  One thread per 16-byte piece, consecutive in the
// staging area (128-byte runs in the cache); a pure copy, bound by HBM and dwarfed by the bus.
// 4096 tokens of 16 heads, out and in again and one frame on top: 131.6 ms with both done on the
// host, 1.84 ms like this, of which 1.64 ms are four copies of 8.4 MB from and to pageable memory.
__device__ inline uint32_t half_to_bf16_bits(uint32_t h) {
  if ((h & 0x7FFFu) > 0x7C00u) return 0x7FC0u | (h & 0x8000u);         // NaN stays NaN
  uint32_t u = __float_as_uint(__half2float(__ushort_as_half((unsigned short)h)));
  u += 0x7FFFu + ((u >> 16) & 1u);                                     // round to nearest even
  return u >> 16;
}
__device__ inline uint32_t bf16_to_half_bits(uint32_t b) {
  const float f = __uint_as_float(b << 16);
  if (f != f) return 0x7E00u;
  return __half_as_ushort(__float2half_rn(fminf(fmaxf(f, -65504.f), 65504.f)));
}

// Slots [slot0, slot0 + rows) of one layer; stage: K rows, then V rows.
template <bool TO_STAGE>
__global__ void __launch_bounds__(256)
checkpoint_kernel(Geom g, char* kv, int layer, int slot0, int rows, char* stage) {
  const size_t total = (size_t)rows * g.H * 8;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int piece = (int)(i & 7);
  const size_t rh = i >> 3;
  const size_t row = rh / g.H;
  const int h = (int)(rh - row * g.H);
  char* cache = (blockIdx.y ? layer_v(kv, g, layer) : layer_k(kv, g, layer)) + ((size_t)h * g.cap + slot0 + row) * 128 + piece * 16;
  char* host = stage + (blockIdx.y ? total * 16 : 0) + i * 16;
  const uint4 w = *(const uint4*)(TO_STAGE ? cache : host);
  uint32_t x[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t lo = x[j] & 0xFFFFu, hi = x[j] >> 16;
    x[j] = TO_STAGE ? half_to_bf16_bits(lo) | half_to_bf16_bits(hi) << 16 : bf16_to_half_bits(lo) | bf16_to_half_bits(hi) << 16;
  }
  *(uint4*)(TO_STAGE ? host : cache) = uint4{x[0], x[1], x[2], x[3]};
}

hipError_t launch_checkpoint(const Geom& g, char* kv, int layer, int slot0, int rows, char* stage, bool to_stage, hipStream_t s) {
  const size_t total = (size_t)rows * g.H * 8;
  dim3 grid((unsigned)((total + 255) / 256), 2);
  if (to_stage) hipLaunchKernelGGL(checkpoint_kernel<true>, grid, dim3(256), 0, s, g, kv, layer, slot0, rows, stage);
  else hipLaunchKernelGGL(checkpoint_kernel<false>, grid, dim3(256), 0, s, g, kv, layer, slot0, rows, stage);
  return hipGetLastError();
}

hipError_t launch_compact(const Geom& g, char* kv, char* meta, int layer0, int nl, hipStream_t s) {
  dim3 grid((unsigned)g.M, (unsigned)nl);      // at most M entries move per frame
  hipLaunchKernelGGL(compact_kernel, grid, dim3(256), 0, s, g, kv, meta, layer0);
  return hipGetLastError();
}

}  // namespace ovggt
