// Kernels around the products: the row argmax, float32 rows to fragments, packers, and a measurement aid.
#ifndef SV_KERNELS_H
#define SV_KERNELS_H

#include "sv_frag.h"
#include "sv_internal.h"

namespace sv {

// ---------------------------------------------------------------------------------------
// Greedy choice per row: index of the largest logit, the lowest index on exact ties (NaN never wins).
// NT threads per row, eight loads in flight per thread: as few round trips as the row allows (60 rows of
// 32000: 17.1 us with 256 threads).  logits_out: also a copy of the row (NULL: none).
// grid = rows, block = NT.
// ---------------------------------------------------------------------------------------
template <int NT>
__global__ __launch_bounds__(NT) void argmax_rows_wide(const float* __restrict__ logits, int n,
                                                        int token_lo, int32_t* __restrict__ out,
                                                        float* __restrict__ logits_out) {
  __shared__ float s_best[NT / 64];
  __shared__ int s_bi[NT / 64];
  const size_t row = blockIdx.x;
  const float* src = logits + row * n;
  float best = -INFINITY;
  int bi = 0x7fffffff;
  for (int i0 = threadIdx.x; i0 < n; i0 += 8 * NT) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = i0 + NT * u < n ? src[i0 + NT * u] : -INFINITY;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = i0 + NT * u;
      if (i >= n) continue;
      if (logits_out) logits_out[row * n + i] = v[u];
      if (v[u] > best || (v[u] == best && i < bi)) {
        best = v[u];
        bi = i;
      }
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const float ov = __shfl_xor(best, off, kWave);
    const int oi = __shfl_xor(bi, off, kWave);
    if (ov > best || (ov == best && oi < bi)) {
      best = ov;
      bi = oi;
    }
  }
  if ((threadIdx.x & 63) == 0) {
    s_best[threadIdx.x >> 6] = best;
    s_bi[threadIdx.x >> 6] = bi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < NT / 64; ++w)
      if (s_best[w] > best || (s_best[w] == best && s_bi[w] < bi)) {
        best = s_best[w];
        bi = s_bi[w];
      }
    out[row] = token_lo + (bi == 0x7fffffff ? 0 : bi);
  }
}

// ---------------------------------------------------------------------------------------
// Measurement aid: reads a buffer once the way the GEMM streams weights (non-temporal 16-byte
// loads, 1 KiB per wave and instruction, 8 KiB per wave in flight) and discards the data.
// grid = any, block = 256.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void stream_read_kernel(const u32x4_t* __restrict__ p, size_t n_vec,
                                                          u32x4_t* __restrict__ sink) {
  typedef const __attribute__((address_space(1))) u32x4_t* gptr_t;
  const gptr_t g = (gptr_t)p;
  const size_t lane = threadIdx.x & 63;
  const size_t n_waves = (size_t)gridDim.x * 4;
  u32x4_t acc = {0u, 0u, 0u, 0u};
  for (size_t blk = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6); blk * 512 < n_vec; blk += n_waves) {
    u32x4_t v[8];
#pragma unroll
    for (int f = 0; f < 8; ++f) {
      const size_t i = blk * 512 + f * 64 + lane;
      v[f] = __builtin_nontemporal_load(g + (i < n_vec ? i : n_vec - 1));
    }
#pragma unroll
    for (int f = 0; f < 8; ++f) acc ^= v[f];
  }
  if (acc[0] == 0x9e3779b9u && acc[1] == 0x7f4a7c15u && acc[2] == 0xf39cc060u) *sink = acc;   // keeps the loads
}

// ---- float32 rows -> fragments -----------------------------------------------------------------
// hi + lo bf16 fragments of x * gain (gain may be NULL) and partial sums of x^2, one plane per 256
// k-values ([K / 256][m_pad], NULL: none).  Rows beyond M become zeros.  grid = (row blocks * 4, K / 256),
// block = 256: one thread turns 8 consecutive k-values of a row into the 16 bytes a lane holds of a
// fragment, a workgroup 8 rows (a launch is one round trip to memory: 60 x 4096 in 4.9 us, 5.9 with 32
// rows per workgroup).
__global__ __launch_bounds__(256) void split_gain_kernel(const float* __restrict__ x, const float* __restrict__ gain,
                                                         int M, int K, int m_pad, int n_rb,
                                                         uint4* __restrict__ Xs, float* __restrict__ ssq) {
  const int mb = blockIdx.x >> 2, kc = blockIdx.y;
  const int r = (blockIdx.x & 3) * 8 + (threadIdx.x >> 5), kq = threadIdx.x & 31;   // row inside the block, 8-wide k chunk inside the 256
  const int row = mb * 32 + r, k = kc * 256 + kq * 8;
  f32x4_t v0 = {0.f, 0.f, 0.f, 0.f}, v1 = v0, g0 = {1.f, 1.f, 1.f, 1.f}, g1 = g0;
  if (gain) {
    g0 = *reinterpret_cast<const f32x4_t*>(gain + k);
    g1 = *reinterpret_cast<const f32x4_t*>(gain + k + 4);
  }
  if (row < M) {
    v0 = *reinterpret_cast<const f32x4_t*>(x + (size_t)row * K + k);
    v1 = *reinterpret_cast<const f32x4_t*>(x + (size_t)row * K + k + 4);
  }
  if (ssq) {
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) s += v0[e] * v0[e] + v1[e] * v1[e];
#pragma unroll
    for (int off = 16; off > 0; off >>= 1) s += __shfl_xor(s, off, kWave);
    if (kq == 0) ssq[(size_t)kc * m_pad + row] = s;
  }
  uint2 h0, l0, h1, l1;
  split4(v0 * g0, h0, l0);
  split4(v1 * g1, h1, l1);
  uint4* dst = Xs + ((size_t)(k / kFragK) * n_rb + mb) * 128 + r + 32 * (kq & 1);
  dst[0] = make_uint4(h0.x, h0.y, h1.x, h1.y);
  dst[64] = make_uint4(l0.x, l0.y, l1.x, l1.y);
}

// ---------------------------------------------------------------------------------------
// Packers (load time).  pack_gain widens a gain vector to float32; pack_rows_plain copies
// a [rows, K] matrix behind `row_off` rows of the destination.
// ---------------------------------------------------------------------------------------
template <typename T>
__global__ void pack_gain(const T* __restrict__ src, float* __restrict__ dst, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = to_f32(src[i]);
}

template <typename T>
__global__ void pack_rows_plain(const T* __restrict__ src, T* __restrict__ dst, size_t n_elems,
                                size_t dst_off) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_elems) dst[dst_off + i] = src[i];
}

}  // namespace sv
#endif
