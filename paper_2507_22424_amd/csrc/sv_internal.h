// Internal helpers shared by the kernels of libspecvla_verify (gfx950 only).
#ifndef SV_INTERNAL_H
#define SV_INTERNAL_H

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "specvla_verify.h"

namespace sv {

constexpr int kWave = 64;           // CDNA wavefront
constexpr int kRowPad = 64;         // float32 buffers and logits are laid out for a multiple of this many rows
constexpr size_t kAlign = 256;      // alignment of every region inside packed blobs / workspace

// bfloat16 stored as its 16 bits.
struct bf16_t {
  uint16_t bits;
};

__host__ __device__ inline float to_f32(bf16_t v) {
  union { uint32_t u; float f; } c;
  c.u = (uint32_t)v.bits << 16;
  return c.f;
}
__host__ __device__ inline float to_f32(float v) { return v; }

__host__ __device__ inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
__host__ __device__ inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Sum over the 64 lanes of a wavefront; every lane gets the total.
__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

// Where the pieces of a packed layer live (bytes from the start of the blob).
struct PackedLayout {
  size_t g1, g2, wqkv, wo, wgu, wd, total;
  size_t sqkv, so, sgu, sd;      // SV_BF16_W8 / SV_BF16_W4: float32 row scales in packed row order
};

inline PackedLayout packed_layout(const sv_model_cfg& c) {
  // half bytes per matrix element: float32 8, bf16 4, E4M3 2, int4 1
  const size_t eh = c.dtype == SV_F32 ? 8 : (c.dtype == SV_BF16_W8 ? 2 : (c.dtype == SV_BF16_W4 ? 1 : 4));
  const size_t H = c.hidden, D = (size_t)c.n_heads * c.head_dim, F = c.mlp_dim;
  PackedLayout L;
  size_t o = 0;
  L.g1 = o;   o = align_up(o + H * 4, kAlign);
  L.g2 = o;   o = align_up(o + H * 4, kAlign);
  L.wqkv = o; o = align_up(o + 3 * D * H * eh / 2, kAlign);
  L.wo = o;   o = align_up(o + H * D * eh / 2, kAlign);
  L.wgu = o;  o = align_up(o + 2 * F * H * eh / 2, kAlign);
  L.wd = o;   o = align_up(o + H * F * eh / 2, kAlign);
  L.sqkv = L.so = L.sgu = L.sd = 0;
  if (c.dtype == SV_BF16_W8 || c.dtype == SV_BF16_W4) {
    L.sqkv = o; o = align_up(o + 3 * D * 4, kAlign);
    L.so = o;   o = align_up(o + H * 4, kAlign);
    L.sgu = o;  o = align_up(o + 2 * F * 4, kAlign);
    L.sd = o;   o = align_up(o + H * 4, kAlign);
  }
  L.total = o;
  return L;
}

// Device scratch of one call (bytes from the start of the workspace).
struct WorkspaceLayout {
  size_t q, attn, total;         // float32, both storage types
  // float32 models
  size_t act;
  // bf16 models: counters of the workgroups that share an output (+ status word).  They alone outlive a call
  // and have to be zero when one begins, so their place and extent are the same for every row count, number of
  // scored rows and model: one workspace serves calls of any sizes that fit it, layers and heads.
  size_t counters, counter_bytes;
  // activation fragments of the residual stream, the attention output and the SwiGLU output, partial row sums
  // of x^2, sums that cross workgroups, partial results of a split tree attention
  size_t xs_x, xs_attn, xs_act, ssq, xch, att_part;
  // heads: logits; packed (bf16 models, scored rows a multiple of 32)
  size_t head_logits, head_xs, head_ssq, head_xch;
  int m_pad, n_rb;               // rows as laid out, row blocks of 32
};

}  // namespace sv
#endif
