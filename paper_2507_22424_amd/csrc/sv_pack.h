// Load-time packers: weight matrices into the order the kernels stream them.
//
// A matrix [rows, K] becomes loads of 1 KiB: 32 rows x 16 k-values of bf16 (exactly one operand of
// v_mfma_f32_32x32x16_bf16: lane l holds the 8 consecutive k-values (l / 32) * 8 .. + 7 of row l % 32), or
// the codes of two (E4M3) or four (int4) consecutive k-steps, 16 bytes per lane either way.  The loads are
// stored load-major: [K / (16, 32 or 64)][rows / 32 tiles] - at one k-step all tiles are neighbours.
#ifndef SV_PACK_H
#define SV_PACK_H

#include "sv_frag.h"

namespace sv {

// Row permutation:
//   PACK_PLAIN        dst row = off + n
//   PACK_PAIR16_HEAD  heads of 128 rows; row d of a head goes to 32*((d%64)/16) + 16*(d/64) + d%16
//                     (a tile holds 16 rows j and their rotary partners j + 64)
//   PACK_PAIR16_GU    dst row = 32*(n/16) + off + n%16   (off = 0 gate, 16 up)
__device__ inline int packed_row(int n_src, int mode, int off) {
  if (mode == PACK_PAIR16_HEAD) {
    const int d = n_src % 128;
    return off + (n_src - d) + 32 * ((d % 64) / 16) + 16 * (d / 64) + d % 16;
  }
  if (mode == PACK_PAIR16_GU) return 32 * (n_src / 16) + off + n_src % 16;
  return off + n_src;
}

// V = 8 consecutive k-values of a row as stored in `src` [rows][K / 8]: uint4 (bf16), uint2 (E4M3), uint32_t
// (int4, even k in the low nibble).  WF = 0, 1, 2: a lane's 16 bytes carry 1, 2, 4 k-steps.  A workgroup
// moves 32 source rows x 256 k-values through LDS: reads run along k, writes along the rows of a load.
// grid = (rows / 32, K / 256), block = 256.
template <typename V, int WF>
__global__ __launch_bounds__(256) void pack_rows(const V* __restrict__ src, V* __restrict__ dst, int K, int n_tiles,
                                                 int mode, int off) {
  __shared__ V box[32][33];
  const int r0 = blockIdx.x * 32, k0 = blockIdx.y * 32;      // first row, first 8-wide k chunk
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int c = it * 256 + threadIdx.x;
    box[c >> 5][c & 31] = src[(size_t)(r0 + (c >> 5)) * (K / 8) + k0 + (c & 31)];
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int c = it * 256 + threadIdx.x;
    const int r = c & 31, kc = k0 + (c >> 5);
    const int n = packed_row(r0 + r, mode, off);
    const size_t load = (size_t)(kc >> (1 + WF)) * n_tiles + n / kFragRows;
    const int lane = n % kFragRows + 32 * (kc & 1), step = (kc >> 1) & ((1 << WF) - 1);
    V v = box[r][c >> 5];
    if constexpr (WF == 2) v ^= 0x88888888u;                 // code c (c - 8) -> 4-bit two's complement
    dst[((load * 64 + lane) << WF) + step] = v;
  }
}

// unit: what a code of 1 is multiplied as, inverted (a power of two)
__global__ void pack_row_scales(const float* __restrict__ src, float* __restrict__ dst, int rows,
                                int mode, int off, float unit) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < rows) dst[packed_row(i, mode, off)] = src[i] * unit;
}

}  // namespace sv
#endif
