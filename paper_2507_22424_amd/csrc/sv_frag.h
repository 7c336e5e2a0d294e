// Matrix-core fragments: types, sizes and the conversions between the storage formats and bf16
// operands that the products and the attention share.
#ifndef SV_FRAG_H
#define SV_FRAG_H

#include <type_traits>

#include "sv_internal.h"

namespace sv {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));

constexpr int kFragRows = 32;    // weight rows per fragment and per tile (MFMA N)
constexpr int kFragK = 16;       // k-values per fragment (MFMA K)
constexpr int kXcds = 8, kCusPerXcd = 32;
constexpr int kCntStride = 32;     // 32-bit words per group's counters: a 128-byte line of its own
// Groups of workgroups that share an output in one launch, at most, over all XCDs of a device: a product with
// more is not split along K.  (8192 x 28672 at 18464 rows asks for 3712; up to 1024 rows the largest of many shapes asks for 608.)
constexpr int kMaxGroups = 4096;

enum { EPI_QKV = 0, EPI_RESID = 1, EPI_SWIGLU = 2, EPI_OUT = 3 };
enum { PACK_PLAIN = 0, PACK_PAIR16_HEAD = 1, PACK_PAIR16_GU = 2 };

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

// Two floats -> packed bf16 (round to nearest even; one v_cvt_pk_bf16_f32 on gfx950).
__device__ inline uint32_t pack_bf16x2(float a, float b) {
  const f32x2_t v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}
__device__ inline float bf16_lo_f32(uint32_t packed) { return __uint_as_float(packed << 16); }
__device__ inline float bf16_hi_f32(uint32_t packed) { return __uint_as_float(packed & 0xffff0000u); }

// four float32 values -> 8 bytes of hi parts, 8 bytes of lo parts
__device__ inline void split4(const f32x4_t v, uint2& hi, uint2& lo) {
  hi.x = pack_bf16x2(v[0], v[1]);
  hi.y = pack_bf16x2(v[2], v[3]);
  lo.x = pack_bf16x2(v[0] - bf16_lo_f32(hi.x), v[1] - bf16_hi_f32(hi.x));
  lo.y = pack_bf16x2(v[2] - bf16_lo_f32(hi.y), v[3] - bf16_hi_f32(hi.y));
}

// Four consecutive k-values (k a multiple of 4) of activation row m -> fragments of a K = 16 * nks
// operand: [k-step][row block][hi, lo][64 lanes] x 16 bytes.
__device__ inline void store_frag4(uint4* xs, int n_rb, int m, int k, const f32x4_t v) {
  uint2 hi, lo;
  split4(v, hi, lo);
  uint2* dst = reinterpret_cast<uint2*>(xs + ((size_t)(k >> 4) * n_rb + (m >> 5)) * 128 + (m & 31) + 32 * ((k >> 3) & 1)) + ((k >> 2) & 1);
  dst[0] = hi;
  dst[128] = lo;
}

// x * sigmoid(x) with the hardware exponential and reciprocal (1 ulp each)
__device__ inline float silu_fast(float x) {
  return x * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * x));
}

// The bf16 operand of k-step kk out of one weight load of a lane (of up to 16 bytes: 1, 2 or 4 k-steps).
//   WF = 0: the load is the operand.
//   WF = 1: 8 bytes of E4M3 codes per k-step, one hardware conversion per pair (gfx950; scale 1).  Exact, every E4M3
//           value is a bf16 value.
//   WF = 2: integers -8 .. 7 in 4-bit two's complement, one 32-bit word per k-step, value i of a word in bits
//           4i .. 4i+3.  v_cvt_off_f32_i4 takes the low four bits of a byte and gives a sixteenth of the integer; the
//           sixteen is in the packed row scales.  Exact.  (Bit-field extract, integer conversion and a flip of the
//           top bits, as before, are 21 instead of 13 instructions for eight weights, next to four matrix
//           instructions at up to 64 rows.)
constexpr float kInt4Unit = 16.0f;
// Word j (two weights) of it; odd: scratch that the words 0 .. 3 of an operand share (int4: the odd nibbles).
template <int WF, typename T>
__device__ inline uint32_t weight_word(const T raw, int kk, int j, unsigned& odd) {
  if constexpr (WF == 1)        // (the half of the word is an immediate)
    return j & 1 ? __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw[2 * kk + j / 2], 1.0f, true))
                 : __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw[2 * kk + j / 2], 1.0f, false));
  if constexpr (WF == 2) {
    if (j == 0) {
      odd = raw[kk] >> 4;
      asm("" : "+v"(odd));      // (else each odd nibble is extracted on its own)
    }
    return pack_bf16x2(__builtin_amdgcn_cvt_off_f32_i4((int)(raw[kk] >> (8 * j)) & 0xff), __builtin_amdgcn_cvt_off_f32_i4((int)(odd >> (8 * j)) & 0xff));
  }
  return raw[j];
}
template <int WF, typename T>
__device__ inline bf16x8_t weight_operand(const T raw, int kk) {
  u32x4_t o;
  unsigned odd = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) o[j] = weight_word<WF>(raw, kk, j, odd);
  return __builtin_bit_cast(bf16x8_t, o);
}

// Scheduling barrier that matrix instructions do not cross and everything else does.
constexpr int kMfmaOrder = 0x2 | 0x4 | 0x10 | 0x20 | 0x40 | 0x80 | 0x100 | 0x200 | 0x400;

// XCD (accelerator complex die) this wave runs on: bits 3:0 of the XCC_ID hardware register.
__device__ inline int xcd_actual(int n_xcd) {
  return (int)(__builtin_amdgcn_s_getreg((4 - 1) << 11 | 0 << 6 | 20) & 0xf) % n_xcd;
}

}  // namespace sv
#endif
