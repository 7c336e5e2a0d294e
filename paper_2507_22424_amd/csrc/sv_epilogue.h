// What the products of a layer do with their sums: RMSNorm scale, row scales of coded weights, RoPE and
// K/V append, residual, SwiGLU, plain output - and the meeting of workgroups that share an output.
//
// All products are computed as W X^T.  Accumulator register r of lane l of a 32 x 32 unit is output
// column 8*(r/4) + 4*(l/32) + r%4 of the weight tile and activation row l%32: a lane holds one row and,
// per register quad (4q .. 4q+3), four consecutive output columns.  The rows of W are permuted at pack
// time so that the partners of a pair (rotary pair j, j + 64 of a head; gate and up of a column) are rows
// j and j + 16 of a tile: quads p and p + 2 of the same lane.  Stores are 16 bytes per lane and the
// fragments of the next product leave as whole 512-byte runs.
#ifndef SV_EPILOGUE_H
#define SV_EPILOGUE_H

#include "sv_frag.h"

namespace sv {

struct EpiArgs {
  int M, n_rb, m_pad;        // activation rows, row blocks of 32, stride of the row-sum planes
  int K;                     // row length the norm averages over
  float eps;
  // EPI_QKV, EPI_SWIGLU, EPI_OUT: RMSNorm of the input, applied to the sums: 1 / rms of row m from
  // n_ssq partial sums of x^2, [n_ssq][m_pad]
  const float* ssq;
  int n_ssq;
  const float* wscale;       // 8-bit / 4-bit weights: scale of each packed row
  // EPI_RESID: x[m][n] += Y; next_gain != nullptr: also the fragments of x * next_gain and partial sums
  // of x^2 (ssq_out, planes as ssq)
  float* x;
  const float* next_gain;
  float* ssq_out;
  uint4* xs_out;             // EPI_RESID, EPI_SWIGLU: fragments for the next product
  float* out;                // EPI_OUT: [M, N]
  float* q_out;              // EPI_QKV: [M, nh*128] float32, rotated
  bf16_t* kc;                // caches [B][nh][cap][128]
  bf16_t* vc;
  const int32_t* depth;
  const int32_t* prefix_len;
  int p_max, cap, T, nh;
  float theta;
};

constexpr bool epi_pairs(int epi) { return epi == EPI_QKV || epi == EPI_SWIGLU; }

// Row sums of x^2 of N_ROWS activation rows from m0 on, by 256 threads: thread (part, row) = (tid / N_ROWS,
// tid % N_ROWS) adds every 256 / N_ROWS-th plane.  request() asks for the first BATCH of them, sum() for the rest.
// Eights behind the last plane are left out: asked for all the same (the last plane again), they took 2 of the 48 us of
// a layer of H = 512 and 65 - 128 rows, where a thread has 8 planes to add and not 64.
template <int N_ROWS, int BATCH>
struct SsqSums {
  static constexpr int kParts = 256 / N_ROWS;
  static_assert(BATCH % 8 == 0, "eights");
  const float* src;
  int n, stride, part;
  float v[BATCH];
  __device__ SsqSums(const EpiArgs& e, int m0, int tid)
      : src(e.ssq + min(m0 + tid % N_ROWS, e.m_pad - 1)), n(e.n_ssq), stride(e.m_pad), part(tid / N_ROWS) {}
  __device__ void request(int first = 0) {
#pragma unroll
    for (int i0 = 0; i0 < BATCH; i0 += 8) {
      if (i0 && kParts * (first + i0) >= n) break;       // (there is one at least)
#pragma unroll
      for (int i = i0; i < i0 + 8; ++i) v[i] = src[(size_t)(min(part + kParts * (first + i), n - 1)) * stride];
    }
  }
  __device__ float sum() {
    float s = 0.f;
    for (int first = 0;;) {
#pragma unroll
      for (int i0 = 0; i0 < BATCH; i0 += 8) {
        if (i0 && kParts * (first + i0) >= n) break;
#pragma unroll
        for (int i = i0; i < i0 + 8; ++i) s += part + kParts * (first + i) < n ? v[i] : 0.f;
      }
      first += BATCH;
      if (kParts * first >= n) return s;
      request(first);
    }
  }
};

// EPI_QKV: what the tables below need of activation row m, requested early.
struct EpiRow {
  int P, depth, b, t;
};
__device__ inline EpiRow epi_row_fetch(const EpiArgs& e, int m) {
  EpiRow r;
  r.b = m / e.T;
  r.t = m - r.b * e.T;
  r.P = e.prefix_len[r.b];
  r.depth = e.depth[m];
  return r;
}
// EPI_QKV: rotary position and cache row of the workgroup's n_rows activation rows (thread i % n_rows has row
// i's `r`), and the 64 rotary frequencies in turns per position.
__device__ inline void epi_tables(const EpiArgs& e, const EpiRow& r, int tid, int n_rows, float* s_pos, int* s_crow, float* s_freq) {
  if (tid < n_rows) {
    const int P = r.P < 0 ? 0 : (r.P > e.p_max ? e.p_max : r.P);
    s_pos[tid] = (float)(P + r.depth);
    s_crow[tid] = r.b * e.nh * e.cap + P + r.t;    // + head * cap, times 128, in the epilogue
  }
  if (tid < 64) s_freq[tid] = exp2f(-(float)tid * (1.0f / 64.0f) * log2f(e.theta)) * 0.15915494309189535f;
}

// What an item's epilogue reads from memory besides the sums, fetched together with them.
struct EpiLoads {
  f32x4_t xres, gain, ws0, ws1;
};
template <int EPI, int WF>
__device__ inline void epi_fetch(const EpiArgs& e, int N, int tile, int q, int m, int h, EpiLoads& l) {
  const int n = tile * 32 + 8 * q + 4 * h;
  if (EPI == EPI_RESID) {
    l.xres = *reinterpret_cast<const f32x4_t*>(e.x + (size_t)min(m, e.M - 1) * N + n);
    if (e.next_gain) l.gain = *reinterpret_cast<const f32x4_t*>(e.next_gain + n);
  }
  if (WF) {
    l.ws0 = *reinterpret_cast<const f32x4_t*>(e.wscale + n);
    if (epi_pairs(EPI)) l.ws1 = *reinterpret_cast<const f32x4_t*>(e.wscale + n + 16);
  }
}

// The finished sums of quad q (and quad q + 2 where the epilogue works on pairs) of a tile for activation
// row m of this lane (pos, crow: its entries of the tables).  Returns the lane's sum of x^2 (EPI_RESID).
template <int EPI, int WF>
__device__ inline float epi_quad(const EpiArgs& e, int N, int tile, int q, int m, int h, float rstd, float pos, int crow,
                                 const float* s_freq, f32x4_t v0, f32x4_t v1, const EpiLoads& l) {
  if (WF) {
    v0 *= l.ws0;
    if (epi_pairs(EPI)) v1 *= l.ws1;
  }
  if (EPI != EPI_RESID) {
    v0 *= rstd;
    if (epi_pairs(EPI)) v1 *= rstd;
  }
  const bool on = m < e.M;
  if (EPI == EPI_RESID) {
    const int n = tile * 32 + 8 * q + 4 * h;
    const f32x4_t x = l.xres + v0;
    if (on) *reinterpret_cast<f32x4_t*>(e.x + (size_t)m * N + n) = x;
    if (!e.next_gain) return 0.f;
    if (on) store_frag4(e.xs_out, e.n_rb, m, n, x * l.gain);
    return x[0] * x[0] + x[1] * x[1] + x[2] * x[2] + x[3] * x[3];
  }
  if (EPI == EPI_OUT) {
    if (on) *reinterpret_cast<f32x4_t*>(e.out + (size_t)m * N + tile * 32 + 8 * q + 4 * h) = v0;
  }
  if (EPI == EPI_SWIGLU) {
    f32x4_t a;
#pragma unroll
    for (int j = 0; j < 4; ++j) a[j] = silu_fast(v0[j]) * v1[j];
    if (on) store_frag4(e.xs_out, e.n_rb, m, tile * 16 + 8 * q + 4 * h, a);
  }
  if (EPI == EPI_QKV) {
    const int per_mat = e.nh * 4;                            // 128 rows per head = 4 tiles
    const int which = tile >= 2 * per_mat ? 2 : (tile >= per_mat ? 1 : 0);   // q, k, v
    const int head = (tile - which * per_mat) >> 2;
    const int j0 = 16 * (tile & 3) + 8 * q + 4 * h;          // first rotary pair index, 0..63 (per_mat is a multiple of 4)
    if (which != 2) {
      const f32x4_t f = *reinterpret_cast<const f32x4_t*>(s_freq + j0);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float turns = pos * f[j];                            // angle / (2 pi), reduced to [0, 1)
        turns -= floorf(turns);
        const float c = __builtin_amdgcn_cosf(turns), s = __builtin_amdgcn_sinf(turns);
        const float a = v0[j], b = v1[j];
        v0[j] = a * c - b * s;
        v1[j] = b * c + a * s;
      }
    }
    if (on) {
      if (which == 0) {
        float* dst = e.q_out + (size_t)m * e.nh * 128 + head * 128 + j0;
        *reinterpret_cast<f32x4_t*>(dst) = v0;
        *reinterpret_cast<f32x4_t*>(dst + 64) = v1;
      } else {
        bf16_t* dst = (which == 1 ? e.kc : e.vc) + ((size_t)crow + (size_t)head * e.cap) * 128 + j0;
        *reinterpret_cast<uint2*>(dst) = make_uint2(pack_bf16x2(v0[0], v0[1]), pack_bf16x2(v0[2], v0[3]));
        *reinterpret_cast<uint2*>(dst + 64) = make_uint2(pack_bf16x2(v1[0], v1[1]), pack_bf16x2(v1[2], v1[3]));
      }
    }
  }
  return 0.f;
}

// Sum of v over the lane pair (l, l ^ 32), in both.
__device__ inline float lane_pair32_sum(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// ... over the lane pair (l, l ^ 16), and over the lanes l, l ^ 16, l ^ 32, l ^ 48, in all of them.
__device__ inline float lane_pair16_sum(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ inline float lane_quad16_sum(float v) { return lane_pair32_sum(lane_pair16_sum(v)); }
// a's lanes 32 .. 63 change places with b's lanes 0 .. 31.
__device__ inline void lane_pair32_swap(f32x4_t& a, f32x4_t& b) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a[i]), __float_as_uint(b[i]), false, false);
    a[i] = __uint_as_float(r[0]);
    b[i] = __uint_as_float(r[1]);
  }
}

// ---- workgroups that share an output along K ---------------------------------------------------
// They run on one XCD and exchange float32 sums through that XCD's L2: plain stores, wait for their
// completion, arrival at a counter, bounded wait until all have arrived, L1 invalidate, loads.  The
// hardware deals workgroups to the XCDs in turn (the grid's x dimension is the XCD) and the workgroups of
// a group are neighbours in dispatch order, so the wait is short.  The placement is checked, not assumed:
// the count lives in the 4-bit field of the XCD a workgroup really runs on, and arrivals in more than one
// field, or a wait that runs out, raise a sticky status word (SV_WS_STATUS).  By one thread.
__device__ inline void group_arrive_and_wait(unsigned* cnt, int S, int n_xcd, int* status) {
  const unsigned field = 4u * (unsigned)xcd_actual(n_xcd);
  // the value the add returns is the first look at the counter: the last workgroup to arrive - the one
  // the group's finish time hangs on - goes on without a second round trip
  unsigned v = __hip_atomic_fetch_add(cnt, 1u << field, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + (1u << field);
  unsigned n = 0;
  for (int spin = 0; spin < (1 << 16); ++spin) {
    n = 0;
#pragma unroll
    for (int x = 0; x < kXcds; ++x) n += (v >> (4 * x)) & 15u;
    if (n >= (unsigned)S) break;
    __builtin_amdgcn_s_sleep(4);             // polls are device-scope round trips, keep them few
    v = __hip_atomic_load(cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // not from L1
  }
  int bad = 0;
  if (n < (unsigned)S) bad |= 2;                                  // gave up waiting
  else if (v != ((unsigned)S << field)) bad |= 1;                 // on several XCDs
  if (bad) __hip_atomic_fetch_or(status, bad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Departure: the last of the S workgroups clears the group's two words for the next launch.
__device__ inline void group_leave(unsigned* cnt, int S) {
  if (__hip_atomic_fetch_add(cnt + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)(S - 1)) {
    cnt[0] = 0;
    cnt[1] = 0;
  }
}

}  // namespace sv
#endif
