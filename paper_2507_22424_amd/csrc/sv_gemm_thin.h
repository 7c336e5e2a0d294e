// The layer's products for up to 16 rows of activations (plain decoding, small trees): gemm_skinny with half of its
// rows left out.
//
// v_mfma_f32_16x16x32_bf16 instead of 32x32x16: an activation fragment holds 32 rows, of which only the first 16 are
// fetched and multiplied.  What bounds these products is the weight stream (and the launch around it); the
// activations that every workgroup reads through the same paths, the sums in exchange and the matrix work - which,
// with the conversions of coded weights, costs power and with it clock - are halved.  The weights are the same
// packed tiles: a lane's eight k-values are half of a 32-row fragment's k-step, taken from two k-steps.
// One layer of the 7B shape, attention included, us, gemm_skinny / this: one row 102.4 / 97.1 (bf16), 80.8 / 71.8 (8 bits),
// 71.7 / 67.9 (4 bits); 16 rows 102.9 / 97.9, 81.2 / 73.5, 72.0 / 68.6.  The same form with more rows, four products: 32 rows
// 86.2 / 89.6, 62.2 / 68.1, 55.0 / 57.8 - its steps are twice as deep, so more is in flight that the next phase has to wait
// for -, 48 rows of coded weights 86 / 81.5, 78 / 73; only this one is built.
#ifndef SV_GEMM_THIN_H
#define SV_GEMM_THIN_H

#include "sv_gemm_skinny.h"

namespace sv {

constexpr int kThinRows = 16;
constexpr int thin_items(int nt) { return (nt + 3) / 4; }          // tiles a wave finishes

// Steps in flight: 24 KiB of weights per wave (codes: a step more than the one that is being converted, as far as
// the load counter goes).  A step is what one weight load covers, KK matrix instructions (32 k-values each).
template <int NT, int WF>
struct ThinRing {
  static constexpr int KK = WF == 2 ? 2 : 1;
  static constexpr int D = WF == 0 ? (NT > 4 ? 2 : (NT > 3 ? 3 : 4)) : (WF == 2 && NT > 4 ? 3 : 4);
  static_assert(D * (2 * NT + 2 * KK) <= 60, "load counter");
};
// k-values of a step
constexpr int thin_step_k(int wf) { return wf == 2 ? 64 : 32; }

// (arguments and the meeting of the workgroups: see skinny_body)
template <int NT, int EPI, int WF>
__device__ __forceinline__ void thin_body(const SkinnyArgs& a, f32x4_t* lds, float* s_rows, float* s_pos, int* s_crow,
                                          float* s_freq, const int xcd, const int ug, const int sp) {
  typedef ThinRing<NT, WF> Ring;
  constexpr int KK = Ring::KK, D = Ring::D;
  constexpr bool PAIR = epi_pairs(EPI);
  constexpr int NI = thin_items(NT), NQ = 2 * NI;        // items (16 rows x weight tile), accumulators of a wave
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int S = 1 << a.lgS;
  const int g = xcd * a.gpx + ug;
  const SkinnyTiles tl = skinny_tiles(a, g);
  const int t_begin = tl.begin, t_count = tl.count;

  // this wave's run of steps
  const int ws = sp * 4 + wave;
  const int u0 = ws * a.uq + min(ws, a.urem);
  const int n_units = a.uq + (ws < a.urem ? 1 : 0);

  SsqSums<kThinRows, 8> rows(a.e, 0, tid);
  if (EPI == EPI_OUT) rows.request();

  // Lane (i16, g16) of v_mfma_f32_16x16x32_bf16 holds eight k-values of weight (or activation) row i16.  Out of the
  // 32-row fragments: k-half g16 % 2 of k-step KK * (g16 / 2) + kk.  Coded weights: a 16-byte piece covers two
  // k-steps (E4M3) or four (int4), of which a lane fetches its own 8 bytes.
  // Addresses are a uniform pointer, which moves, and a lane's offset in bytes, which does not.
  typedef const __attribute__((address_space(1))) char* gptr_t;
  typedef typename std::conditional<WF == 0, u32x4_t, u32x2_t>::type wload_t;
  const int g16 = lane >> 4, i16 = lane & 15, k_half = 32 * (g16 & 1);
  const unsigned w_row = (unsigned)(a.N / kFragRows) * 1024u;      // bytes of all tiles at one k-step (or row of pieces)
  const unsigned w_step = WF ? w_row : 2 * w_row;
  const unsigned x_kstep = a.e.n_rb * 2048u;
  gptr_t wp = (gptr_t)a.Wp + (size_t)u0 * w_step + (size_t)t_begin * 1024;
  gptr_t xp = (gptr_t)a.Xs + (size_t)u0 * 2 * KK * x_kstep;
  unsigned w_lane = ((i16 & 7) + 16 * (i16 >> 3) + k_half) * 16u + (g16 >> 1) * (WF ? 8u : w_row);
  const unsigned x_lane = (i16 + k_half) * 16u + (g16 >> 1) * KK * x_kstep;
  u32x4_t xr[D * KK][2];
  wload_t wr[D][2 * NT];
  int w_left = n_units, x_left = n_units * KK;
  if (n_units == 0) {
    wp = xp = (gptr_t)a.Xs;
    w_lane = i16 * 16u;
  }
  // (the activations' steps are those of the instructions: kk = 0, 1 of a weight step with codes of 4 bits)
  auto issue_x = [&](int x) {
#pragma unroll
    for (int hl = 0; hl < 2; ++hl) xr[x][hl] = *(const __attribute__((address_space(1))) u32x4_t*)(xp + hl * 1024 + x_lane);
  };
  // (once nothing is left the loads repeat the activations' first fragments, which the caches hold, so that the number
  // of younger loads behind any slot is a compile-time constant and the waits are exact)
  auto next_x = [&](int kk) {
    if (--x_left > 0) xp += KK == 1 ? 2 * x_kstep : (kk == 0 ? x_kstep : 3 * x_kstep);
    else xp = (gptr_t)a.Xs;
  };
  auto issue_w = [&](int d, int t) {
    // (fewer tiles than NT: the last one again, dropped below; a half that is not this group's: the other half again)
    const int half = t < 2 && tl.skip_first ? 1 : ((t >> 1) >= t_count - 1 && tl.skip_last ? 0 : t & 1);
    const unsigned piece = min(t >> 1, t_count - 1) * 1024u + half * 128u;
    wr[d][t] = __builtin_nontemporal_load((const __attribute__((address_space(1))) wload_t*)(wp + piece + w_lane));   // streamed once
  };
  auto next_w = [&]() {
    if (--w_left > 0) {
      wp += w_step;
    } else {
      wp = (gptr_t)a.Xs;
      w_lane = i16 * 16u;
    }
  };
#pragma unroll
  for (int d = 0; d < D; ++d) {
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      issue_x(d * KK + kk);
      next_x(kk);
    }
#pragma unroll
    for (int t = 0; t < 2 * NT; ++t) issue_w(d, t);
    next_w();
    __builtin_amdgcn_sched_barrier(0);                    // (in this order: see SkinnyRing)
  }

  f32x4_t acc[2 * NT];                                    // 16 activation rows x 16 weight rows each
#pragma unroll
  for (int t = 0; t < 2 * NT; ++t) acc[t] = f32x4_t{};

  // Codes are converted one instruction step ahead, a few words next to every two matrix instructions.
  bf16x8_t w[2 * NT];
  if (WF) {
#pragma unroll
    for (int t = 0; t < 2 * NT; ++t) w[t] = weight_operand<WF>(wr[0][t], 0);
  }
  int left = n_units;
  while (left > 0) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        const int x = d * KK + kk, dn = kk + 1 < KK ? d : (d + 1) % D, kn = (kk + 1) % KK;
        u32x4_t wn[2 * NT];
        unsigned odd = 0;
        if (left > d) {
#pragma unroll
          for (int t = 0; t < 2 * NT; ++t) {
            bf16x8_t wt = w[t];
            if constexpr (WF == 0) wt = __builtin_bit_cast(bf16x8_t, wr[d][t]);
#pragma unroll
            for (int hl = 0; hl < 2; ++hl)
              acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wt, __builtin_bit_cast(bf16x8_t, xr[x][hl]), acc[t], 0, 0, 0);
            if constexpr (WF != 0) {
#pragma unroll
              for (int j = 0; j < 4; ++j) wn[t][j] = weight_word<WF>(wr[dn][t], kn, j, odd);
            }
            if constexpr (WF != 0) __builtin_amdgcn_sched_barrier(0);
            else __builtin_amdgcn_sched_barrier(kMfmaOrder);
          }
        }
        __builtin_amdgcn_sched_barrier(0);                // (the loads stay behind what they replace)
        issue_x(x);
        __builtin_amdgcn_sched_barrier(0);
        next_x(kk);
        if constexpr (WF != 0) {
#pragma unroll
          for (int t = 0; t < 2 * NT; ++t) w[t] = __builtin_bit_cast(bf16x8_t, wn[t]);
        }
      }
#pragma unroll
      for (int t = 0; t < 2 * NT; ++t) issue_w(d, t);
      next_w();
      __builtin_amdgcn_sched_barrier(0);
    }
    left -= D;
  }

  // what the epilogue needs to know of the rows: see skinny_body (the head's planes too)
  if (epi_pairs(EPI)) rows.request();
  EpiRow er;
  if (EPI == EPI_QKV) er = epi_row_fetch(a.e, min(tid % kThinRows, a.e.M - 1));

  // ---- the four waves' sums meet in LDS: tile t is wave t % 4's ----
  f32x4_t mine[NQ];
  const int n_mine = (NT - wave + 3) / 4;
  auto hand_over = [&](auto me) {
    constexpr int W = decltype(me)::value;
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
      for (int k = 0; k < NQ; ++k) {
        const int t = 4 * (k >> 1) + d;
        if (t >= NT) continue;
        if (d == W) mine[k] = acc[2 * t + (k & 1)];
        else lds[((d * 3 + (W < d ? W : W - 1)) * NQ + k) * 64 + lane] = acc[2 * t + (k & 1)];
      }
  };
  if (wave == 0) hand_over(std::integral_constant<int, 0>{});
  else if (wave == 1) hand_over(std::integral_constant<int, 1>{});
  else if (wave == 2) hand_over(std::integral_constant<int, 2>{});
  else hand_over(std::integral_constant<int, 3>{});
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
  for (int k = 0; k < NQ; ++k) {
    if ((k >> 1) < n_mine) {
#pragma unroll
      for (int s = 0; s < 3; ++s) mine[k] += lds[((wave * 3 + s) * NQ + k) * 64 + lane];
    }
  }

  // ---- the S workgroups' sums meet in the XCD's L2 ----
  // item k of a wave is finished by slice (wave * NI + k) % S
  const size_t unit = (size_t)xcd * a.ucap + ug * S;               // first workgroup of the group
#pragma unroll
  for (int k = 0; k < NI; ++k) {
    if (k >= n_mine || ((wave * NI + k) & (S - 1)) == sp) continue;
    f32x4_t* dst = a.xch + (unit + sp) * a.unit_stride + (size_t)(wave * (NQ + 1) + k * 2) * 64 + lane;
    dst[0] = mine[2 * k];
    dst[64] = mine[2 * k + 1];
  }
  if (EPI != EPI_RESID) s_rows[tid] = rows.sum();
  if (EPI == EPI_QKV) epi_tables(a.e, er, tid, kThinRows, s_pos, s_crow, s_freq);
  const auto gcnt = a.group_cnt + ((size_t)xcd * a.gcap + ug) * kCntStride;
  if (S > 1) __builtin_amdgcn_s_waitcnt(0);         // this wave's sums are in the L2
  __syncthreads();
  if (S > 1) {
    if (tid == 0) group_arrive_and_wait(gcnt, S, a.n_xcd, a.status);
    __syncthreads();
    asm volatile("buffer_inv sc0" ::: "memory");                   // drop stale L1 lines (the L2 is shared)
  }

  // The halves of a tile change places between the lanes l and l + 32: lane (i16, h, q) then has quads q and q + 2 of
  // row i16.
  const int q = lane >> 5, h = g16 & 1;
  float rs = 1.f;                                         // 1 / rms of the lane's row
  if (EPI != EPI_RESID) {
    float t = 0.f;
#pragma unroll
    for (int p = 0; p < 256 / kThinRows; ++p) t += s_rows[p * kThinRows + i16];
    rs = 1.0f / sqrtf(t / (float)a.e.K + a.e.eps);
  }
  const float pos = EPI == EPI_QKV ? s_pos[i16] : 0.f;
  const int crow = EPI == EPI_QKV ? s_crow[i16] : 0;
  auto finish = [&](auto split) {
    constexpr int SS = decltype(split)::value;
#pragma unroll
    for (int k = 0; k < NI; ++k) {
      const int t = 4 * k + wave;
      if (k >= n_mine || ((wave * NI + k) & (SS - 1)) != sp || t >= t_count) continue;
      f32x4_t part[2][SS];
      EpiLoads ld[2];
#pragma unroll
      for (int s2 = 1; s2 < SS; ++s2) {
        const f32x4_t* src = a.xch + (unit + ((sp + s2) & (SS - 1))) * a.unit_stride + (size_t)(wave * (NQ + 1) + k * 2) * 64 + lane;
        part[0][s2] = src[0];
        part[1][s2] = src[64];
      }
      const bool off = (t == 0 && tl.skip_first && q == 0) || (t == t_count - 1 && tl.skip_last && q == 1);
      const int m = off ? a.e.M : i16;
      epi_fetch<EPI, WF>(a.e, a.N, t_begin + t, q, m, h, ld[0]);
      if (!PAIR) epi_fetch<EPI, WF>(a.e, a.N, t_begin + t, q + 2, m, h, ld[1]);
      f32x4_t v0 = mine[2 * k], v1 = mine[2 * k + 1];
#pragma unroll
      for (int s2 = 1; s2 < SS; ++s2) {
        v0 += part[0][s2];
        v1 += part[1][s2];
      }
      lane_pair32_swap(v0, v1);
      float sq = epi_quad<EPI, WF>(a.e, a.N, t_begin + t, q, m, h, rs, pos, crow, s_freq, v0, v1, ld[0]);
      if (!PAIR) sq += epi_quad<EPI, WF>(a.e, a.N, t_begin + t, q + 2, m, h, rs, pos, crow, s_freq, v1, v1, ld[1]);
      if (EPI == EPI_RESID && a.e.next_gain) {            // partial sums of x^2 of the new rows: one plane per tile
        sq = lane_quad16_sum(sq);
        if (lane < kThinRows) a.e.ssq_out[(size_t)(t_begin + t) * a.e.m_pad + i16] = sq;
      }
    }
  };
  if (S == 1) finish(std::integral_constant<int, 1>{});
  else if (S == 2) finish(std::integral_constant<int, 2>{});
  else if (S == 4) finish(std::integral_constant<int, 4>{});
  else finish(std::integral_constant<int, 8>{});
  if (S > 1 && tid == 0) group_leave(gcnt, S);
}

// grid = (n_xcd, gpx * S), block = 256: as gemm_skinny.
template <int NTM, int EPI, int WF>
__global__ __launch_bounds__(256, 1) void gemm_thin(const SkinnyArgs a) {
  __shared__ f32x4_t lds[12 * 2 * thin_items(NTM) * 64];
  __shared__ float s_rows[256];
  __shared__ float s_pos[EPI == EPI_QKV ? kThinRows : 1];
  __shared__ int s_crow[EPI == EPI_QKV ? kThinRows : 1];
  __shared__ __attribute__((aligned(16))) float s_freq[64];
  const int ug = (int)blockIdx.y >> a.lgS, sp = (int)blockIdx.y & ((1 << a.lgS) - 1);
  const int t_count = skinny_tiles(a, (int)blockIdx.x * a.gpx + ug).count;
  if (t_count == 0) return;
  if (t_count == NTM) thin_body<NTM, EPI, WF>(a, lds, s_rows, s_pos, s_crow, s_freq, blockIdx.x, ug, sp);
  else thin_body<NTM - 1, EPI, WF>(a, lds, s_rows, s_pos, s_crow, s_freq, blockIdx.x, ug, sp);
}

}  // namespace sv
#endif
