// The layer's products for up to 128 rows of activations (up to 16 see sv_gemm_thin.h): every weight byte is needed once per step,
// so the products are bound by HBM (above 64 rows by HBM and the matrix cores alike), and what is kept
// small is everything around the weight stream.
//
//   Y[m][n] = sum_k X[m][k] * W[n][k],   X = up to 128 activation rows, W = [N, K] packed.
//
//   * The activations arrive as matrix-core fragments (hi + lo bf16 parts of the float32 value,
//     1 KiB = 32 rows x 16 k-values, lane-major), written that way by whatever produced them.  Both
//     operands therefore go from memory straight into operand registers: no staging, no LDS and no
//     barrier in the main loop, and the weight stream starts with the first instruction of a launch.
//   * A workgroup owns NT weight tiles (32 rows of W each) and a K slice; its four waves take a
//     quarter of the slice each and multiply all NT tiles by all rows, so an activation fragment is
//     fetched by one wave of the workgroup only.  The four sums meet in LDS.
//   * S workgroups share the tiles along K (same XCD, same L2).  A workgroup keeps 1/S of its sums
//     and sends the rest to the others as float32.
//     60 rows of the 7B shape, us for gate+up / q,k,v / down / output: 39.0 / 27.2 / 25.1 / 14.5; the form before
//     this one (activations staged in LDS, therefore eight slices of 512 k-values, 16-bit partial
//     tiles) 47 / 31.5 / 31 / 16.  128 rows, q,k,v / output: 38.2 / 19.0 (the other two are gemm_mid's) against 36 / 19
//     of float32 partial planes plus the split, norm and reduction launches they needed, 60 over the four.
//   * The weights are packed load-major: at one k-step all tiles lie next to each other, so what the
//     chip reads at a time is spread over all memory channels (tile-major, with the tiles 256 KiB
//     apart, the same stream reached 4.1 instead of 6.0 TB/s where four tiles are read per wave).
#ifndef SV_GEMM_SKINNY_H
#define SV_GEMM_SKINNY_H

#include "sv_epilogue.h"

namespace sv {

// ---- the kernel ------------------------------------------------------------------------------
constexpr int kSkinnyMaxRows = 128;
constexpr int kSkinnyMaxUnits = 12;        // 32 x 32 accumulators of a wave (12 KiB of registers)
constexpr int skinny_max_tiles(int rb) { return rb <= 2 ? 6 : 3; }   // weight tiles per workgroup
// float4 a workgroup may send to the others of its group (odd number of KiB: regions of neighbours do not
// share memory channels)
constexpr int kSkinnyUnitStride = 4 * (kSkinnyMaxUnits + 1) * 64 + 64;

struct SkinnyArgs {
  const uint4* Xs;           // activation fragments [K / 16][row block][hi, lo][64]
  const uint4* Wp;           // packed weights [K / (16 << WF)][N / 32][64]
  int N;                     // output columns
  int lgS;                   // S = 1 << lgS workgroups along K
  int gpx, n_xcd;            // tile groups per XCD, XCDs
  // tiles per group, groups with one more, both in half tiles (lgH = 0) or tiles (1).  Half h of a tile:
  // its rows 8h .. 8h+7 and 16+8h .. 16+8h+7, the quads q with q % 2 == h
  int tq, trem, lgH;
  int uq, urem;              // weight loads (units of 16, 32 or 64 k-values) per wave, waves with one more
  // scratch of the sums that cross workgroups: one region per workgroup, and within a launch every region (and
  // for good every counter) belongs to one XCD, so that what one workgroup writes another reads through the same
  // L2.  From launch to launch a region may pass to another XCD: a launch reads only what it has written itself.
  f32x4_t* xch;              // [n_xcd][ucap][unit_stride]
  unsigned* group_cnt;       // [n_xcd][gcap][kCntStride], zero between launches
  int* status;
  int ucap, unit_stride, gcap;
  EpiArgs e;
};

// The tiles of group g: the first, how many, and which halves at the ends belong to its neighbours.
struct SkinnyTiles {
  int begin, count;
  bool skip_first, skip_last;
};
__device__ inline SkinnyTiles skinny_tiles(const SkinnyArgs& a, int g) {
  const int h0 = (g * a.tq + min(g, a.trem)) << a.lgH, h1 = h0 + ((a.tq + (g < a.trem ? 1 : 0)) << a.lgH);
  return {h0 >> 1, h1 > h0 ? ((h1 + 1) >> 1) - (h0 >> 1) : 0, (h0 & 1) != 0, (h1 & 1) != 0};
}

// LDS: the sums in exchange between the waves, [dest wave][source][quads][64] x 16 bytes
template <int RB, int NT, int EPI>
constexpr int skinny_items() { return epi_pairs(EPI) ? (RB * NT + 1) / 2 : RB * NT; }   // per wave
template <int RB, int NT, int EPI>
constexpr int skinny_quads() { return skinny_items<RB, NT, EPI>() * (epi_pairs(EPI) ? 2 : 1); }

// Weight loads in flight per wave and tile (DW) and k-steps of activations in flight (DX): about 24 KiB of
// weights per wave (more measured the same or slower), less where the load counter (63) or the registers
// (512, less the accumulators) do not hold them.  Loads return in order, so neither may run far ahead of
// the other.
template <int RB, int NT, int WF>
struct SkinnyRing {
  static constexpr int UK = 1 << WF;                     // k-steps of a weight load
  static constexpr int kRegs = (456 - 16 * RB * NT) / 4, kStep = UK * 2 * RB + NT;   // 16-byte registers; loads per weight step
  static constexpr int kFit = kRegs / kStep < 60 / kStep ? kRegs / kStep : 60 / kStep;
  static constexpr int kMost = WF == 0 ? (RB > 2 ? 4 : 3) : (WF == 1 ? 3 : 2);
  static constexpr int DW = WF == 2 ? 2 : (kFit > kMost ? kMost : kFit);
  static constexpr int DX = WF == 2 ? (RB > 2 ? 4 : 8) : DW * UK;
  static_assert(DW >= 2 && (DW * UK) % DX == 0, "ring");
  // Whether the loads ahead of the loop keep their order: the waits in the loop hold for both ways into it, so a slot
  // asked for last there is waited for as the last one in every round; against that stands what the scheduler gains by
  // mixing them with the set-up.  us of a layer, scheduler's order / this: 8 bits, 32 rows 7B 83.9 / 80.9, H = 5120
  // 106.1 / 99.8; 4 bits 32 rows H = 5120 92.1 / 87.6, 96 rows 7B 123.0 / 116.5; but bf16, 60 rows 7B 119.9 / 127.5,
  // H = 2048 69.2 / 72.3; 8 bits 33 - 128 rows the same within 1 %.  The head, 256 columns of H = 4096, 17, 60 and 240 rows
  // 11.5 / 11.2, 13.5 / 13.0, 20.4 / 19.8.
  static constexpr bool in_order(int epi) { return epi == EPI_OUT || WF == 2 || (WF == 1 && RB == 1); }
};

template <int RB, int NT, int EPI, int WF>
__device__ __forceinline__ void skinny_body(const SkinnyArgs& a, f32x4_t* lds, float* s_rows, float* s_pos, int* s_crow,
                                            float* s_freq, const int xcd, const int ug, const int mt, const int sp) {
  typedef SkinnyRing<RB, NT, WF> Ring;
  constexpr int U = RB * NT, UK = Ring::UK, DW = Ring::DW, DX = Ring::DX;
  constexpr bool PAIR = epi_pairs(EPI);
  constexpr int QI = PAIR ? 2 : 1;                       // quads per item
  constexpr int NI = skinny_items<RB, NT, EPI>();        // items per wave
  constexpr int NQ = NI * QI;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int S = 1 << a.lgS;
  const int g = xcd * a.gpx + ug;
  const int m0 = EPI == EPI_OUT ? mt * RB * 32 : 0;      // first row of this block
  const int gm = EPI == EPI_OUT ? mt * a.gpx + ug : ug;  // group of workgroups that share sums, on this XCD
  const SkinnyTiles tl = skinny_tiles(a, g);
  const int t_begin = tl.begin, t_count = tl.count;

  // this wave's run of weight loads
  const int ws = sp * 4 + wave;
  const int u0 = ws * a.uq + min(ws, a.urem);
  const int n_units = a.uq + (ws < a.urem ? 1 : 0);

  constexpr int kRows = RB * 32;
  SsqSums<kRows, (EPI == EPI_OUT ? 8 : (RB > 2 ? 64 : 32))> rows(a.e, EPI == EPI_OUT ? m0 : 0, tid);
  if (EPI == EPI_OUT) rows.request();

  // Rings.  Every step issues exactly as many loads as it has used - from the activations' first fragments,
  // which the caches hold, once nothing is left - so that the number of younger loads behind any slot is
  // a compile-time constant and the waits are exact.
  typedef const __attribute__((address_space(1))) u32x4_t* gptr_t;
  const size_t w_step = (size_t)(a.N / kFragRows) * 64;
  gptr_t wp = (gptr_t)a.Wp + (size_t)u0 * w_step + (size_t)t_begin * 64;
  const unsigned x_step = a.e.n_rb * 128u;
  gptr_t xp = (gptr_t)a.Xs + (size_t)u0 * UK * x_step;
  unsigned w_off[NT], x_off[RB];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    // (fewer tiles than NT: the last one again, dropped below; a half that is not this group's: the other half again)
    const unsigned l = t == 0 && tl.skip_first ? lane | 8 : (t >= t_count - 1 && tl.skip_last ? lane & ~8 : lane);
    w_off[t] = (unsigned)min(t, t_count - 1) * 64u + l;
  }
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) x_off[rb] = (EPI == EPI_OUT ? (unsigned)min(mt * RB + rb, a.e.n_rb - 1) : rb) * 128u + lane;
  u32x4_t xr[DX][2 * RB], wr[DW][NT];
  int w_left = n_units, x_left = n_units * UK;
  if (n_units == 0) wp = xp = (gptr_t)a.Xs;
  auto issue_x = [&](int d) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      xr[d][2 * rb] = xp[x_off[rb]];
      xr[d][2 * rb + 1] = xp[x_off[rb] + 64u];
    }
    if (--x_left > 0) xp += x_step;
    else xp = (gptr_t)a.Xs;
  };
  auto issue_w = [&](int d) {
#pragma unroll
    for (int t = 0; t < NT; ++t) wr[d][t] = __builtin_nontemporal_load(wp + w_off[t]);   // streamed once
    if (--w_left > 0) wp += w_step;
    else wp = (gptr_t)a.Xs;
  };
#pragma unroll
  for (int d = 0; d < DX || d < DW; ++d) {
    if (d < DX) issue_x(d);
    if (d < DW) issue_w(d);
    if (Ring::in_order(EPI)) __builtin_amdgcn_sched_barrier(0);
  }
  f32x16_t acc[NT][RB];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) acc[t][rb] = f32x16_t{};

  int left = n_units;
  while (left > 0) {
#pragma unroll
    for (int d = 0; d < DW; ++d) {
#pragma unroll
      for (int kk = 0; kk < UK; ++kk) {
        const int xs = (d * UK + kk) % DX;
        if (left > d) {
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            const bf16x8_t w = weight_operand<WF>(wr[d][t], kk);
#pragma unroll
            for (int hl = 0; hl < 2; ++hl)
#pragma unroll
              for (int rb = 0; rb < RB; ++rb)
                acc[t][rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, __builtin_bit_cast(bf16x8_t, xr[xs][2 * rb + hl]), acc[t][rb], 0, 0, 0);
          }
        }
        issue_x(xs);
      }
      issue_w(d);
    }
    left -= DW;
  }

  // What the epilogue needs to know of the rows: row sums of x^2 - thread (row, part) adds its share of the
  // planes - and rotary positions.  Requested here, answered while the sums meet.  (Requested and waited for
  // ahead of the loop they held it up by 2.5 us, by 9 us at 128 rows.  The head's few planes are requested there.)
  if (epi_pairs(EPI)) rows.request();
  EpiRow er;
  if (EPI == EPI_QKV) er = epi_row_fetch(a.e, min(tid % kRows, a.e.M - 1));

  // ---- the four waves' sums meet in LDS ----
  // A wave finishes, of every unit, the quad of its own number (of every second unit the quads p and
  // p + 2 where the epilogue works on pairs); it hands the other quads to their waves.
  auto quad = [&](int u, int q) -> f32x4_t {
    const f32x16_t& c = acc[u / RB][u % RB];
    return f32x4_t{c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]};
  };
  f32x4_t mine[NQ];
  const int n_mine = PAIR ? (U - (wave >> 1) + 1) / 2 : U;         // items of this wave
  auto hand_over = [&](auto me) {
    constexpr int W = decltype(me)::value;
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
      for (int k = 0; k < NQ; ++k) {
        const int jj = k / QI, qi = k % QI;
        const int u = PAIR ? 2 * jj + (d >> 1) : jj, q = PAIR ? (d & 1) + 2 * qi : d;
        if (u >= U) continue;
        if (d == W) mine[k] = quad(u, q);
        else lds[((d * 3 + (W < d ? W : W - 1)) * NQ + k) * 64 + lane] = quad(u, q);
      }
  };
  if (wave == 0) hand_over(std::integral_constant<int, 0>{});
  else if (wave == 1) hand_over(std::integral_constant<int, 1>{});
  else if (wave == 2) hand_over(std::integral_constant<int, 2>{});
  else hand_over(std::integral_constant<int, 3>{});
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
  for (int k = 0; k < NQ; ++k) {
    if (k / QI < n_mine) {
#pragma unroll
      for (int s = 0; s < 3; ++s) mine[k] += lds[((wave * 3 + s) * NQ + k) * 64 + lane];
    }
  }
  // (other waves may still read their shares: the items kept by this one go to its own)
  f32x4_t* own = lds + (size_t)wave * 3 * NQ * 64 + lane;

  // ---- the S workgroups' sums meet in the XCD's L2 ----
  // item j of a wave is finished by slice j % S
  const size_t unit = (size_t)xcd * a.ucap + gm * S;               // first workgroup of the group
#pragma unroll
  for (int j = 0; j < NI; ++j) {
    if (j >= n_mine) continue;
    if ((j & (S - 1)) == sp) {
#pragma unroll
      for (int qi = 0; qi < QI; ++qi) own[(j * QI + qi) * 64] = mine[j * QI + qi];
    } else {
      f32x4_t* dst = a.xch + (unit + sp) * a.unit_stride + (size_t)(wave * (NQ + 1) + j * QI) * 64 + lane;
#pragma unroll
      for (int qi = 0; qi < QI; ++qi) dst[qi * 64] = mine[j * QI + qi];
    }
  }
  if (EPI != EPI_RESID) s_rows[tid] = rows.sum();
  if (EPI == EPI_QKV) epi_tables(a.e, er, tid, kRows, s_pos, s_crow, s_freq);
  const auto gcnt = a.group_cnt + ((size_t)xcd * a.gcap + gm) * kCntStride;
  if (S > 1) __builtin_amdgcn_s_waitcnt(0);         // this wave's sums are in the L2
  __syncthreads();
  if (S > 1) {
    if (tid == 0) group_arrive_and_wait(gcnt, S, a.n_xcd, a.status);
    __syncthreads();
    asm volatile("buffer_inv sc0" ::: "memory");                   // drop stale L1 lines (the L2 is shared)
  }

  const int h = lane >> 5;
  // 1 / rms of the rows of this lane: every wave works out those of all row blocks, for itself
  float* const s_rstd = s_rows + 256 + wave * kRows;
  if (EPI != EPI_RESID) {
    if (lane < 32) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        float t = 0.f;
#pragma unroll
        for (int p = 0; p < 256 / kRows; ++p) t += s_rows[p * kRows + rb * 32 + lane];
        s_rstd[rb * 32 + lane] = 1.0f / sqrtf(t / (float)a.e.K + a.e.eps);
      }
    }
  }
  // Items of this slice, a few at a time with all their loads in flight together.
  auto finish = [&](auto split) {
    constexpr int SS = decltype(split)::value;
    constexpr int BT = SS == 8 ? 1 : (SS == 4 ? 2 : 3);
    for (int k0 = sp; k0 < n_mine; k0 += SS * BT) {
      f32x4_t part[BT][QI][SS];
      EpiLoads ld[BT];
#pragma unroll
      for (int b = 0; b < BT; ++b) {
        const int j = min(k0 + b * SS, n_mine - 1);
        const int u = PAIR ? 2 * j + (wave >> 1) : j, q = PAIR ? (wave & 1) : wave;
        const int t = min(u / RB, t_count - 1), rb = u % RB;
#pragma unroll
        for (int s2 = 1; s2 < SS; ++s2) {
          const f32x4_t* src = a.xch + (unit + ((sp + s2) & (SS - 1))) * a.unit_stride + (size_t)(wave * (NQ + 1) + j * QI) * 64 + lane;
#pragma unroll
          for (int qi = 0; qi < QI; ++qi) part[b][qi][s2] = src[qi * 64];
        }
        epi_fetch<EPI, WF>(a.e, a.N, t_begin + t, q, rb * 32 + (lane & 31), h, ld[b]);
#pragma unroll
        for (int qi = 0; qi < QI; ++qi) part[b][qi][0] = own[(j * QI + qi) * 64];
      }
      asm volatile("" ::: "memory");
#pragma unroll
      for (int b = 0; b < BT; ++b) {
        const int j = k0 + b * SS;
        if (j >= n_mine) break;
        const int u = PAIR ? 2 * j + (wave >> 1) : j, q = PAIR ? (wave & 1) : wave;
        const int t = u / RB, rb = u % RB;
        if (t >= t_count) break;
        if ((t == 0 && tl.skip_first && !(q & 1)) || (t == t_count - 1 && tl.skip_last && (q & 1))) continue;
        f32x4_t v[2] = {part[b][0][0], part[b][QI - 1][0]};
#pragma unroll
        for (int s2 = 1; s2 < SS; ++s2) {
          v[0] += part[b][0][s2];
          if (PAIR) v[1] += part[b][QI - 1][s2];
        }
        const int ml = rb * 32 + (lane & 31);
        const float pos = EPI == EPI_QKV ? s_pos[ml] : 0.f;
        const int crow = EPI == EPI_QKV ? s_crow[ml] : 0;
        const float rs = EPI != EPI_RESID ? s_rstd[ml] : 1.f;
        float sq = epi_quad<EPI, WF>(a.e, a.N, t_begin + t, q, m0 + ml, h, rs, pos, crow, s_freq, v[0], v[1], ld[b]);
        if (EPI == EPI_RESID) {
          sq = lane_pair32_sum(sq);
          if (h == 0) s_rows[(wave * U + u) * 32 + lane] = sq;
        }
      }
    }
  };
  if (S == 1) finish(std::integral_constant<int, 1>{});
  else if (S == 2) finish(std::integral_constant<int, 2>{});
  else if (S == 4) finish(std::integral_constant<int, 4>{});
  else finish(std::integral_constant<int, 8>{});

  // partial sums of x^2 of the new rows: one plane per tile, the four quads added in order
  if (EPI == EPI_RESID && a.e.next_gain) {
    __syncthreads();
    for (int i = tid; i < U * 32; i += 256) {
      const int u = i >> 5, t = u / RB, m = (u % RB) * 32 + (i & 31);
      if ((u & (S - 1)) != sp || t >= t_count) continue;
      a.e.ssq_out[(size_t)(t_begin + t) * a.e.m_pad + m] = (s_rows[i] + s_rows[U * 32 + i]) + (s_rows[2 * U * 32 + i] + s_rows[3 * U * 32 + i]);
    }
  }
  if (S > 1 && tid == 0) group_leave(gcnt, S);
}

// grid = (n_xcd, gpx * S, blocks of RB row blocks: EPI_OUT, else 1), block = 256, one workgroup per CU.  The
// hardware deals workgroups to the XCDs in turn, so x is the XCD; in y the S slices of a tile group follow each
// other.  A group has NTM or NTM - 1 tiles (fewer: the spare ones are multiplied and dropped).
template <int RB, int NTM, int EPI, int WF>
__global__ __launch_bounds__(256, 1) void gemm_skinny(const SkinnyArgs a) {
  constexpr int kRowWords = EPI == EPI_RESID ? 4 * RB * NTM * 32 : 256 + 4 * RB * 32;
  __shared__ f32x4_t lds[12 * skinny_quads<RB, NTM, EPI>() * 64];
  __shared__ float s_rows[kRowWords];
  __shared__ float s_pos[EPI == EPI_QKV ? 32 * RB : 1];
  __shared__ int s_crow[EPI == EPI_QKV ? 32 * RB : 1];
  __shared__ __attribute__((aligned(16))) float s_freq[64];
  const int ug = (int)blockIdx.y >> a.lgS, sp = (int)blockIdx.y & ((1 << a.lgS) - 1), mt = EPI == EPI_OUT ? (int)blockIdx.z : 0;
  const int t_count = skinny_tiles(a, (int)blockIdx.x * a.gpx + ug).count;
  if (t_count == 0) return;
  if (t_count == NTM) skinny_body<RB, NTM, EPI, WF>(a, lds, s_rows, s_pos, s_crow, s_freq, blockIdx.x, ug, mt, sp);
  else skinny_body<RB, NTM - 1, EPI, WF>(a, lds, s_rows, s_pos, s_crow, s_freq, blockIdx.x, ug, mt, sp);
}

}  // namespace sv
#endif
