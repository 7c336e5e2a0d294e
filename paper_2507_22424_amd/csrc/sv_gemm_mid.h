// The layer's products for more than 128 rows of activations, and some of 65 - 128 rows of bf16 weights (plan_product).
//
// With this many rows the matrix cores set the time, at the clock that their power leaves on real data.  On random
// data, all CUs, nothing but matrix instructions, v_mfma_f32_32x32x16_bf16 sustains 1.75 - 1.8 PFLOP/s in any order of
// its operands, 16x16x32 1.7 with the weight tiles outermost, 2.06 with the rows outermost, 2.25 where besides both
// parts of a row are added to the same sums one after the other; hence that instruction in that order.  The main
// loop issues 1.5 PFLOP/s (hi and lo half of the activations counted; 1.35 with 32x32x16), a large bf16 product of the
// vendor's library 1.16 on the same card.  What is left to lose is around the loop and in work on rows that do not
// exist (7B layer, four products and attention: 3 x 50 rows 210 us with 32x32x16, 194 now; 16 x 60 rows 787, 705), hence:
//   * blocks of RB = 3, 4 or 5 row blocks of 32 rows x 4 waves x NT weight tiles; the host weighs rows that
//     are only padding against whole rounds of the chip (150 rows: 192 are multiplied, two blocks of 3, which fill
//     the chip with half the K slices, and so less exchange, than one of 5 would need);
//   * a weight tile belongs to one wave: its fragments go from memory straight into operand registers,
//     through a ring of D chunks.  The activations of a chunk (two k-steps; four with coded weights, see mid_kk) are
//     fetched once per workgroup, each wave loading a quarter of the fragments into registers and writing
//     them to LDS one chunk ahead of their use; one barrier per chunk, three LDS buffers.  Every load is
//     one the compiler knows of, in a fixed order, so its waits are exact;
//   * S workgroups share an output block along K (same XCD) and exchange float32 sums through its L2;
//     every one of them finishes 1/S of the block with the epilogue fused.  No partial planes, no
//     reduction launches, no launches that split activations: the epilogues leave fragments.
#ifndef SV_GEMM_MID_H
#define SV_GEMM_MID_H

#include "sv_epilogue.h"

namespace sv {

struct MidArgs {
  const uint4* Xs;           // activation fragments [K / 16][row block][hi, lo][64]
  const uint4* Wp;           // packed weights [K / (16 << WF)][N / 32][64]
  int N;                     // output columns
  int lgS;                   // S = 1 << lgS workgroups along K
  int gpx, n_xcd, m_tiles;   // column groups per XCD, XCDs, blocks of rows
  int tq, trem;              // tiles per column group, groups with one more
  int cq, crem;              // chunks per K slice, slices with one more
  int planes;                // EPI_RESID: row-sum planes per column group
  // scratch of the sums that cross workgroups, by XCD: see gemm_skinny
  f32x4_t* xch;              // [n_xcd][ucap][unit_stride]
  unsigned* group_cnt;       // [n_xcd][gcap][kCntStride], zero between launches
  int* status;
  int ucap, unit_stride, gcap;
  EpiArgs e;
};

constexpr int kMidMaxTiles = 3;            // weight tiles per wave
constexpr int kMidMaxRows = 5;             // row blocks per workgroup

// An item = 16 rows of a weight tile (32 x 16 sums: two accumulators, whose quads are p and p + 2 of a lane).
// A wave has 2 * RB * NT items, 16 rows after 16 rows; slice sp finishes the items from mid_first(sp) on.
constexpr int mid_items(int rb, int nt) { return 2 * rb * nt; }
__host__ __device__ constexpr int mid_first(int items, int lgS, int sp) { return (sp * items + (1 << lgS) - 1) >> lgS; }
__host__ __device__ constexpr int mid_owner(int items, int lgS, int i) { return (i << lgS) / items; }
// slices that finish a part of the items of 16 rows, at most: the planes of row sums
constexpr int mid_planes(int rb, int nt, int lgS) {
  int most = 1;
  for (int r = 0; r < 2 * rb; ++r) {
    const int n = mid_owner(mid_items(rb, nt), lgS, (r + 1) * nt - 1) - mid_owner(mid_items(rb, nt), lgS, r * nt) + 1;
    most = n > most ? n : most;
  }
  return most;
}
// float4 a workgroup may send (4 waves, padded so that the regions do not share memory channels)
constexpr int mid_unit_stride(int rb, int nt) { return (4 * (rb * nt * 4 + 1) + 5) * 64; }

// A chunk is KK matrix instructions deep (32 k-values each): one with bf16 weights, two with codes - but one for E4M3
// where accumulators (240 of 512 registers) and a ring of two such chunks leave too little for the operands:
// gemm_mid<5, 3, *, 1> then kept 300 registers in scratch memory, 7B, 8 bits, us a layer of 300 / 600 / 1800 rows
// 538 / 1236 / 2910, 279 / 454 / 1274 with one.  Elsewhere two are faster (400 rows 370 / 383, 960 rows 692 / 700).
constexpr int mid_kk(int rb, int nt, int wf) { return wf == 2 || (wf == 1 && rb * nt < 15) ? 2 : 1; }
constexpr int mid_chunk_k(int rb, int nt, int wf) { return 32 * mid_kk(rb, nt, wf); }
template <int RB, int NT, int WF>
struct MidShape {
  static constexpr int KK = mid_kk(RB, NT, WF), CK = 2 * KK;   // matrix instructions, k-steps of a chunk
  static constexpr int CW = CK >> WF, WU = 2 / CW;             // weight units of a chunk; loads in a 16-byte piece
  static constexpr int LW = 2 * NT, LX = CK * RB / 2;          // loads of a wave per chunk
  // chunks in flight: what the load counter (63) and the registers hold, 12 k-steps at most
  static constexpr int kCnt = 60 / (LW + LX), kReg = (416 - 16 * RB * NT) / (4 * LX + 4 / WU * LW);
  static constexpr int D0 = kCnt < kReg ? kCnt : kReg;
  static constexpr int D = D0 > 12 / CK ? 12 / CK : D0;
  static_assert(D >= 2, "ring too short");
};

// grid = (n_xcd, gpx * m_tiles * S), block = 256, one workgroup per CU: x is the XCD; in y the S slices of
// an output block follow each other, then the blocks of rows of a column group, which read the same
// weights at about the same time.
template <int RB, int NT, int EPI, int WF>
__global__ __launch_bounds__(256, 1) void gemm_mid(const MidArgs a) {
  typedef MidShape<RB, NT, WF> Sh;
  constexpr int KK = Sh::KK, CK = Sh::CK, LX = Sh::LX, D = Sh::D, R = 2 * RB;
  constexpr int E = KK * R, PD = NT == 1 ? 4 : 2;              // steps (16 rows) of a chunk; operands are read PD steps ahead
  // LDS operations end in order: a wave's writes of the next chunk have ended once no more operations are under way
  // than the reads that it has issued behind them, two for each of the E - PD steps up to the barrier.  A wait for
  // 2 * PD of them, all that are needed later, covers the writes only if that is no more (RB = 3, NT = 1: 4, not 8).
  constexpr int kBehind = 2 * (E - PD), kUnderWay = 2 * PD < kBehind ? 2 * PD : kBehind;
  static_assert(E > PD && kUnderWay <= kBehind && kUnderWay <= 15, "the barrier's wait has to cover the LDS writes");
  constexpr int kChunk = CK * RB * 2;                          // activation fragments of a chunk
  constexpr bool PAIR = epi_pairs(EPI);
  constexpr int NI = mid_items(RB, NT), NQ = 2 * NI;           // items, quads of a wave
  constexpr int kLdsFr = 3 * kChunk > NQ * 2 ? 3 * kChunk : NQ * 2;   // ring; after the loop, half of the sums
  __shared__ u32x4_t lds[kLdsFr][64];
  __shared__ float s_rows[EPI == EPI_RESID ? 4 * RB * 32 : (RB * 32 > 256 ? RB * 32 : 256)];
  __shared__ float s_rstd[EPI != EPI_RESID ? RB * 32 : 1];
  __shared__ float s_pos[EPI == EPI_QKV ? 32 * RB : 1];
  __shared__ int s_crow[EPI == EPI_QKV ? 32 * RB : 1];
  __shared__ __attribute__((aligned(16))) float s_freq[64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int S = 1 << a.lgS;
  const int xcd = blockIdx.x, sp = (int)blockIdx.y & (S - 1), gm = (int)blockIdx.y >> a.lgS;
  const int ug = gm / a.m_tiles, mt = gm - ug * a.m_tiles;
  const int g = xcd * a.gpx + ug;
  const int t_begin = g * a.tq + min(g, a.trem);
  const int t_count = a.tq + (g < a.trem ? 1 : 0);
  if (t_count == 0) return;
  const int m0 = mt * RB * 32;
  const int n_tiles = a.N / kFragRows;
  const int c0 = sp * a.cq + min(sp, a.crem);
  const int n = a.cq + (sp < a.crem ? 1 : 0);                  // chunks of this slice

  // Lane (i, g) = (lane % 16, lane / 16) of v_mfma_f32_16x16x32_bf16 holds eight k-values of weight row (or
  // activation row) i.  Out of the 32-row fragments: k-half g % 2 of k-step KK * (g / 2) + kk, whichever way round
  // as long as both operands agree.  Coded weights: a 16-byte piece covers two k-steps (E4M3) or four (int4);
  // where it is all that a chunk takes (CW = 1), a lane fetches its half of it.
  typedef const __attribute__((address_space(1))) u32x4_t* gptr_t;
  typedef typename std::conditional<Sh::WU == 2, u32x2_t, u32x4_t>::type wload_t;
  typedef const __attribute__((address_space(1))) wload_t* wptr_t;
  constexpr int CW = Sh::CW, WU = Sh::WU;
  const int g16 = lane >> 4, i16 = lane & 15, in_frag = i16 + 32 * (g16 & 1);
  wptr_t wp = (wptr_t)((gptr_t)a.Wp + ((size_t)c0 * CW * n_tiles + t_begin) * 64);
  const unsigned w_row = n_tiles * 64u;
  const size_t w_step = (size_t)CW * w_row * WU;
  unsigned w_lane = in_frag * WU + (WU == 2 ? g16 >> 1 : (g16 >> 1) * w_row);
  gptr_t xp = (gptr_t)a.Xs + (size_t)c0 * CK * a.e.n_rb * 128;
  const unsigned x_step = CK * a.e.n_rb * 128u;
  unsigned x_off[LX];
#pragma unroll
  for (int i = 0; i < LX; ++i) {     // fragment f of the chunk: row block, k-step, hi / lo
    const int f = wave * LX + i;
    x_off[i] = ((unsigned)(f % (2 * CK) / 2) * a.e.n_rb + min(mt * RB + f / (2 * CK), a.e.n_rb - 1)) * 128u + (f & 1) * 64u + lane;
  }
  u32x4_t xin[D][LX];
  wload_t wr[D][2 * NT];
  int wl = n, xl = n;                                          // chunks still to be requested
  // (once nothing is left the loads repeat the first activations, which the caches hold: the number of
  // loads in flight stays fixed)
  auto issue_x = [&](int d) {
#pragma unroll
    for (int i = 0; i < LX; ++i) xin[d][i] = xp[x_off[i]];
    if (--xl > 0) xp += x_step;
    else xp = (gptr_t)a.Xs;
  };
  auto issue_w = [&](int d) {
#pragma unroll
    for (int t = 0; t < 2 * NT; ++t) {   // (beyond the group's tiles: the last one again, dropped at the end)
      const unsigned piece = (min(wave * NT + t / 2, t_count - 1) * 64u + (t & 1) * 16u) * WU;
      wr[d][t] = __builtin_nontemporal_load(wp + piece + w_lane);
    }
    const bool more = --wl > 0;
    wp = more ? wp + w_step : (wptr_t)a.Xs;
    w_lane = more ? w_lane : (unsigned)i16;
  };
  auto put_x = [&](int d, int buf) {
#pragma unroll
    for (int i = 0; i < LX; ++i) lds[buf * kChunk + wave * LX + i][lane] = xin[d][i];
  };

#pragma unroll
  for (int d = 0; d < D; ++d) {
    issue_x(d);
    issue_w(d);
    __builtin_amdgcn_sched_barrier(0);                         // (in this order: see SkinnyRing)
  }
  f32x4_t acc[R][2 * NT];                                      // 16 activation rows x 16 weight rows each
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int j = 0; j < 2 * NT; ++j) acc[i][j] = f32x4_t{};

  put_x(0, 0);
  issue_x(0);
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  u32x4_t xo[PD + 1][2];
  const u32x4_t* const x_lane = &lds[0][0] + (g16 >> 1) * KK * 128 + in_frag;
  auto get = [&](int s, int buf, int e) {                      // step e = kk * R + 16-row block
    const int r = e % R, f = buf * kChunk + ((r >> 1) * CK + e / R) * 2;
    xo[s][0] = x_lane[f * 64 + (r & 1) * 16];
    xo[s][1] = x_lane[(f + 1) * 64 + (r & 1) * 16];
  };
#pragma unroll
  for (int e = 0; e < PD; ++e) get(e, 0, e);
  int buf = 0, left = n;
  while (left > 0) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      // The next chunk's activations go to LDS now; the barrier before their first read is PD steps from
      // the end.  Their buffer held the chunk before the last one, which every wave had read before the
      // barrier of the last.
      const int nb = buf == 2 ? 0 : buf + 1;
      put_x((d + 1) % D, nb);
      issue_x((d + 1) % D);
      if (left > d) {
        bf16x8_t w[2 * NT];
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const int kk = e / R, r = e % R;
          if (e == E - PD) asm volatile("s_waitcnt lgkmcnt(%0)\n\ts_barrier" ::"n"(kUnderWay) : "memory");
          if (e + PD < E) get((e + PD) % (PD + 1), buf, e + PD);
          else get((e + PD) % (PD + 1), nb, e + PD - E);
          if (r == 0) {
#pragma unroll
            for (int t = 0; t < 2 * NT; ++t) w[t] = weight_operand<WF>(wr[d][t], kk);
          }
          // hi and lo of the same rows into the same sums, one after the other, then the next weights: the
          // cheapest order for the power that sets the clock
#pragma unroll
          for (int t = 0; t < 2 * NT; ++t) {
#pragma unroll
            for (int hl = 0; hl < 2; ++hl)
              acc[r][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[t], __builtin_bit_cast(bf16x8_t, xo[e % (PD + 1)][hl]), acc[r][t], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(kMfmaOrder);
          }
          __builtin_amdgcn_sched_barrier(0);   // left alone the scheduler sinks the operand reads to their use
        }
        buf = nb;
        if (E % (PD + 1) != 0) {               // the next chunk counts its steps from 0 again
          u32x4_t tmp[PD][2];
#pragma unroll
          for (int k = 0; k < PD; ++k)
#pragma unroll
            for (int hl = 0; hl < 2; ++hl) tmp[k][hl] = xo[(E + k) % (PD + 1)][hl];
#pragma unroll
          for (int k = 0; k < PD; ++k)
#pragma unroll
            for (int hl = 0; hl < 2; ++hl) xo[k][hl] = tmp[k][hl];
        }
      }
      issue_w(d);
    }
    left -= D;
  }
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // all waves have read the ring

  // ---- output ----
  // (row sums and rotary positions: see gemm_skinny)
  constexpr int kRows = RB * 32;
  SsqSums<kRows, 32> rows(a.e, m0, tid);
  if (EPI != EPI_RESID) rows.request();
  EpiRow er;
  if (EPI == EPI_QKV) er = epi_row_fetch(a.e, min(m0 + tid % kRows, a.e.M - 1));
  const size_t unit = (size_t)xcd * a.ucap + (size_t)gm * S;       // first workgroup of the group
  const auto gcnt = a.group_cnt + ((size_t)xcd * a.gcap + gm) * kCntStride;
  f32x4_t* const stage = reinterpret_cast<f32x4_t*>(&lds[0][0]) + lane;
  // item i = tile i % NT of this wave, rows 16 * (i / NT) ..: lane (i16, g) has activation row i16, quad g / 2 of the
  // tile and its partner, quad g / 2 + 2
  const int h = g16 & 1, p = g16 >> 1;
  auto item_quad = [&](int i, int qi) -> f32x4_t { return acc[i / NT][2 * (i % NT) + qi]; };
  const int b0 = mid_first(NI, a.lgS, sp), b1 = mid_first(NI, a.lgS, sp + 1);   // this slice's items
  f32x4_t* const own = stage + (size_t)wave * (NQ / 2) * 64;
  if (S > 1) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      if (i >= b0 && i < b1) {
        own[(i - b0) * 128] = item_quad(i, 0);
        own[(i - b0) * 128 + 64] = item_quad(i, 1);
      } else {
        f32x4_t* dst = a.xch + (unit + sp) * a.unit_stride + (size_t)(wave * (NQ + 1) + i * 2) * 64 + lane;
        dst[0] = item_quad(i, 0);
        dst[64] = item_quad(i, 1);
      }
    }
  }
  if (EPI != EPI_RESID) {
    const float ss = rows.sum();
    if (tid < rows.kParts * kRows) s_rows[tid] = ss;
  }
  if (EPI == EPI_QKV) epi_tables(a.e, er, tid, kRows, s_pos, s_crow, s_freq);
  if (EPI == EPI_RESID)
    for (int i = tid; i < 4 * RB * 32; i += 256) s_rows[i] = 0.f;
  if (S > 1) __builtin_amdgcn_s_waitcnt(0);         // this wave's sums are in the L2
  __syncthreads();
  if (EPI != EPI_RESID && tid < kRows) {            // 1 / rms of the rows, while the group meets
    const float t = s_rows[tid] + (rows.kParts > 1 ? s_rows[kRows + tid] : 0.f);
    s_rstd[tid] = 1.0f / sqrtf(t / (float)a.e.K + a.e.eps);
  }
  if (S > 1 && tid == 0) group_arrive_and_wait(gcnt, S, a.n_xcd, a.status);
  if (S > 1 || EPI != EPI_RESID) __syncthreads();
  if (S > 1) asm volatile("buffer_inv sc0" ::: "memory");          // drop stale L1 lines (the L2 is shared)
  struct Loads {
    EpiLoads l[PAIR ? 1 : 2];
  };
  auto fetch = [&](int i, Loads& l) {
    const int m = m0 + (i / NT) * 16 + i16, t = t_begin + min(wave * NT + i % NT, t_count - 1);
    epi_fetch<EPI, WF>(a.e, a.N, t, p, m, h, l.l[0]);
    if (!PAIR) epi_fetch<EPI, WF>(a.e, a.N, t, p + 2, m, h, l.l[PAIR ? 0 : 1]);
  };
  auto finish_item = [&](int i, const f32x4_t v0, const f32x4_t v1, const Loads& l) {
    const int ml = (i / NT) * 16 + i16, t = wave * NT + i % NT;
    if (t >= t_count) return;
    const float pos = EPI == EPI_QKV ? s_pos[ml] : 0.f;
    const int crow = EPI == EPI_QKV ? s_crow[ml] : 0;
    const float rs = EPI != EPI_RESID ? s_rstd[ml] : 1.f;
    float sq = epi_quad<EPI, WF>(a.e, a.N, t_begin + t, p, m0 + ml, h, rs, pos, crow, s_freq, v0, v1, l.l[0]);
    if (!PAIR) sq += epi_quad<EPI, WF>(a.e, a.N, t_begin + t, p + 2, m0 + ml, h, rs, pos, crow, s_freq, v1, v1, l.l[PAIR ? 0 : 1]);
    if (EPI == EPI_RESID) {
      sq = lane_quad16_sum(sq);
      if (lane < 16) s_rows[wave * RB * 32 + ml] += sq;    // (this lane's own word)
    }
  };
  auto finish = [&](auto split) {
    constexpr int SS = decltype(split)::value;
    constexpr int BT = SS == 8 ? 2 : (SS == 4 ? 3 : 4);    // items whose loads are in flight together
    for (int i0 = b0; i0 < b1; i0 += BT) {
      f32x4_t part[BT][2][SS];
      Loads ld[BT];
#pragma unroll
      for (int b = 0; b < BT; ++b) {
        const int i = min(i0 + b, b1 - 1);
#pragma unroll
        for (int s2 = 1; s2 < SS; ++s2) {
          const f32x4_t* p = a.xch + (unit + ((sp + s2) & (SS - 1))) * a.unit_stride + (size_t)(wave * (NQ + 1) + i * 2) * 64 + lane;
          part[b][0][s2] = p[0];
          part[b][1][s2] = p[64];
        }
        fetch(i, ld[b]);
        part[b][0][0] = own[(i - b0) * 128];
        part[b][1][0] = own[(i - b0) * 128 + 64];
      }
      asm volatile("" ::: "memory");
#pragma unroll
      for (int b = 0; b < BT; ++b) {
        if (i0 + b >= b1) break;
        f32x4_t v0 = part[b][0][0], v1 = part[b][1][0];
#pragma unroll
        for (int s2 = 1; s2 < SS; ++s2) {
          v0 += part[b][0][s2];
          v1 += part[b][1][s2];
        }
        finish_item(i0 + b, v0, v1, ld[b]);
      }
    }
  };
  if (S == 1) {
    // 16 rows at a time through LDS, so that the epilogue is a short loop
    f32x4_t* const st = stage + (size_t)wave * (NT * 2) * 64;
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
      for (int k = 0; k < NT; ++k) {
        st[(2 * k) * 64] = item_quad(r * NT + k, 0);
        st[(2 * k + 1) * 64] = item_quad(r * NT + k, 1);
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll 1
      for (int k = 0; k < NT; ++k) {
        Loads l;
        fetch(r * NT + k, l);
        finish_item(r * NT + k, st[(2 * k) * 64], st[(2 * k + 1) * 64], l);
      }
    }
  } else if (S == 2) finish(std::integral_constant<int, 2>{});
  else if (S == 4) finish(std::integral_constant<int, 4>{});
  else finish(std::integral_constant<int, 8>{});

  // Partial sums of x^2 of the new rows: every slice that has finished items of a row writes what it
  // has of its rows to a plane of its own; the last of them clears the planes that are left over.
  if (EPI == EPI_RESID && a.e.next_gain) {
    __syncthreads();
    for (int ml = tid; ml < RB * 32; ml += 256) {
      const int r = ml >> 4;
      const int o0 = mid_owner(NI, a.lgS, r * NT), o1 = mid_owner(NI, a.lgS, (r + 1) * NT - 1);
      if (sp < o0 || sp > o1 || m0 + ml >= a.e.m_pad) continue;
      float* dst = a.e.ssq_out + (size_t)(g * a.planes + sp - o0) * a.e.m_pad + m0 + ml;
      *dst = (s_rows[ml] + s_rows[RB * 32 + ml]) + (s_rows[2 * RB * 32 + ml] + s_rows[3 * RB * 32 + ml]);
      if (sp == o1)
        for (int p = o1 - o0 + 1; p < a.planes; ++p) dst[(size_t)(p - (sp - o0)) * a.e.m_pad] = 0.f;
    }
  }
  if (S > 1 && tid == 0) group_leave(gcnt, S);
}

}  // namespace sv
#endif
