// Float32 models (and the LM head on raw rows): products on the float32 matrix instruction and the tree
// attention, any sizes.
//
// These models are small: a launch moves little and its time is a chain of memory round trips, so a layer is
// five launches (it was nine) and every launch asks for its operands at once: no staging, the waves of a
// workgroup split K, both operands go from memory into matrix-core operands, the norm's row sums of x^2 come
// from the very values that are multiplied, and the epilogue follows in the same launch.
#ifndef SV_F32_H
#define SV_F32_H

#include "sv_epilogue.h"

namespace sv {

template <typename TW, typename TG>
struct F32Args {
  const float* X;            // [M, K]
  const TG* gain;            // QKV, SWIGLU, OUT: RMSNorm of the rows of X, gain [K]
  const TW* W;               // [rows, K]
  int M, N, K;               // N: outputs per row; rotary or gate/up pairs where the epilogue works on pairs
  float eps;
  float* out;                // RESID: x [M, N], added to; OUT: logits [M, N]; SWIGLU: [M, N]; QKV: q [M, D]
  // EPI_QKV
  float* kc;                 // caches [B][nh][cap][d]
  float* vc;
  const int32_t* depth;
  const int32_t* prefix_len;
  int p_max, cap, T, nh, d;
  float theta;
};

// four consecutive values from p on; VEC: one load
template <bool VEC>
__device__ inline f32x4_t f32_quad(const float* p, int left) {
  if (VEC) return *reinterpret_cast<const f32x4_t*>(p);
  f32x4_t v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (j < left) v[j] = p[j];
  return v;
}
template <bool VEC>
__device__ inline f32x4_t f32_quad(const bf16_t* p, int left) {
  if (VEC) {
    const uint2 r = *reinterpret_cast<const uint2*>(p);
    return f32x4_t{bf16_lo_f32(r.x), bf16_hi_f32(r.x), bf16_lo_f32(r.y), bf16_hi_f32(r.y)};
  }
  f32x4_t v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (j < left) v[j] = to_f32(p[j]);
  return v;
}

// Y = X W^T with the epilogue EPI (see sv_epilogue.h for their names).
// A workgroup makes RT x CT tiles of 16 rows x 16 outputs; its NW waves take the 16-value pieces of K in turn.
// v_mfma_f32_16x16x4_f32 with W as the first operand: lane l holds W[row l % 16] and X[row l % 16] at k-values
// 4 * (l / 16) .. + 3 of a piece (one 16-byte load each; instruction j multiplies element j of all lanes) and
// the sums of activation row l % 16, outputs 4 * (l / 16) .. + 3.  Where the epilogue works on pairs, tiles 2i
// and 2i + 1 hold the partners.
// VEC: K a multiple of 4, operands aligned for it.   grid = (outputs, rows), block = 64 * NW.
template <int EPI, int RT, int CT, int NW, bool VEC, typename TW, typename TG>
__global__ __launch_bounds__(64 * NW) void f32_product(const F32Args<TW, TG> a) {
  constexpr bool PAIR = epi_pairs(EPI), NORM = EPI != EPI_RESID;
  constexpr int CG = PAIR ? CT / 2 : CT;                 // groups of 16 outputs
  constexpr int U = RT * CT <= 2 ? 4 : 2;                // pieces whose loads are in flight together
  __shared__ f32x4_t s_acc[NW][RT * CT][64];
  __shared__ float s_ss[NORM ? NW : 1][NORM ? RT * 16 : 1];
  __shared__ float s_cs[EPI == EPI_QKV ? RT * 16 * CG * 16 : 1], s_sn[EPI == EPI_QKV ? RT * 16 * CG * 16 : 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane & 15, kq = lane >> 4;
  const int m0 = blockIdx.y * RT * 16, n0 = blockIdx.x * CG * 16;
  const int half = a.d >> 1, D = a.nh * a.d;

  const float* xp[RT];
  const TW* wp[CT];
#pragma unroll
  for (int i = 0; i < RT; ++i) xp[i] = a.X + (size_t)min(m0 + 16 * i + r16, a.M - 1) * a.K;
#pragma unroll
  for (int t = 0; t < CT; ++t) {
    const int n = min(n0 + 16 * (PAIR ? t >> 1 : t) + r16, a.N - 1);
    size_t row = n;
    if (EPI == EPI_SWIGLU) row = (size_t)n + (t & 1) * a.N;
    if (EPI == EPI_QKV) row = (size_t)(n / half) * a.d + n % half + (t & 1) * half;   // q, k, v heads follow each other
    wp[t] = a.W + row * a.K;
  }
  f32x4_t xv[U][RT], wv[U][CT], gv[U];
  auto load = [&](int c0) {                              // this wave's pieces c0, c0 + NW, ...
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = (c0 + u * NW) * 16 + 4 * kq, left = a.K - k;
      const bool on = left > 0;
      const int kk = on ? k : 0;
#pragma unroll
      for (int i = 0; i < RT; ++i) xv[u][i] = f32_quad<VEC>(xp[i] + kk, left);
#pragma unroll
      for (int t = 0; t < CT; ++t) wv[u][t] = f32_quad<VEC>(wp[t] + kk, left);
      if (NORM) gv[u] = f32_quad<VEC>(a.gain + kk, left);
      if (VEC && !on) {
#pragma unroll
        for (int i = 0; i < RT; ++i) xv[u][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < CT; ++t) wv[u][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if (NORM) gv[u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      }
    }
  };
  const int pieces = (a.K + 15) / 16;
  load(wave);

  if (EPI == EPI_QKV) {
    // Rotation of the workgroup's rows and pairs, while the loads are under way.  The angle is evaluated in
    // double so that positions in the thousands keep 1e-5 parity.
    for (int i = tid; i < RT * 16 * CG * 16; i += 64 * NW) {
      const int m = min(m0 + i / (CG * 16), a.M - 1), n = min(n0 + i % (CG * 16), a.N - 1);
      int P = a.prefix_len[m / a.T];
      P = P < 0 ? 0 : (P > a.p_max ? a.p_max : P);
      const double inv = pow((double)a.theta, -2.0 * (double)(n % half) / (double)a.d);
      double s_ = 0.0, c_ = 1.0;
      if (n < 2 * a.nh * half) sincos((double)(P + a.depth[m]) * inv, &s_, &c_);   // (v is not rotated)
      s_cs[i] = (float)c_;
      s_sn[i] = (float)s_;
    }
  }

  f32x4_t acc[RT][CT];
  float ss[RT];
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    ss[i] = 0.f;
#pragma unroll
    for (int t = 0; t < CT; ++t) acc[i][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }
  for (int c = wave; c < pieces; c += U * NW) {
    f32x4_t x[U][RT], w[U][CT];
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int i = 0; i < RT; ++i) {
        x[u][i] = xv[u][i];
        if (NORM) {
#pragma unroll
          for (int j = 0; j < 4; ++j) ss[i] += x[u][i][j] * x[u][i][j];
          x[u][i] *= gv[u];
        }
      }
#pragma unroll
      for (int t = 0; t < CT; ++t) w[u][t] = wv[u][t];
    }
    if (c + U * NW < pieces) load(c + U * NW);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
          for (int t = 0; t < CT; ++t) acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u][t][j], x[u][i][j], acc[i][t], 0, 0, 0);
  }

#pragma unroll
  for (int i = 0; i < RT; ++i) {
#pragma unroll
    for (int t = 0; t < CT; ++t) s_acc[wave][i * CT + t][lane] = acc[i][t];
    if (NORM) {
      float s = ss[i];
      s += __shfl_xor(s, 16, kWave);
      s += __shfl_xor(s, 32, kWave);
      if (kq == 0) s_ss[wave][i * 16 + r16] = s;
    }
  }
  __syncthreads();
  // units (row tile, output group) are dealt to the waves; the waves' sums are added in order
  for (int u = wave; u < RT * CG; u += NW) {
    const int i = u / CG, g = u % CG;
    const int m = m0 + 16 * i + r16;
    f32x4_t v0 = s_acc[0][i * CT + (PAIR ? 2 * g : g)][lane], v1 = v0;
    if (PAIR) v1 = s_acc[0][i * CT + 2 * g + 1][lane];
#pragma unroll
    for (int w = 1; w < NW; ++w) {
      v0 += s_acc[w][i * CT + (PAIR ? 2 * g : g)][lane];
      if (PAIR) v1 += s_acc[w][i * CT + 2 * g + 1][lane];
    }
    if (NORM) {
      float s = s_ss[0][i * 16 + r16];
#pragma unroll
      for (int w = 1; w < NW; ++w) s += s_ss[w][i * 16 + r16];
      const float rstd = 1.0f / sqrtf(s / (float)a.K + a.eps);
      v0 *= rstd;
      v1 *= rstd;
    }
    if (m >= a.M) continue;
    const int nb = n0 + 16 * g + 4 * kq;
    if (EPI == EPI_QKV) {
      const int b = m / a.T, t = m - b * a.T;
      int P = a.prefix_len[b];
      P = P < 0 ? 0 : (P > a.p_max ? a.p_max : P);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int n = nb + j;
        if (n >= a.N) continue;
        const int head3 = n / half, jj = n - head3 * half, which = head3 / a.nh, h = head3 - which * a.nh;
        const float c = s_cs[(i * 16 + r16) * CG * 16 + 16 * g + 4 * kq + j], s = s_sn[(i * 16 + r16) * CG * 16 + 16 * g + 4 * kq + j];
        const float e0 = which == 2 ? v0[j] : v0[j] * c - v1[j] * s, e1 = which == 2 ? v1[j] : v1[j] * c + v0[j] * s;
        float* dst = which == 0 ? a.out + (size_t)m * D + h * a.d
                                : (which == 1 ? a.kc : a.vc) + (((size_t)b * a.nh + h) * a.cap + (size_t)(P + t)) * a.d;
        dst[jj] = e0;
        dst[jj + half] = e1;
      }
    } else {
      float* dst = a.out + (size_t)m * a.N + nb;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (nb + j >= a.N) continue;
        if (EPI == EPI_RESID) dst[j] += v0[j];
        else if (EPI == EPI_SWIGLU) dst[j] = v0[j] / (1.0f + expf(-v0[j])) * v1[j];
        else dst[j] = v0[j];
      }
    }
  }
}

// Few outputs: one tile (pair) per workgroup, 8 waves along K, so that many CUs ask for the weights and each
// wave has one or two round trips.  From 96 workgroups of 64 x 64 outputs on, those: every operand is then
// used four times as often.  us, 16 x 16 / 64 x 64 outputs at so many of the latter: float32, K = 256: 16: 10.3 /
// 14.3, 128: 25.0 / 15.6, 512: 75.7 / 26.9; bf16 weights, K = 4096: 60: 69 / 106, 128: 136 / 109, 500: 506 / 189.
template <int EPI, typename TW, typename TG>
void f32_launch(const F32Args<TW, TG>& a, hipStream_t st) {
  const bool vec = a.K % 4 == 0 && (uintptr_t)a.X % 16 == 0 && (uintptr_t)a.W % (4 * sizeof(TW)) == 0 &&
                   (EPI == EPI_RESID || (uintptr_t)a.gain % (4 * sizeof(TG)) == 0);
  constexpr int P = epi_pairs(EPI) ? 2 : 1;
  const long long big = (long long)ceil_div(a.M, 64) * ceil_div(a.N, 64 / P);
  const dim3 wide(ceil_div(a.N, 64 / P), ceil_div(a.M, 64)), small(ceil_div(a.N, 16), ceil_div(a.M, 16));
  if (big >= 96) {
    if (vec) f32_product<EPI, 4, 4, 4, true, TW, TG><<<wide, 256, 0, st>>>(a);
    else f32_product<EPI, 4, 4, 4, false, TW, TG><<<wide, 256, 0, st>>>(a);
  } else {
    if (vec) f32_product<EPI, 1, P, 8, true, TW, TG><<<small, 512, 0, st>>>(a);
    else f32_product<EPI, 1, P, 8, false, TW, TG><<<small, 512, 0, st>>>(a);
  }
}

// ---------------------------------------------------------------------------------------
// Tree attention of float32 models: one workgroup per (query node, head); the node attends to every prefix
// key and to the tree nodes whose bit is set in its ancestor mask.  A thread takes a key: all 256 dot products
// of a pass (head_dim values each) have their loads in flight together; then the threads are dealt over (value
// columns, key groups) for the second product.  Online softmax in float32 between passes of 256 keys.
// (One wave per query walking the keys one after the other, as before, is a chain of as many memory round
// trips and reductions as there are keys.)
// VW: values per load (4 where head_dim and the caches allow it).   grid = (M, nh), block = 256.
// ---------------------------------------------------------------------------------------
template <int VW>
__global__ __launch_bounds__(256) void tree_attention_f32(
    const float* __restrict__ q, const float* __restrict__ kc, const float* __restrict__ vc,
    const int32_t* __restrict__ prefix_len, int p_max, const uint64_t* __restrict__ anc,
    int n_words, int T, int nh, int d, int cap, float* __restrict__ out) {
  __shared__ float s_q[128], s_p[256], s_red[8], s_o[256 * VW];
  const int tid = threadIdx.x, m = blockIdx.x, h = blockIdx.y;
  const int b = m / T;
  const size_t D = (size_t)nh * d;
  int P = prefix_len[b];
  P = P < 0 ? 0 : (P > p_max ? p_max : P);
  const int nkeys = P + T;
  const uint64_t mask0 = anc[(size_t)m * n_words], mask1 = n_words > 1 ? anc[(size_t)m * n_words + 1] : 0ull;
  const float* kb = kc + ((size_t)b * nh + h) * cap * d;
  const float* vb = vc + ((size_t)b * nh + h) * cap * d;
  const float scale = 1.0f / sqrtf((float)d);
  if (tid < d) s_q[tid] = q[m * D + (size_t)h * d + tid] * scale;
  __syncthreads();
  const int nd = d / VW, groups = 256 / nd, dq = tid % nd, kg = tid / nd;   // (threads beyond groups * nd idle)
  float o[VW], l = 0.f, mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < VW; ++i) o[i] = 0.f;
  for (int j0 = 0; j0 < nkeys; j0 += 256) {
    const int j = j0 + tid, node = j - P;
    const bool vis = j < P || (j < nkeys && ((node < 64 ? mask0 >> node : mask1 >> (node - 64)) & 1ull));
    float s = -INFINITY;
    if (vis) {
      const float* kr = kb + (size_t)j * d;
      float part[VW];
#pragma unroll
      for (int i = 0; i < VW; ++i) part[i] = 0.f;
#pragma unroll 8
      for (int e = 0; e < nd; ++e) {
        if (VW == 4) {
          const f32x4_t kv = *reinterpret_cast<const f32x4_t*>(kr + 4 * e);
#pragma unroll
          for (int i = 0; i < VW; ++i) part[i] = fmaf(s_q[4 * e + i], kv[i], part[i]);
        } else {
          part[0] = fmaf(s_q[e], kr[e], part[0]);
        }
      }
      s = part[0];
#pragma unroll
      for (int i = 1; i < VW; ++i) s += part[i];
    }
    float top = s;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) top = fmaxf(top, __shfl_xor(top, off, kWave));
    if ((tid & 63) == 0) s_red[tid >> 6] = top;
    __syncthreads();
    const float mn = fmaxf(mx, fmaxf(fmaxf(s_red[0], s_red[1]), fmaxf(s_red[2], s_red[3])));
    const float corr = mx == mn ? 1.f : expf(mx - mn);      // exp(-inf) = 0 in the first pass
    const float p = vis ? expf(s - mn) : 0.f;
    s_p[tid] = vis ? p : -1.f;                               // a key that is not visible is not read
    const float ps = wave_sum(p);
    if ((tid & 63) == 0) s_red[4 + (tid >> 6)] = ps;
    __syncthreads();
    l = l * corr + ((s_red[4] + s_red[5]) + (s_red[6] + s_red[7]));
    mx = mn;
    if (kg < groups) {
#pragma unroll
      for (int i = 0; i < VW; ++i) o[i] *= corr;
      const int n = min(256, nkeys - j0);
#pragma unroll 4
      for (int jj = kg; jj < n; jj += groups) {
        const float pj = s_p[jj];
        if (pj < 0.f) continue;
        const float* vr = vb + (size_t)(j0 + jj) * d + dq * VW;
        if (VW == 4) {
          const f32x4_t v = *reinterpret_cast<const f32x4_t*>(vr);
#pragma unroll
          for (int i = 0; i < VW; ++i) o[i] = fmaf(pj, v[i], o[i]);
        } else {
          o[0] = fmaf(pj, vr[0], o[0]);
        }
      }
    }
    __syncthreads();
  }
  if (kg < groups) {
#pragma unroll
    for (int i = 0; i < VW; ++i) s_o[kg * d + dq * VW + i] = o[i];
  }
  __syncthreads();
  if (tid < d) {
    float v = 0.f;
    for (int g = 0; g < groups; ++g) v += s_o[g * d + tid];
    out[m * D + (size_t)h * d + tid] = v * (1.0f / l);
  }
}

}  // namespace sv
#endif
