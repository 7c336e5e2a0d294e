// C-ABI entry points of libspecvla_verify: argument checks, launch planning, launches.
// No allocation, no global state, no synchronisation.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <mutex>

#include "specvla_verify.h"
#include "specvla_verify_aux.h"
#include "sv_accept.h"
#include "sv_attention.h"
#include "sv_f32.h"
#include "sv_internal.h"
#include "sv_kernels.h"
#include "sv_pack.h"
#include "sv_products.h"
#include "sv_tree_build.h"

namespace sv {

static int check_cfg(const sv_model_cfg* c) {
  if (!c) return SV_ERR_NULL;
  if (c->dtype != SV_F32 && c->dtype != SV_BF16 && c->dtype != SV_BF16_W8 && c->dtype != SV_BF16_W4)
    return SV_ERR_DTYPE;
  if (c->hidden < 1 || c->n_heads < 1 || c->head_dim < 2 || c->mlp_dim < 1 || c->vocab < 1)
    return SV_ERR_SHAPE;
  if ((c->head_dim & 1) || c->head_dim > 128) return SV_ERR_SHAPE;
  if (!(c->rms_eps >= 0.f) || !(c->rope_theta > 0.f)) return SV_ERR_SHAPE;
  if (c->dtype != SV_F32) {
    if (c->hidden % 256 || c->head_dim != 128 || c->n_heads % 2 || c->mlp_dim % 256)
      return SV_ERR_SHAPE;
  }
  return SV_OK;
}

// Workgroups that share the keys of one (episode, head, 16 queries) task of the tree attention:
// more than one where the tasks alone would leave the chip short of waves (long prefix, one
// episode), at least 8 key tiles each.
static int attention_splits(int n_tasks, int n_keys) {
  int s = 1;
  while (s < 8 && n_tasks * s < kAttSplitFill && (n_keys / kAttKeys) / (2 * s) >= 8) s *= 2;
  return s;
}

static int device_xcds() {
  static int cached[64] = {0};               // hardware facts only; a race rewrites the same value
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 1;
  if (cached[dev] == 0) {
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) cus = 32;
    int x = cus / 32;
    cached[dev] = x < 1 ? 1 : (x > kXcds ? kXcds : x);
  }
  return cached[dev];
}

static int weight_format(const sv_model_cfg& c) { return c.dtype == SV_BF16_W8 ? 1 : (c.dtype == SV_BF16_W4 ? 2 : 0); }

// The four products of a layer (bf16 models) and the head's, for one XCD count.
struct LayerPlan {
  ProductPlan qkv, o, gu, down;
};
static LayerPlan plan_layer(const sv_model_cfg& c, int m_rows, int n_xcd) {
  const int H = c.hidden, D = c.n_heads * c.head_dim, F = c.mlp_dim, wf = weight_format(c);
  LayerPlan p;
  p.qkv = plan_product(m_rows, 3 * D, H, wf, n_xcd);
  p.o = plan_product(m_rows, H, D, wf, n_xcd);
  p.gu = plan_product(m_rows, 2 * F, H, wf, n_xcd);
  p.down = plan_product(m_rows, H, F, wf, n_xcd);
  return p;
}

static WorkspaceLayout workspace_layout(const sv_model_cfg& c, int m_rows, int n_scored) {
  const size_t H = c.hidden, D = (size_t)c.n_heads * c.head_dim, F = c.mlp_dim;
  WorkspaceLayout L;
  memset(&L, 0, sizeof(L));
  const size_t mp = (size_t)ceil_div(m_rows, kRowPad) * kRowPad;
  L.n_rb = ceil_div(m_rows, 32);
  L.m_pad = c.dtype == SV_F32 ? (int)mp : L.n_rb * 32;
  size_t o = 0;
  if (c.dtype != SV_F32) {
    // sized for the largest split over the XCD counts a device can have
    const size_t mr = L.m_pad;
    size_t xch = 0, planes = H / 256;
    for (int n_xcd = 1; n_xcd <= kXcds; n_xcd *= 2) {
      const LayerPlan p = plan_layer(c, m_rows, n_xcd);
      for (const ProductPlan* q : {&p.qkv, &p.o, &p.gu, &p.down}) {
        const size_t x = (size_t)n_xcd * q->wg_x * q->unit_stride * 16;
        xch = x > xch ? x : xch;
      }
      for (const ProductPlan* q : {&p.o, &p.down}) planes = (size_t)q->n_planes > planes ? q->n_planes : planes;
    }
    L.counter_bytes = align_up((kMaxGroups * kCntStride + 64) * sizeof(int), kAlign);   // group counters + status word
    L.counters = o; o += L.counter_bytes;
    L.xs_x = o;     o = align_up(o + mr * H * 4, kAlign);
    L.xs_attn = o;  o = align_up(o + mr * D * 4, kAlign);
    L.xs_act = o;   o = align_up(o + mr * F * 4, kAlign);
    L.ssq = o;      o = align_up(o + mr * planes * 4, kAlign);
    L.xch = o;      o = align_up(o + xch, kAlign);
    L.q = o;        o = align_up(o + mr * D * 4, kAlign);
    L.attn = o;     o = align_up(o + mr * D * 4, kAlign);
    // partial results of the tree attention when the keys of a task are split
    L.att_part = o; o = align_up(o + 8 * mr * c.n_heads * kAttPartStride * 4, kAlign);
  } else {
    L.q = o;        o = align_up(o + mp * D * 4, kAlign);
    L.attn = o;     o = align_up(o + mp * D * 4, kAlign);
    L.act = o;      o = align_up(o + mp * F * 4, kAlign);
  }
  L.head_logits = o; o = align_up(o + mp * (size_t)(n_scored > 0 ? n_scored : 0) * 4, kAlign);
  // (the regions above do not move with n_scored: a layer call finds them without knowing it)
  if (c.dtype != SV_F32 && n_scored > 0 && n_scored % kFragRows == 0) {
    size_t xch = 0;
    for (int n_xcd = 1; n_xcd <= kXcds; n_xcd *= 2) {
      const ProductPlan p = plan_head(m_rows, n_scored, (int)H, n_xcd);
      const size_t x = (size_t)n_xcd * p.wg_x * p.unit_stride * 16;
      xch = x > xch ? x : xch;
    }
    L.head_xs = o;  o = align_up(o + (size_t)L.m_pad * H * 4, kAlign);
    L.head_ssq = o; o = align_up(o + (size_t)L.m_pad * (H / 256) * 4, kAlign);
    L.head_xch = o; o = align_up(o + xch, kAlign);
  }
  // (Once a product's ring has used up its weights it goes on reading the first of its activation fragments, a KiB per
  // weight tile of the workgroup: twelve at most, and the fragments of 32 rows have 32 KiB and more.)
  L.total = o;
  return L;
}

// Packed head: float32 gain, then the scored rows in fragment order.
struct HeadLayout {
  size_t gain, w, total;
};
static HeadLayout head_layout(const sv_model_cfg& c, int n) {
  HeadLayout L;
  L.gain = 0;
  L.w = align_up((size_t)c.hidden * 4, kAlign);
  L.total = L.w + align_up((size_t)n * c.hidden * 2, kAlign);
  return L;
}
static int check_packed_head(const sv_model_cfg* cfg, int vocab_lo, int vocab_hi) {
  const int rc = check_cfg(cfg);
  if (rc != SV_OK) return rc;
  if (cfg->dtype == SV_F32) return SV_ERR_DTYPE;
  if (vocab_lo < 0 || vocab_lo >= vocab_hi || vocab_hi > cfg->vocab ||
      (vocab_hi - vocab_lo) % kFragRows)
    return SV_ERR_SHAPE;
  return SV_OK;
}

static inline int launch_status() { return hipGetLastError() == hipSuccess ? SV_OK : SV_ERR_LAUNCH; }

__global__ void zero_ints(int* p, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// ---- float32 models: five launches per layer ------------------------------------------------

static int verify_layer_f32(const sv_model_cfg& c, const WorkspaceLayout& wl, const char* packed, float* x,
                            const sv_kv_view& kv, const sv_tree& tree, int B, char* ws,
                            hipStream_t st, hipEvent_t* ev) {
  const int T_ = tree.n_nodes, M = B * T_;
  auto mark = [&](int i) {
    if (ev) (void)hipEventRecord(ev[i], st);
  };
  const int H = c.hidden, d = c.head_dim, D = c.n_heads * d, F = c.mlp_dim;
  const PackedLayout pl = packed_layout(c);
  float* q = (float*)(ws + wl.q);
  float* attn = (float*)(ws + wl.attn);
  float* act = (float*)(ws + wl.act);
  auto product = [&](auto epi, const float* X, size_t w_off, const float* gain, int N, int K, float* out) {
    F32Args<float, float> a;
    memset(&a, 0, sizeof(a));
    a.X = X; a.gain = gain; a.W = (const float*)(packed + w_off); a.M = M; a.N = N; a.K = K; a.eps = c.rms_eps; a.out = out;
    a.kc = (float*)kv.k; a.vc = (float*)kv.v; a.depth = tree.depth; a.prefix_len = kv.prefix_len; a.p_max = kv.prefix_len_max;
    a.cap = kv.capacity; a.T = T_; a.nh = c.n_heads; a.d = d; a.theta = c.rope_theta;
    f32_launch<decltype(epi)::value>(a, st);
  };
  mark(0);
  product(std::integral_constant<int, EPI_QKV>{}, x, pl.wqkv, (const float*)(packed + pl.g1), 3 * D / 2, H, q);
  mark(1);
  mark(2);
  auto attention = d % 4 == 0 && (uintptr_t)kv.k % 16 == 0 && (uintptr_t)kv.v % 16 == 0 ? tree_attention_f32<4> : tree_attention_f32<1>;
  attention<<<dim3(M, c.n_heads), 256, 0, st>>>(q, (const float*)kv.k, (const float*)kv.v, kv.prefix_len, kv.prefix_len_max,
                                                tree.anc_mask, tree.n_words, T_, c.n_heads, d, kv.capacity, attn);
  mark(3);
  product(std::integral_constant<int, EPI_RESID>{}, attn, pl.wo, nullptr, H, D, x);
  mark(4);
  mark(5);
  product(std::integral_constant<int, EPI_SWIGLU>{}, x, pl.wgu, (const float*)(packed + pl.g2), F, H, act);
  mark(6);
  mark(7);
  product(std::integral_constant<int, EPI_RESID>{}, act, pl.wd, nullptr, H, F, x);
  mark(8);
  return launch_status();
}

// ---- bf16 models: five launches per layer ---------------------------------------------------

// What the layers of one call have in common.
struct LayerCall {
  WorkspaceLayout wl;
  LayerPlan plan;
  int n_xcd;
};
static LayerCall layer_call(const sv_model_cfg& c, int m_rows) {
  LayerCall l;
  l.wl = workspace_layout(c, m_rows, 0);
  if (c.dtype != SV_F32) {
    l.n_xcd = device_xcds();
    l.plan = plan_layer(c, m_rows, l.n_xcd);
  }
  return l;
}

// first: x has to be turned into fragments here (otherwise the layer before has left them in the
// workspace); next_packed: the layer after this one, whose first gain goes into the fragments this layer
// leaves (NULL: it leaves none).
static int verify_layer_bf16(const sv_model_cfg& c, const LayerCall& lc, const char* packed, float* x,
                             const sv_kv_view& kv, const sv_tree& tree, int B, char* ws, hipStream_t st,
                             hipEvent_t* ev, bool first, const char* next_packed) {
  const int T_ = tree.n_nodes, M = B * T_;
  auto mark = [&](int i) {
    if (ev) (void)hipEventRecord(ev[i], st);
  };
  const int H = c.hidden, D = c.n_heads * c.head_dim, F = c.mlp_dim, wf = weight_format(c);
  const PackedLayout pl = packed_layout(c);
  const WorkspaceLayout& wl = lc.wl;
  uint4* xs_x = (uint4*)(ws + wl.xs_x);
  uint4* xs_attn = (uint4*)(ws + wl.xs_attn);
  uint4* xs_act = (uint4*)(ws + wl.xs_act);
  float* ssq = (float*)(ws + wl.ssq);
  float* q = (float*)(ws + wl.q);
  float* attn = (float*)(ws + wl.attn);
  ProductScratch scratch;
  scratch.xch = (f32x4_t*)(ws + wl.xch);
  scratch.group_cnt = (unsigned*)(ws + wl.counters);
  scratch.status = (int*)(ws + wl.counters + wl.counter_bytes) - 1;   // last word of the counter region
  auto epilogue = [&](int K, size_t scale_off) {
    EpiArgs e;
    memset(&e, 0, sizeof(e));
    e.M = M; e.n_rb = wl.n_rb; e.m_pad = wl.m_pad; e.K = K; e.eps = c.rms_eps;
    e.wscale = wf ? (const float*)(packed + scale_off) : nullptr;
    return e;
  };
  auto product = [&](const ProductPlan& p, int epi, const uint4* xs, size_t w_off, int N, int K, const EpiArgs& e) {
    launch_product(p, epi, wf, lc.n_xcd, xs, (const uint4*)(packed + w_off), N, K, scratch, e, st);
  };
  if (first)
    split_gain_kernel<<<dim3(wl.n_rb * 4, H / 256), 256, 0, st>>>(x, (const float*)(packed + pl.g1), M, H, wl.m_pad, wl.n_rb, xs_x, ssq);
  mark(0);
  {
    EpiArgs e = epilogue(H, pl.sqkv);
    e.ssq = ssq; e.n_ssq = first ? H / 256 : lc.plan.down.n_planes;
    e.q_out = q; e.kc = (bf16_t*)kv.k; e.vc = (bf16_t*)kv.v; e.depth = tree.depth; e.prefix_len = kv.prefix_len;
    e.p_max = kv.prefix_len_max; e.cap = kv.capacity; e.T = T_; e.nh = c.n_heads; e.theta = c.rope_theta;
    product(lc.plan.qkv, EPI_QKV, xs_x, pl.wqkv, 3 * D, H, e);
  }
  mark(1);
  mark(2);
  {
    const int ns = attention_splits(B * ceil_div(T_, kAttQ) * c.n_heads, kv.prefix_len_max + T_);
    float* apart = (float*)(ws + wl.att_part);
    tree_attention_mfma<4><<<dim3(B * ceil_div(T_, kAttQ), c.n_heads, ns), 256, 0, st>>>(
        q, (const bf16_t*)kv.k, (const bf16_t*)kv.v, kv.prefix_len, kv.prefix_len_max,
        tree.anc_mask, tree.n_words, T_, c.n_heads, kv.capacity, attn, xs_attn, wl.n_rb, apart, M);
    if (ns > 1)
      attention_merge_kernel<<<dim3(M, ceil_div(c.n_heads, 16)), 256, 0, st>>>(apart, ns, M, c.n_heads, attn, xs_attn, wl.n_rb);
  }
  mark(3);
  {
    EpiArgs e = epilogue(D, pl.so);
    e.x = x; e.next_gain = (const float*)(packed + pl.g2); e.xs_out = xs_x; e.ssq_out = ssq;
    product(lc.plan.o, EPI_RESID, xs_attn, pl.wo, H, D, e);
  }
  mark(4);
  mark(5);
  {
    EpiArgs e = epilogue(H, pl.sgu);
    e.ssq = ssq; e.n_ssq = lc.plan.o.n_planes; e.xs_out = xs_act;
    product(lc.plan.gu, EPI_SWIGLU, xs_x, pl.wgu, 2 * F, H, e);
  }
  mark(6);
  mark(7);
  {
    EpiArgs e = epilogue(F, pl.sd);
    e.x = x;
    if (next_packed) {
      e.next_gain = (const float*)(next_packed + pl.g1); e.xs_out = xs_x; e.ssq_out = ssq;
    }
    product(lc.plan.down, EPI_RESID, xs_act, pl.wd, H, F, e);
  }
  mark(8);
  return launch_status();
}

template <typename T>
static int pack_layer_t(const sv_model_cfg& c, const sv_layer_weights& w, char* packed,
                        hipStream_t st) {
  const PackedLayout pl = packed_layout(c);
  const int H = c.hidden, D = c.n_heads * c.head_dim, F = c.mlp_dim;
  pack_gain<T><<<ceil_div(H, 256), 256, 0, st>>>((const T*)w.g1, (float*)(packed + pl.g1), H);
  pack_gain<T><<<ceil_div(H, 256), 256, 0, st>>>((const T*)w.g2, (float*)(packed + pl.g2), H);
  // float32: q|k|v and gate|up stacked, row-major.  bf16: fragment order with the row
  // permutations of the tile-local epilogues (rotary pairs / gate-up pairs 16 lanes apart).
  struct Piece {
    const void* src; size_t dst; int rows, k;
    int plain_off;                 // float32: first destination row
    int mode, off, tiles;          // bf16: see pack_rows; tiles of the whole fused matrix
  };
  const Piece pieces[] = {
      {w.wq, pl.wqkv, D, H, 0, PACK_PAIR16_HEAD, 0, 3 * D / 32},
      {w.wk, pl.wqkv, D, H, D, PACK_PAIR16_HEAD, D, 3 * D / 32},
      {w.wv, pl.wqkv, D, H, 2 * D, PACK_PAIR16_HEAD, 2 * D, 3 * D / 32},
      {w.wo, pl.wo, H, D, 0, PACK_PLAIN, 0, H / 32},
      {w.wg, pl.wgu, F, H, 0, PACK_PAIR16_GU, 0, F / 16},
      {w.wu, pl.wgu, F, H, F, PACK_PAIR16_GU, 16, F / 16},
      {w.wd, pl.wd, H, F, 0, PACK_PLAIN, 0, H / 32}};
  for (const Piece& p : pieces) {
    if (c.dtype == SV_F32) {
      const size_t n = (size_t)p.rows * p.k;
      pack_rows_plain<float><<<(unsigned)((n + 255) / 256), 256, 0, st>>>(
          (const float*)p.src, (float*)(packed + p.dst), n, (size_t)p.plain_off * p.k);
    } else {
      pack_rows<uint4, 0><<<dim3(p.rows / 32, p.k / 256), 256, 0, st>>>(
          (const uint4*)p.src, (uint4*)(packed + p.dst), p.k, p.tiles, p.mode, p.off);
    }
  }
  return launch_status();
}

// (a row of up to 2048 is one round trip for 256 threads)
static void launch_argmax(const float* logits, int n_rows, int n, int lo, int32_t* out_token, float* copy, hipStream_t st) {
  if (n > 2048) argmax_rows_wide<1024><<<n_rows, 1024, 0, st>>>(logits, n, lo, out_token, copy);
  else argmax_rows_wide<256><<<n_rows, 256, 0, st>>>(logits, n, lo, out_token, copy);
}

// The head on raw rows: logits (to `logits_ws`, [n_rows, hi - lo], if the caller wants none), then the row
// argmax.
template <typename T>
static int head_t(const sv_model_cfg& c, const T* g_final, const T* w_lm, const float* x,
                  int n_rows, int lo, int hi, int32_t* out_token, float* out_logits, float* logits_ws, hipStream_t st) {
  F32Args<T, T> a;
  memset(&a, 0, sizeof(a));
  a.X = x; a.gain = g_final; a.W = w_lm + (size_t)lo * c.hidden; a.M = n_rows; a.N = hi - lo; a.K = c.hidden; a.eps = c.rms_eps;
  a.out = out_logits ? out_logits : logits_ws;
  a.T = 1; a.nh = 1; a.d = 2;
  f32_launch<EPI_OUT>(a, st);
  launch_argmax(a.out, n_rows, a.N, lo, out_token, nullptr, st);
  return launch_status();
}

// Scratch of sv_action_head_argmax_noalloc: the logits of one call, in device memory that belongs to the
// library image (one copy per GPU, for the life of the process).  Host code never uses the array's name as an
// address: scratch_address() asks the runtime where the current device's copy lives, once per device.
// The logits do not grow with `hidden`; its limit is part of the documented call (what was refused stays so).
constexpr int kNoallocMaxRows = 64, kNoallocMaxScored = 256, kNoallocMaxHidden = 8192;
constexpr size_t kNoallocScratchBytes = (size_t)kNoallocMaxRows * kNoallocMaxScored * 4;
static __device__ __align__(256) unsigned char scratch[kNoallocScratchBytes];

static int scratch_address(unsigned char** out) {
  static void* per_device[64] = {nullptr};
  static std::mutex lock;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return SV_ERR_LAUNCH;
  std::lock_guard<std::mutex> guard(lock);
  if (!per_device[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return SV_ERR_LAUNCH;
    per_device[dev] = p;
  }
  *out = (unsigned char*)per_device[dev];
  return SV_OK;
}

// Packed head: the rows become fragments with the final gain, 1 / rms is applied to the sums, logits to
// the workspace, then the row argmax.
static int head_packed(const sv_model_cfg& c, const char* packed, const float* x, int n_rows,
                       int lo, int hi, int32_t* out_token, float* out_logits, char* ws,
                       hipStream_t st) {
  const int n = hi - lo, H = c.hidden;
  const WorkspaceLayout wl = workspace_layout(c, n_rows, n);
  const HeadLayout hl = head_layout(c, n);
  const int n_xcd = device_xcds();
  // (the product stores 16 bytes at a time)
  float* logits = out_logits && (uintptr_t)out_logits % 16 == 0 ? out_logits : (float*)(ws + wl.head_logits);
  uint4* xs = (uint4*)(ws + wl.head_xs);
  float* ssq = (float*)(ws + wl.head_ssq);
  split_gain_kernel<<<dim3(wl.n_rb * 4, H / 256), 256, 0, st>>>(x, (const float*)(packed + hl.gain), n_rows, H, wl.m_pad, wl.n_rb, xs, ssq);
  const ProductPlan p = plan_head(n_rows, n, H, n_xcd);
  ProductScratch scratch;
  scratch.xch = (f32x4_t*)(ws + wl.head_xch);
  scratch.group_cnt = (unsigned*)(ws + wl.counters);                  // the layers' counters and status word
  scratch.status = (int*)(ws + wl.counters + wl.counter_bytes) - 1;
  EpiArgs e;
  memset(&e, 0, sizeof(e));
  e.M = n_rows; e.n_rb = wl.n_rb; e.m_pad = wl.m_pad; e.K = H; e.eps = c.rms_eps;
  e.ssq = ssq; e.n_ssq = H / 256; e.out = logits;
  launch_product(p, EPI_OUT, 0, n_xcd, xs, (const uint4*)(packed + hl.w), n, H, scratch, e, st);
  launch_argmax(logits, n_rows, n, lo, out_token, out_logits == logits ? nullptr : out_logits, st);
  return launch_status();
}

}  // namespace sv

using namespace sv;

extern "C" {

const char* sv_version(void) { return "libspecvla_verify 0.1 (gfx950)"; }

const char* sv_strerror(int status) {
  switch (status) {
    case SV_OK: return "ok";
    case SV_ERR_NULL: return "a required pointer is NULL";
    case SV_ERR_SHAPE: return "unsupported size";
    case SV_ERR_TREE: return "parent array is not a valid draft tree (or too deep)";
    case SV_ERR_TOKEN: return "inconsistent action range or threshold";
    case SV_ERR_WORKSPACE: return "workspace or packed buffer too small or misaligned";
    case SV_ERR_DTYPE: return "unknown dtype";
    case SV_ERR_LAUNCH: return "HIP launch error";
    default: return "unknown status";
  }
}

int sv_tree_build_masks(const int32_t* parent, int B, int T, int d_cap, int32_t* depth,
                        uint64_t* anc_mask) {
  if (!parent || !depth || !anc_mask) return SV_ERR_NULL;
  if (B < 1 || T < 1 || T > SV_MAX_TREE_NODES || d_cap < 0 || d_cap > SV_MAX_DEPTH)
    return SV_ERR_SHAPE;
  const int W = (T + 63) / 64;
  for (int b = 0; b < B; ++b) {
    const int32_t* par = parent + (size_t)b * T;
    int32_t* dep = depth + (size_t)b * T;
    uint64_t* anc = anc_mask + (size_t)b * T * W;
    if (par[0] != -1) return SV_ERR_TREE;
    dep[0] = 0;
    for (int w = 0; w < W; ++w) anc[w] = 0;
    anc[0] = 1;
    for (int i = 1; i < T; ++i) {
      const int p = par[i];
      if (p < 0 || p >= i) return SV_ERR_TREE;
      dep[i] = dep[p] + 1;
      if (dep[i] > d_cap) return SV_ERR_TREE;
      for (int w = 0; w < W; ++w) anc[(size_t)i * W + w] = anc[(size_t)p * W + w];
      anc[(size_t)i * W + (i >> 6)] |= 1ull << (i & 63);
    }
  }
  return SV_OK;
}

int sv_packed_layer_bytes(const sv_model_cfg* cfg, size_t* bytes) {
  if (!bytes) return SV_ERR_NULL;
  const int rc = check_cfg(cfg);
  if (rc != SV_OK) return rc;
  *bytes = packed_layout(*cfg).total;
  return SV_OK;
}

int sv_pack_layer(const sv_model_cfg* cfg, const sv_layer_weights* raw, void* packed,
                  size_t packed_bytes, void* stream) {
  const int rc = check_cfg(cfg);
  if (rc != SV_OK) return rc;
  if (!raw || !packed || !raw->g1 || !raw->wq || !raw->wk || !raw->wv || !raw->wo || !raw->g2 ||
      !raw->wg || !raw->wu || !raw->wd)
    return SV_ERR_NULL;
  if (packed_bytes < packed_layout(*cfg).total || ((uintptr_t)packed % kAlign))
    return SV_ERR_WORKSPACE;
  if (cfg->dtype == SV_BF16_W8 || cfg->dtype == SV_BF16_W4) return SV_ERR_DTYPE;   // sv_pack_layer_w8 / _w4 take the scales
  if (cfg->dtype == SV_F32) return pack_layer_t<float>(*cfg, *raw, (char*)packed, (hipStream_t)stream);
  return pack_layer_t<bf16_t>(*cfg, *raw, (char*)packed, (hipStream_t)stream);
}

static int pack_layer_codes(const sv_model_cfg* cfg, const sv_layer_weights* raw,
                            const sv_layer_scales* sc, void* packed_v, size_t packed_bytes,
                            void* stream, int dtype) {
  const int rc = check_cfg(cfg);
  if (rc != SV_OK) return rc;
  if (cfg->dtype != dtype) return SV_ERR_DTYPE;
  if (!raw || !sc || !packed_v || !raw->g1 || !raw->wq || !raw->wk || !raw->wv || !raw->wo ||
      !raw->g2 || !raw->wg || !raw->wu || !raw->wd || !sc->sq || !sc->sk || !sc->sv || !sc->so ||
      !sc->sg || !sc->su || !sc->sd)
    return SV_ERR_NULL;
  const sv_model_cfg& c = *cfg;
  const PackedLayout pl = packed_layout(c);
  if (packed_bytes < pl.total || ((uintptr_t)packed_v % kAlign)) return SV_ERR_WORKSPACE;
  char* packed = (char*)packed_v;
  hipStream_t st = (hipStream_t)stream;
  const int H = c.hidden, D = c.n_heads * c.head_dim, F = c.mlp_dim;
  pack_gain<bf16_t><<<ceil_div(H, 256), 256, 0, st>>>((const bf16_t*)raw->g1, (float*)(packed + pl.g1), H);
  pack_gain<bf16_t><<<ceil_div(H, 256), 256, 0, st>>>((const bf16_t*)raw->g2, (float*)(packed + pl.g2), H);
  struct Piece {
    const void* src; const float* scale; size_t dst, sdst; int rows, k, mode, off, tiles;
  };
  const Piece pieces[] = {
      {raw->wq, sc->sq, pl.wqkv, pl.sqkv, D, H, PACK_PAIR16_HEAD, 0, 3 * D / 32},
      {raw->wk, sc->sk, pl.wqkv, pl.sqkv, D, H, PACK_PAIR16_HEAD, D, 3 * D / 32},
      {raw->wv, sc->sv, pl.wqkv, pl.sqkv, D, H, PACK_PAIR16_HEAD, 2 * D, 3 * D / 32},
      {raw->wo, sc->so, pl.wo, pl.so, H, D, PACK_PLAIN, 0, H / 32},
      {raw->wg, sc->sg, pl.wgu, pl.sgu, F, H, PACK_PAIR16_GU, 0, F / 16},
      {raw->wu, sc->su, pl.wgu, pl.sgu, F, H, PACK_PAIR16_GU, 16, F / 16},
      {raw->wd, sc->sd, pl.wd, pl.sd, H, F, PACK_PLAIN, 0, H / 32}};
  for (const Piece& p : pieces) {
    const dim3 grid(p.rows / 32, p.k / 256);
    if (dtype == SV_BF16_W4)
      pack_rows<uint32_t, 2><<<grid, 256, 0, st>>>((const uint32_t*)p.src, (uint32_t*)(packed + p.dst), p.k, p.tiles, p.mode, p.off);
    else
      pack_rows<uint2, 1><<<grid, 256, 0, st>>>((const uint2*)p.src, (uint2*)(packed + p.dst), p.k, p.tiles, p.mode, p.off);
    pack_row_scales<<<ceil_div(p.rows, 256), 256, 0, st>>>(p.scale, (float*)(packed + p.sdst), p.rows, p.mode, p.off,
                                                           dtype == SV_BF16_W4 ? kInt4Unit : 1.0f);
  }
  return launch_status();
}

int sv_pack_layer_w8(const sv_model_cfg* cfg, const sv_layer_weights* raw,
                     const sv_layer_scales* sc, void* packed_v, size_t packed_bytes,
                     void* stream) {
  return pack_layer_codes(cfg, raw, sc, packed_v, packed_bytes, stream, SV_BF16_W8);
}

int sv_pack_layer_w4(const sv_model_cfg* cfg, const sv_layer_weights* raw,
                     const sv_layer_scales* sc, void* packed_v, size_t packed_bytes,
                     void* stream) {
  return pack_layer_codes(cfg, raw, sc, packed_v, packed_bytes, stream, SV_BF16_W4);
}

static int check_workspace_sizes(const sv_model_cfg* cfg, int B, int T, int n_scored) {
  const int rc = check_cfg(cfg);
  if (rc != SV_OK) return rc;
  if (B < 1 || T < 1 || T > SV_MAX_TREE_NODES || n_scored < 0 || n_scored > cfg->vocab ||
      (long long)B * T > (1 << 15))
    return SV_ERR_SHAPE;
  return SV_OK;
}

// What a call needs depends on how its products are split, and some row counts need more than larger ones
// (7B: 320 rows 144 MB, 384 rows 135).  The bytes handed out are therefore the most that any row count up to
// B * T needs; a call itself asks for its own only.
int sv_workspace_bytes(const sv_model_cfg* cfg, int B, int T, int n_scored, size_t* bytes) {
  if (!bytes) return SV_ERR_NULL;
  const int rc = check_workspace_sizes(cfg, B, T, n_scored);
  if (rc != SV_OK) return rc;
  size_t most = workspace_layout(*cfg, B * T, n_scored).total;
  for (int rows = 32; cfg->dtype != SV_F32 && rows < B * T; rows += 32) {      // (what a plan takes follows from the 32-row blocks)
    const size_t n = workspace_layout(*cfg, rows, n_scored).total;
    most = n > most ? n : most;
  }
  *bytes = most;
  return SV_OK;
}

int sv_workspace_init(const sv_model_cfg* cfg, int B, int T, int n_scored, void* workspace,
                      size_t ws_bytes, void* stream) {
  const int rc = check_workspace_sizes(cfg, B, T, n_scored);
  if (rc != SV_OK) return rc;
  if (!workspace) return SV_ERR_NULL;
  const WorkspaceLayout wl = workspace_layout(*cfg, B * T, n_scored);
  if (((uintptr_t)workspace % kAlign) || ws_bytes < wl.total) return SV_ERR_WORKSPACE;
  const size_t n = wl.counter_bytes / sizeof(int);
  if (n > 0)
    zero_ints<<<(unsigned)((n + 255) / 256), 256, 0, (hipStream_t)stream>>>(
        (int*)((char*)workspace + wl.counters), n);
  return launch_status();
}

int sv_workspace_region(const sv_model_cfg* cfg, int B, int T, int n_scored, int which,
                        size_t* offset, size_t* bytes) {
  if (!offset || !bytes) return SV_ERR_NULL;
  const int rc = check_workspace_sizes(cfg, B, T, n_scored);
  if (rc != SV_OK) return rc;
  const WorkspaceLayout wl = workspace_layout(*cfg, B * T, n_scored);
  const size_t D = (size_t)cfg->n_heads * cfg->head_dim, M = (size_t)B * T;
  if (which == SV_WS_ATTN_OUT) {
    *offset = wl.attn;
    *bytes = M * D * 4;
  } else if (which == SV_WS_Q) {
    *offset = wl.q;
    *bytes = M * D * 4;
  } else if (which == SV_WS_STATUS) {
    *offset = wl.counters + (wl.counter_bytes ? wl.counter_bytes - 4 : 0);
    *bytes = wl.counter_bytes ? 4 : 0;
  } else {
    return SV_ERR_SHAPE;
  }
  return SV_OK;
}

static int verify_layer_dispatch(const sv_model_cfg& c, const LayerCall& lc, const void* packed, float* x,
                                 const sv_kv_view& kv, const sv_tree& tree, int B, void* workspace, void* stream,
                                 hipEvent_t* ev, bool first, const void* next_packed) {
  if (c.dtype == SV_F32)
    return verify_layer_f32(c, lc.wl, (const char*)packed, x, kv, tree, B, (char*)workspace, (hipStream_t)stream, ev);
  return verify_layer_bf16(c, lc, (const char*)packed, x, kv, tree, B, (char*)workspace, (hipStream_t)stream, ev, first,
                           (const char*)next_packed);
}

static int verify_layer_checked(const sv_model_cfg* cfg, const void* packed, float* x,
                                const sv_kv_view* kv, const sv_tree* tree, int B,
                                void* workspace, size_t ws_bytes, void* stream,
                                hipEvent_t* ev) {
  const int rc = check_cfg(cfg);
  if (rc != SV_OK) return rc;
  if (!packed || !x || !kv || !tree || !workspace || !kv->k || !kv->v || !kv->prefix_len ||
      !tree->parent || !tree->depth || !tree->anc_mask)
    return SV_ERR_NULL;
  const int T = tree->n_nodes;
  if (B < 1 || T < 1 || T > SV_MAX_TREE_NODES || tree->n_words != (T + 63) / 64 ||
      (long long)B * T > (1 << 15))
    return SV_ERR_SHAPE;
  if (kv->prefix_len_max < 0 || (long long)kv->capacity < (long long)kv->prefix_len_max + T)
    return SV_ERR_SHAPE;
  if ((long long)B * cfg->n_heads * kv->capacity >= (1ll << 31)) return SV_ERR_SHAPE;   // cache rows are indexed in 32 bits
  if (((uintptr_t)workspace % kAlign) || ((uintptr_t)packed % kAlign)) return SV_ERR_WORKSPACE;
  const LayerCall lc = layer_call(*cfg, B * T);
  if (ws_bytes < lc.wl.total) return SV_ERR_WORKSPACE;
  return verify_layer_dispatch(*cfg, lc, packed, x, *kv, *tree, B, workspace, stream, ev, true, nullptr);
}

int sv_verify_layer(const sv_model_cfg* cfg, const void* packed, float* x, const sv_kv_view* kv,
                    const sv_tree* tree, int B, void* workspace, size_t ws_bytes, void* stream) {
  return verify_layer_checked(cfg, packed, x, kv, tree, B, workspace, ws_bytes, stream, nullptr);
}

int sv_verify_layer_timed(const sv_model_cfg* cfg, const void* packed, float* x,
                          const sv_kv_view* kv, const sv_tree* tree, int B, void* workspace,
                          size_t ws_bytes, void* stream, void* const* events) {
  if (!events) return SV_ERR_NULL;
  hipEvent_t ev[SV_N_TIMING_EVENTS];
  for (int i = 0; i < SV_N_TIMING_EVENTS; ++i) {
    if (!events[i]) return SV_ERR_NULL;
    ev[i] = (hipEvent_t)events[i];
  }
  return verify_layer_checked(cfg, packed, x, kv, tree, B, workspace, ws_bytes, stream, ev);
}

static int verify_stack_args(const sv_model_cfg* cfg, int n_layers, const void* const* packed,
                             float* x, const sv_kv_view* kv, const sv_tree* tree, int B,
                             void* workspace) {
  const int rc = check_cfg(cfg);
  if (rc != SV_OK) return rc;
  if (!packed || !x || !kv || !tree || !workspace || !tree->parent || !tree->depth || !tree->anc_mask)
    return SV_ERR_NULL;
  if (n_layers < 1) return SV_ERR_SHAPE;
  const int T = tree->n_nodes;
  if (B < 1 || T < 1 || T > SV_MAX_TREE_NODES || tree->n_words != (T + 63) / 64 ||
      (long long)B * T > (1 << 15))
    return SV_ERR_SHAPE;
  for (int l = 0; l < n_layers; ++l) {
    if (!packed[l] || !kv[l].k || !kv[l].v || !kv[l].prefix_len) return SV_ERR_NULL;
    if ((uintptr_t)packed[l] % kAlign) return SV_ERR_WORKSPACE;
    if (kv[l].prefix_len_max < 0 || (long long)kv[l].capacity < (long long)kv[l].prefix_len_max + T)
      return SV_ERR_SHAPE;
    if ((long long)B * cfg->n_heads * kv[l].capacity >= (1ll << 31)) return SV_ERR_SHAPE;
  }
  return (uintptr_t)workspace % kAlign ? SV_ERR_WORKSPACE : SV_OK;
}

int sv_verify_stack(const sv_model_cfg* cfg, int n_layers, const void* const* packed, float* x,
                    const sv_kv_view* kv, const sv_tree* tree, int B, void* workspace,
                    size_t ws_bytes, void* stream) {
  const int rc = verify_stack_args(cfg, n_layers, packed, x, kv, tree, B, workspace);
  if (rc != SV_OK) return rc;
  const LayerCall lc = layer_call(*cfg, B * tree->n_nodes);
  if (ws_bytes < lc.wl.total) return SV_ERR_WORKSPACE;
  for (int l = 0; l < n_layers; ++l) {
    const int r2 = verify_layer_dispatch(*cfg, lc, packed[l], x, kv[l], *tree, B, workspace, stream, nullptr, l == 0,
                                         l + 1 < n_layers ? packed[l + 1] : nullptr);
    if (r2 != SV_OK) return r2;
  }
  return SV_OK;
}

int sv_action_head_argmax(const sv_model_cfg* cfg, const void* g_final, const void* w_lm,
                          const float* x, int n_rows, int vocab_lo, int vocab_hi,
                          int32_t* out_token, float* out_logits, void* workspace,
                          size_t ws_bytes, void* stream) {
  const int rc = check_cfg(cfg);
  if (rc != SV_OK) return rc;
  if (!g_final || !w_lm || !x || !out_token || !workspace) return SV_ERR_NULL;
  if (n_rows < 1 || n_rows > (1 << 15) || vocab_lo < 0 || vocab_lo >= vocab_hi ||
      vocab_hi > cfg->vocab)
    return SV_ERR_SHAPE;
  if (((uintptr_t)workspace % kAlign) ||
      ws_bytes < workspace_layout(*cfg, n_rows, vocab_hi - vocab_lo).total)
    return SV_ERR_WORKSPACE;
  const WorkspaceLayout wl = workspace_layout(*cfg, n_rows, vocab_hi - vocab_lo);
  float* logits = (float*)((char*)workspace + wl.head_logits);
  if (cfg->dtype == SV_F32)
    return head_t<float>(*cfg, (const float*)g_final, (const float*)w_lm, x, n_rows, vocab_lo,
                         vocab_hi, out_token, out_logits, logits, (hipStream_t)stream);
  return head_t<bf16_t>(*cfg, (const bf16_t*)g_final, (const bf16_t*)w_lm, x, n_rows, vocab_lo,
                        vocab_hi, out_token, out_logits, logits, (hipStream_t)stream);
}

int sv_action_head_argmax_noalloc(const sv_model_cfg* cfg, const void* g_final, const void* w_lm,
                                  const float* x, int n_rows, int vocab_lo, int vocab_hi,
                                  int32_t* out_token, float* out_logits, void* stream) {
  const int rc = check_cfg(cfg);
  if (rc != SV_OK) return rc;
  if (!g_final || !w_lm || !x || !out_token) return SV_ERR_NULL;
  if (n_rows < 1 || vocab_lo < 0 || vocab_lo >= vocab_hi || vocab_hi > cfg->vocab) return SV_ERR_SHAPE;
  if (n_rows > kNoallocMaxRows || vocab_hi - vocab_lo > kNoallocMaxScored || cfg->hidden > kNoallocMaxHidden)
    return SV_ERR_WORKSPACE;                  // beyond what the built-in scratch holds
  unsigned char* base = nullptr;
  const int rs = scratch_address(&base);
  if (rs != SV_OK) return rs;
  float* logits = (float*)base;
  if (cfg->dtype == SV_F32)
    return head_t<float>(*cfg, (const float*)g_final, (const float*)w_lm, x, n_rows, vocab_lo,
                         vocab_hi, out_token, out_logits, logits, (hipStream_t)stream);
  return head_t<bf16_t>(*cfg, (const bf16_t*)g_final, (const bf16_t*)w_lm, x, n_rows, vocab_lo,
                        vocab_hi, out_token, out_logits, logits, (hipStream_t)stream);
}

int sv_product_plan(const sv_model_cfg* cfg, int n_rows, int which, int n_scored, int n_xcd, int32_t* plan) {
  if (!plan) return SV_ERR_NULL;
  const int rc = check_cfg(cfg);
  if (rc != SV_OK) return rc;
  if (cfg->dtype == SV_F32) return SV_ERR_DTYPE;
  if (n_rows < 1 || n_rows > (1 << 15) || which < SV_PLAN_QKV || which > SV_PLAN_HEAD || n_xcd < 1 || n_xcd > kXcds)
    return SV_ERR_SHAPE;
  if (which == SV_PLAN_HEAD && (n_scored < 1 || n_scored > cfg->vocab || n_scored % kFragRows)) return SV_ERR_SHAPE;
  ProductPlan p;
  if (which == SV_PLAN_HEAD) {
    p = plan_head(n_rows, n_scored, cfg->hidden, n_xcd);
  } else {
    const LayerPlan l = plan_layer(*cfg, n_rows, n_xcd);
    p = which == SV_PLAN_QKV ? l.qkv : (which == SV_PLAN_OUT ? l.o : (which == SV_PLAN_GATE_UP ? l.gu : l.down));
  }
  const int32_t v[6] = {p.kernel, p.rb, p.nt, 1 << p.lgS, p.gpx, p.m_tiles};
  memcpy(plan, v, sizeof(v));
  return SV_OK;
}

int sv_packed_head_bytes(const sv_model_cfg* cfg, int vocab_lo, int vocab_hi, size_t* bytes) {
  if (!bytes) return SV_ERR_NULL;
  const int rc = check_packed_head(cfg, vocab_lo, vocab_hi);
  if (rc != SV_OK) return rc;
  *bytes = head_layout(*cfg, vocab_hi - vocab_lo).total;
  return SV_OK;
}

int sv_pack_head(const sv_model_cfg* cfg, const void* g_final, const void* w_lm, int vocab_lo,
                 int vocab_hi, void* packed_v, size_t packed_bytes, void* stream) {
  const int rc = check_packed_head(cfg, vocab_lo, vocab_hi);
  if (rc != SV_OK) return rc;
  if (!g_final || !w_lm || !packed_v) return SV_ERR_NULL;
  const int n = vocab_hi - vocab_lo, H = cfg->hidden;
  const HeadLayout hl = head_layout(*cfg, n);
  if (packed_bytes < hl.total || ((uintptr_t)packed_v % kAlign)) return SV_ERR_WORKSPACE;
  char* packed = (char*)packed_v;
  hipStream_t st = (hipStream_t)stream;
  pack_gain<bf16_t><<<ceil_div(H, 256), 256, 0, st>>>((const bf16_t*)g_final, (float*)(packed + hl.gain), H);
  pack_rows<uint4, 0><<<dim3(n / 32, H / 256), 256, 0, st>>>((const uint4*)((const bf16_t*)w_lm + (size_t)vocab_lo * H),
                                                            (uint4*)(packed + hl.w), H, n / 32, PACK_PLAIN, 0);
  return launch_status();
}

int sv_action_head_argmax_packed(const sv_model_cfg* cfg, const void* packed_head, const float* x,
                                 int n_rows, int vocab_lo, int vocab_hi, int32_t* out_token,
                                 float* out_logits, void* workspace, size_t ws_bytes,
                                 void* stream) {
  const int rc = check_packed_head(cfg, vocab_lo, vocab_hi);
  if (rc != SV_OK) return rc;
  if (!packed_head || !x || !out_token || !workspace) return SV_ERR_NULL;
  if (n_rows < 1 || n_rows > (1 << 15)) return SV_ERR_SHAPE;
  if (((uintptr_t)workspace % kAlign) || ((uintptr_t)packed_head % kAlign) ||
      ws_bytes < workspace_layout(*cfg, n_rows, vocab_hi - vocab_lo).total)
    return SV_ERR_WORKSPACE;
  return head_packed(*cfg, (const char*)packed_head, x, n_rows, vocab_lo, vocab_hi, out_token,
                     out_logits, (char*)workspace, (hipStream_t)stream);
}

int sv_stream_read(const void* ptr, size_t bytes, void* sink, void* stream) {
  if (!ptr || !sink) return SV_ERR_NULL;
  if (bytes < 16 || (bytes % 16) || ((uintptr_t)ptr % 16) || ((uintptr_t)sink % 16)) return SV_ERR_SHAPE;
  const size_t n_vec = bytes / 16;
  size_t blocks = (n_vec + 2047) / 2048;               // 8 KiB per wave and round
  if (blocks > 2048) blocks = 2048;                    // 8 workgroups per CU walk the buffer
  stream_read_kernel<<<(unsigned)blocks, 256, 0, (hipStream_t)stream>>>((const u32x4_t*)ptr, n_vec,
                                                                       (u32x4_t*)sink);
  return launch_status();
}

int sv_relaxed_accept(const sv_tree* tree, const int32_t* draft_token,
                      const int32_t* target_token, int action_lo, int n_bins, int r, int B,
                      int d_cap, uint8_t* accept_mask, int32_t* accepted_len,
                      int32_t* best_node, int32_t* path, int32_t* out_tokens, void* stream) {
  if (!tree || !tree->parent || !tree->depth || !tree->anc_mask || !draft_token ||
      !target_token || !accept_mask || !accepted_len || !best_node || !path || !out_tokens)
    return SV_ERR_NULL;
  const int T = tree->n_nodes;
  if (B < 1 || B > (1 << 15) || T < 1 || T > SV_MAX_TREE_NODES ||
      tree->n_words != (T + 63) / 64 || d_cap < 0 || d_cap > SV_MAX_DEPTH)
    return SV_ERR_SHAPE;
  if (n_bins < 1 || r < 0 || action_lo < 0) return SV_ERR_TOKEN;
  relaxed_accept_kernel<<<B, 128, 0, (hipStream_t)stream>>>(
      tree->parent, tree->depth, tree->anc_mask, T, tree->n_words, draft_token, target_token,
      action_lo, n_bins, r, d_cap, accept_mask, accepted_len, best_node, path, out_tokens);
  return launch_status();
}

int sv_tree_build_device(const int32_t* cand_parent, const float* cand_logp,
                         const int32_t* cand_token, int n_cand, const int32_t* root_token, int B,
                         int T, int d_cap, int32_t* parent, int32_t* depth, uint64_t* anc_mask,
                         int32_t* draft_token, int32_t* status, void* stream) {
  if (!cand_parent || !cand_logp || !cand_token || !root_token || !parent || !depth || !anc_mask ||
      !draft_token || !status)
    return SV_ERR_NULL;
  if (B < 1 || B > (1 << 15) || T < 1 || T > SV_MAX_TREE_NODES || n_cand < T - 1 ||
      n_cand > kMaxCandidates || d_cap < 0 || d_cap > SV_MAX_DEPTH)
    return SV_ERR_SHAPE;
  tree_build_kernel<<<B, 1024, 0, (hipStream_t)stream>>>(cand_parent, cand_logp, cand_token, n_cand,
                                                        root_token, T, (T + 63) / 64, d_cap, parent,
                                                        depth, anc_mask, draft_token, status);
  return launch_status();
}

int sv_commit_path(const sv_model_cfg* cfg, const sv_kv_view* kv, int T, const int32_t* path,
                   const int32_t* accepted_len, int B, int d_cap, void* stream) {
  const int rc = check_cfg(cfg);
  if (rc != SV_OK) return rc;
  if (!kv || !kv->k || !kv->v || !kv->prefix_len || !path || !accepted_len) return SV_ERR_NULL;
  if (B < 1 || B > (1 << 15) || T < 1 || T > SV_MAX_TREE_NODES || d_cap < 0 || d_cap > SV_MAX_DEPTH)
    return SV_ERR_SHAPE;
  if (kv->prefix_len_max < 0 || (long long)kv->capacity < (long long)kv->prefix_len_max + T)
    return SV_ERR_SHAPE;
  const dim3 grid(B, cfg->n_heads);
  hipStream_t st = (hipStream_t)stream;
  auto commit = [&](auto* k, auto* v, int units) {
    commit_path_kernel<<<grid, 256, 0, st>>>(k, v, kv->prefix_len, kv->prefix_len_max, kv->capacity, T, cfg->n_heads, units,
                                             path, accepted_len, d_cap);
  };
  const int row_bytes = cfg->head_dim * (cfg->dtype == SV_F32 ? 4 : 2);
  if (row_bytes % 16 == 0 && (uintptr_t)kv->k % 16 == 0 && (uintptr_t)kv->v % 16 == 0)
    commit((u32x4_t*)kv->k, (u32x4_t*)kv->v, row_bytes / 16);
  else if (cfg->dtype == SV_F32) commit((float*)kv->k, (float*)kv->v, cfg->head_dim);
  else commit((uint16_t*)kv->k, (uint16_t*)kv->v, cfg->head_dim);
  return launch_status();
}

int sv_advance_prefix(int32_t* prefix_len, const int32_t* accepted_len, int B, int d_cap,
                      void* stream) {
  if (!prefix_len || !accepted_len) return SV_ERR_NULL;
  if (B < 1 || B > (1 << 15) || d_cap < 0 || d_cap > SV_MAX_DEPTH) return SV_ERR_SHAPE;
  advance_prefix_kernel<<<(B + 63) / 64, 64, 0, (hipStream_t)stream>>>(prefix_len, accepted_len, B,
                                                                       d_cap);
  return launch_status();
}

}  // extern "C"
