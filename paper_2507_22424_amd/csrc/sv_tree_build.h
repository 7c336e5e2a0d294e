// Draft tree from the recorded top-K predictions of the draft model, built on the device.
//
// Sec. 4.1: the top-K predictions of the drafter are recorded and form a tree with several
// paths (the dynamic draft tree strategy the paper adopts; Sec. 5.1: top 8, at most 50 nodes).
// This is the final selection of that strategy: every candidate's score is the joint
// log-probability of its path (float32, accumulated from the root down, one addition per
// edge), the n_nodes - 1 best candidates are kept (lower candidate index wins ties, so a
// parent is never dropped before its child), and the kept nodes are numbered breadth first
// behind the root.  Output = exactly the arrays the verification calls take (parent, depth,
// ancestor-or-self bitmask, draft tokens), so a step needs no host round trip for its tree.
//
// One workgroup of 1024 threads per episode, a thread per candidate (at most 1024, kept in LDS).  Latency
// bound: the paper's setting (264 candidates, 50 nodes, 16 episodes) took 37 us with 256 threads that walk
// and sum every path on their own and count over all candidates twice.
#ifndef SV_TREE_BUILD_H
#define SV_TREE_BUILD_H

#include "sv_internal.h"

namespace sv {

constexpr int kMaxCandidates = 1024;

// status[b]: 0 ok; bit 0 = a candidate's parent index is not an earlier candidate;
// bit 1 = a kept candidate is deeper than d_cap; bit 2 = a kept candidate's parent was not kept
// (log-probabilities above zero).  A flagged episode gets a root-only chain
// (every node a child of the root) so that later calls stay in bounds.
__global__ __launch_bounds__(1024) void tree_build_kernel(
    const int32_t* __restrict__ cand_parent, const float* __restrict__ cand_logp,
    const int32_t* __restrict__ cand_token, int n_cand, const int32_t* __restrict__ root_token,
    int T, int n_words, int d_cap, int32_t* __restrict__ parent, int32_t* __restrict__ depth,
    uint64_t* __restrict__ anc_mask, int32_t* __restrict__ draft_token, int32_t* __restrict__ status) {
  __shared__ float s_score[kMaxCandidates];
  __shared__ int s_par[kMaxCandidates];
  __shared__ int s_rank[kMaxCandidates];
  __shared__ int s_key[SV_MAX_TREE_NODES];     // kept candidates in order of rank: depth * 1024 + index
  __shared__ short s_node[kMaxCandidates];     // node index of a kept candidate, -1 otherwise
  __shared__ int s_bad, s_levels;
  const int b = blockIdx.x, tid = threadIdx.x;
  const int n_keep = T - 1;
  const bool own = tid < n_cand;               // this thread's candidate is tid
  int par = -1, dep = 0, tok = 0;
  float lp = 0.f;
  if (tid == 0) s_bad = s_levels = 0;
  __syncthreads();
  if (own) {
    par = cand_parent[(size_t)b * n_cand + tid];
    lp = cand_logp[(size_t)b * n_cand + tid];
    tok = cand_token[(size_t)b * n_cand + tid];
    s_par[tid] = par;
    s_rank[tid] = 0;
    s_node[tid] = -1;
    if (par < -1 || par >= tid) atomicOr(&s_bad, 1);
  }
  __syncthreads();
  bool kept = false;
  if (s_bad == 0) {
    bool deep = false;                         // deeper than any tree this library takes
    if (own) {
      int node = tid;
      while (node >= 0 && dep <= SV_MAX_DEPTH) {
        ++dep;
        node = s_par[node];
      }
      deep = node >= 0;
      atomicMax(&s_levels, dep);
    }
    __syncthreads();
    // scores from the root down, level after level: one addition per edge, in the order of the sequential
    // definition
    const int levels = s_levels;
    for (int l = 1; l <= levels; ++l) {
      if (own && !deep && dep == l) s_score[tid] = (par < 0 ? 0.f : s_score[par]) + lp;
      __syncthreads();
    }
    if (own) {
      const float sc = deep ? -__builtin_inff() : s_score[tid];
      s_score[tid] = sc == sc ? sc : -__builtin_inff();     // NaN sorts last: the order stays total
    }
    __syncthreads();
    // rank among all candidates: higher score first, lower index first on ties.  `parts` threads count for a
    // candidate, each over its share of the others.
    const int parts = n_cand > 0 ? 1024 / n_cand : 0, part = parts ? tid / n_cand : 0, c = tid - part * n_cand;
    if (part < parts) {
      const int j0 = n_cand * part / parts, j1 = n_cand * (part + 1) / parts;
      const float sc = s_score[c];
      int rank = 0;
#pragma unroll 8
      for (int j = j0; j < j1; ++j) {
        const float sj = s_score[j];
        rank += (sj > sc || (sj == sc && j < c)) ? 1 : 0;
      }
      atomicAdd(&s_rank[c], rank);
    }
    __syncthreads();
    if (own) {
      const int rank = s_rank[tid];
      kept = rank < n_keep;
      if (kept) {
        s_key[rank] = dep * kMaxCandidates + tid;
        s_node[tid] = 0;
        if (dep > d_cap) atomicOr(&s_bad, 2);
      }
    }
    __syncthreads();
    // log-probabilities above zero can rank a child before its parent: not a tree
    if (kept && par >= 0 && s_node[par] < 0) atomicOr(&s_bad, 4);
    __syncthreads();
  }
  int32_t* par_o = parent + (size_t)b * T;
  int32_t* dep_o = depth + (size_t)b * T;
  int32_t* tok_o = draft_token + (size_t)b * T;
  uint64_t* anc_o = anc_mask + (size_t)b * T * n_words;
  if (s_bad != 0) {
    for (int i = tid; i < T; i += 1024) {
      par_o[i] = i == 0 ? -1 : 0;
      dep_o[i] = i == 0 ? 0 : 1;
      tok_o[i] = root_token[b];
      for (int w = 0; w < n_words; ++w) anc_o[(size_t)i * n_words + w] = 0;
      anc_o[(size_t)i * n_words + (i >> 6)] |= 1ull << (i & 63);
      anc_o[(size_t)i * n_words] |= 1ull;
    }
    if (tid == 0) status[b] = s_bad;
    return;
  }
  // breadth-first number of a kept candidate: 1 + kept candidates before it in (depth, index)
  int node_index = 0;
  if (kept) {
    const int key = dep * kMaxCandidates + tid;
    node_index = 1;
#pragma unroll 8
    for (int j = 0; j < n_keep; ++j) node_index += s_key[j] < key ? 1 : 0;
    s_node[tid] = (short)node_index;
  }
  __syncthreads();
  if (tid == 0) {
    par_o[0] = -1;
    dep_o[0] = 0;
    tok_o[0] = root_token[b];
    for (int w = 0; w < n_words; ++w) anc_o[w] = 0;
    anc_o[0] = 1ull;
    status[b] = 0;
  }
  if (kept) {
    par_o[node_index] = par < 0 ? 0 : s_node[par];
    dep_o[node_index] = dep;
    tok_o[node_index] = tok;
    uint64_t m[2] = {1ull, 0ull};                      // the root
    for (int node = tid; node >= 0; node = s_par[node]) {
      const int ni = s_node[node];
      if (ni < 64) m[0] |= 1ull << ni;
      else m[1] |= 1ull << (ni - 64);
    }
    anc_o[(size_t)node_index * n_words] = m[0];
    if (n_words > 1) anc_o[(size_t)node_index * n_words + 1] = m[1];
  }
}

}  // namespace sv
#endif
