// Draft-tree bookkeeping on the device: per-row log-softmax + top-K over the draft vocabulary, the
// per-level frontier choice by cumulative log-probability, and the final global rerank.  Ordering rule
// everywhere: larger score first, ties -> smaller id.  Everything here is latency-bound integer/compare
// work on a few hundred candidates, done with wavefront shuffles and LDS reductions; no host round trip.
#include <limits.h>

#include <algorithm>

#include "common.hpp"
#include "draft_row.hpp"
#include "kernels.hpp"

namespace {

__device__ __forceinline__ bool better(float va, int ia, float vb, int ib) { return va > vb || (va == vb && ia < ib); }

// Row top-K in two levels, no workgroup barrier anywhere.
// Level 1: one wavefront per 512 consecutive logits (8 per lane, held in registers) finds its own top K by K
// rounds of a wavefront max, and the (max, sum of exp) of its span.  Where the max sits is read from the lanes that hold it
// (compares and scalar bit operations) instead of being carried through the reduction.
// Candidates are stored [row][rank][span], so that level 2 reads them with consecutive lanes.
constexpr int TOPK_SPAN = 512;
__global__ __launch_bounds__(256) void topk_spans_kernel(const float* __restrict__ z, int ld, int row0, int V, int K,
                                                        int n_spans, float* __restrict__ cand_val,
                                                        int32_t* __restrict__ cand_idx, float* __restrict__ span_stat) {
  const int lane = threadIdx.x & 63, span = blockIdx.x * 4 + (threadIdx.x >> 6), row = blockIdx.y;
  if (span >= n_spans) return;
  const float* zr = z + (size_t)(row0 + row) * ld;
  const int base = span * TOPK_SPAN;
  float v[8];
  float mx = -INFINITY;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int c = base + j * 64 + lane;
    v[j] = c < V ? zr[c] : -INFINITY;
    mx = fmaxf(mx, v[j]);
  }
  mx = wave_max(mx);
  float sum = 0.f;
#pragma unroll
  for (int j = 0; j < 8; ++j) sum += expf(v[j] - mx);  // exp(-inf) = 0 for the padding
  sum = wave_sum_butterfly(sum);
  const size_t o = (size_t)row * n_spans + span;
  if (lane == 0) { span_stat[2 * o] = mx; span_stat[2 * o + 1] = sum; }
  for (int r = 0; r < K; ++r) {
    if (r > 0) {
      mx = v[0];
#pragma unroll
      for (int j = 1; j < 8; ++j) mx = fmaxf(mx, v[j]);
      mx = wave_max(mx);
    }
    // first entry equal to the max: smallest j, then smallest lane
    int at = INT_MAX;
#pragma unroll
    for (int j = 7; j >= 0; --j) {
      const unsigned long long eq = __ballot(v[j] == mx);
      if (eq) at = j * 64 + __ffsll((long long)eq) - 1;
    }
    if (!(mx > -INFINITY)) at = INT_MAX;               // fewer than K entries above -inf (a NaN is none): no candidate
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (at == j * 64 + lane) v[j] = -INFINITY;
    if (lane == 0) {
      const size_t c = ((size_t)row * K + r) * n_spans + span;
      cand_val[c] = mx;
      cand_idx[c] = at == INT_MAX ? INT_MAX : base + at;
    }
  }
}

// What topk_spans_kernel leaves for the rows of a launch; or, above 64 spans, what topk_merge_kernel makes of it.
struct Candidates {
  const float* val;        // [row][rank][span]
  const int32_t* idx;
  const float* stat;       // [row][span] (max, sum of exp)
  int n_spans;
  const float* top_val;    // [row][K], merged (KM = 0)
  const int32_t* top_idx;
};
constexpr int TOPK_MAX_SPANS = 1024, TOPK_MAX_K = 16;

// Level 2, in the kernel that uses the result: one wavefront per row.  KM > 0 (K <= KM): up to 64 spans (32768 entries), lane = span,
// its K candidates in registers, all requested in one memory round trip.  Round r takes the best head (ties: the lowest span, which holds the
// smaller ids) and moves the winner's list up by one.  As a launch of its own 10 rows of 32000 took 4.7 us, against 9.9 us by ranking the survivors of
// a bound.  KM = 0: the merged top K is read.  Lane r < K ends with rank r: its log-probability, draft id and target id.
template <int KM>
__device__ __forceinline__ void merge_row(const Candidates& c, const int32_t* __restrict__ d2t, int row, int K, int lane, float& out_v,
                                          int& out_i, int& out_t) {
  if constexpr (KM == 0) {
    out_v = c.top_val[row * K + min(lane, K - 1)];
    out_i = c.top_idx[row * K + min(lane, K - 1)];
  } else {
    const int n_spans = c.n_spans, span = min(lane, n_spans - 1);
    const bool real = lane < n_spans;
    const float* val = c.val + (size_t)row * K * n_spans;      // the same for the whole wavefront
    const int32_t* idx = c.idx + (size_t)row * K * n_spans;
    float v[KM];
    int id[KM];
#pragma unroll
    for (int r = 0; r < KM; ++r) {
      v[r] = val[min(r, K - 1) * n_spans + span];
      id[r] = idx[min(r, K - 1) * n_spans + span];
    }
    const float2 st = *(const float2*)(c.stat + (size_t)row * n_spans * 2 + span * 2);
#pragma unroll
    for (int r = 0; r < KM; ++r)
      if (!real || r >= K) { v[r] = -INFINITY; id[r] = INT_MAX; }
    const float mx = wave_max(real ? st.x : -INFINITY);
    const float lse = logf(wave_sum_butterfly(real ? st.y * expf(st.x - mx) : 0.f));
    out_v = 0.f;
    out_i = 0;
    for (int r = 0; r < K; ++r) {
      const float best = wave_max(v[0]);
      const unsigned long long eq = __ballot(v[0] == best);
      const int win = eq ? __ffsll((long long)eq) - 1 : 0;
      const int win_id = __builtin_amdgcn_readlane(id[0], win);
      if (lane == r) { out_v = best - mx - lse; out_i = win_id == INT_MAX ? 0 : win_id; }
      if (lane == win) {
#pragma unroll
        for (int j = 0; j + 1 < KM; ++j) { v[j] = v[j + 1]; id[j] = id[j + 1]; }
        v[KM - 1] = -INFINITY;
        id[KM - 1] = INT_MAX;
      }
    }
  }
  out_t = d2t[out_i];
}

// Level 2 for more spans, a launch of its own: one wavefront per row merges the spans' candidates and statistics, without sequential selection rounds.
// In the order (value desc, index asc) the K-th best of the spans' BEST candidates bounds the answer from below:
// at least K candidates are not worse than it, so only candidates not worse than it can be among the top K, and
// those come from exactly K spans (at most K * K survivors).  The survivors are ranked by counting, and rank r < K
// is output r.  Entries without a candidate (-inf or NaN) never survive; when fewer than K spans have one there is no
// bound, and fewer than K * K survivors.  Ranks that are left over get index 0.
__global__ __launch_bounds__(64) void topk_merge_kernel(const float* __restrict__ cand_val, const int32_t* __restrict__ cand_idx,
                                                       const float* __restrict__ span_stat, int n_spans, int K,
                                                       float* __restrict__ top_val, int32_t* __restrict__ top_idx) {
  __shared__ float head_v[TOPK_MAX_SPANS];
  __shared__ int head_i[TOPK_MAX_SPANS];
  __shared__ float surv_v[TOPK_MAX_K * TOPK_MAX_K];
  __shared__ int surv_i[TOPK_MAX_K * TOPK_MAX_K];
  __shared__ float bound_v;
  __shared__ int bound_i, n_surv;
  const int lane = threadIdx.x, row = blockIdx.x;
  const float* st = span_stat + (size_t)row * n_spans * 2;
  float mx = -INFINITY;
  for (int i = lane; i < n_spans; i += 64) mx = fmaxf(mx, st[2 * i]);
  mx = wave_max(mx);
  float sum = 0.f;
  for (int i = lane; i < n_spans; i += 64) sum += st[2 * i + 1] * expf(st[2 * i] - mx);
  sum = wave_sum_butterfly(sum);
  const float lse = logf(sum);
  const int C = n_spans * K;
  const float* cv = cand_val + (size_t)row * C;
  const int32_t* ci = cand_idx + (size_t)row * C;
  for (int i = lane; i < n_spans; i += 64) { head_v[i] = cv[i]; head_i[i] = ci[i]; }
  if (lane == 0) { n_surv = 0; bound_v = -INFINITY; bound_i = INT_MAX; }
  __syncthreads();
  const int kth = K - 1;
  for (int i = lane; i < n_spans; i += 64) {
    const float v = head_v[i];
    const int id = head_i[i];
    int rank = 0;
    for (int j = 0; j < n_spans; ++j) rank += better(head_v[j], head_i[j], v, id) ? 1 : 0;
    if (rank == kth && v > -INFINITY) { bound_v = v; bound_i = id; }
  }
  __syncthreads();
  const float bv = bound_v;
  const int bi = bound_i;
  for (int i = lane; i < n_spans; i += 64) {
    if (better(bv, bi, head_v[i], head_i[i])) continue;                        // the whole span is worse than the bound
    for (int r = 0; r < K; ++r) {
      const float v = cv[r * n_spans + i];
      const int id = ci[r * n_spans + i];
      if (!(v > -INFINITY) || better(bv, bi, v, id)) break;                    // a span's candidates are in order
      const int pos = atomicAdd(&n_surv, 1);
      surv_v[pos] = v;
      surv_i[pos] = id;
    }
  }
  __syncthreads();
  const int T = n_surv;
  if (lane >= T && lane < K) {
    top_val[row * K + lane] = -INFINITY - mx - lse;
    top_idx[row * K + lane] = 0;
  }
  for (int t = lane; t < T; t += 64) {
    const float v = surv_v[t];
    const int id = surv_i[t];
    int rank = 0;
    for (int j = 0; j < T; ++j) rank += better(surv_v[j], surv_i[j], v, id) ? 1 : 0;
    if (rank < K) {
      top_val[row * K + rank] = v - mx - lse;
      top_idx[row * K + rank] = id;
    }
  }
}

__device__ __forceinline__ int level_base(int level, int K) { return level <= 1 ? 1 : 1 + K + (level - 2) * K * K; }

// (score, id) as one number that is larger for the better entry: larger score first, ties -> smaller id
__device__ __forceinline__ unsigned long long rank_key(float score, int id) {
  const uint32_t u = __float_as_uint(score + 0.f);                       // -0 and 0 are equal
  return (unsigned long long)((u >> 31) ? ~u : u | 0x80000000u) << 32 | (uint32_t)~id;
}

// The merged top K of every row of the last forward, entry K row + rank: log-probability, draft id, target id.  A level's candidates
// are these, at most 256, one per thread.
struct Top { float v[256]; int32_t i[256], t[256]; };
template <int KM>
__device__ __forceinline__ void merge_rows(const Candidates& c, const int32_t* __restrict__ d2t, int n_rows, int K, Top& top) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (wave >= n_rows) return;
  float v;
  int id, target;
  merge_row<KM>(c, d2t, wave, K, lane, v, id, target);
  if (lane < K) { top.v[wave * K + lane] = v; top.i[wave * K + lane] = id; top.t[wave * K + lane] = target; }
}
// Candidate of this thread: those of wavefronts that merge no row, where they are enough, so that what hangs on a candidate's parent
// arrives in the meantime.
__device__ __forceinline__ int candidate_of_thread(int n_rows, int n_cand) {
  const int free = (int)blockDim.x - 64 * n_rows;
  return free >= n_cand ? (int)threadIdx.x - 64 * n_rows : (int)threadIdx.x;
}
__device__ __forceinline__ void write_pool(const DraftState& s, int at, int level, int tok, int par, float score) {
  s.pool_tok[at] = tok;
  s.pool_parent[at] = par;
  s.pool_depth[at] = level;
  s.pool_score[at] = score;
}
__device__ __forceinline__ void write_root(const DraftState& s) {
  s.pool_tok[0] = 0; s.pool_parent[0] = -1; s.pool_depth[0] = 0; s.pool_score[0] = 0.f;
}

// From one draft forward to the next: top-K merge, frontier choice, bookkeeping and input row, one workgroup per row of the next forward.
// As three launches, each of which waits for the one before, they took 4.7 + 4.9 + 6.1 us (K = 10, 8B width), where a launch that does next
// to nothing takes 4.6; here every workgroup repeats the merge (one wavefront per row of the last forward) and the choice (one thread
// per candidate), and the first one writes what is kept of them.  Nothing that is written here is read by another workgroup of the launch.
// K = 10, 8B width: 15.5 us as three launches, 11.2 here, most of it the last round trips (parents, target ids, embedding and feature rows) with
// cold caches; 12.7 with the rotary table (formed by draft_first_kernel for all forwards) and more passes over a row than there are (code that
// arrives a line at a time).  With draft_finish_kernel and draft_first_kernel, both builds in turn: an 8B step 6253 -> 6221 us,
// one layer 1580 -> 1542, the tiny fp32 step 237 -> 210 or, on another box, 220 -> 217.
template <bool BF16, int VPT, int KM>
__global__ __launch_bounds__(1024) void draft_level_kernel(DraftState s, Candidates c, const int32_t* __restrict__ d2t,
                                                          const int32_t* __restrict__ kv_indptr, const int32_t* __restrict__ prefix_len,
                                                          int level, int K, int n_new, DraftInput<BF16> in, const float* __restrict__ feat) {
  __shared__ unsigned long long key[256];
  __shared__ Top top;
  __shared__ RowSums sums;
  __shared__ int row_tok, row_src;
  const int r = row_of_workgroup<BF16>(blockIdx.x);
  if (r >= K) return;
  const int n_rows = level == 1 ? 1 : K, n_cand = n_rows * K, base = level_base(level, K), e = candidate_of_thread(n_rows, n_cand);
  const bool real = e >= 0 && e < n_cand;
  const int P = prefix_len[0], kv_base = kv_indptr[0];
  DraftGains<BF16, VPT> gains;
  load_gains(in, gains);
  int par = 0;
  float before = 0.f;
  uint4 mask = make_uint4(0u, 0u, 0u, 0u);
  if (level > 1 && real) {
    par = s.frontier[(level - 2) * K + e / K];
    before = s.row_score[level & 1][e / K];
    mask = *(const uint4*)(s.row_mask[level & 1] + e / K * 4);
  }
  merge_rows<KM>(c, d2t, n_rows, K, top);
  __syncthreads();
  const float score = real ? (level > 1 ? before + top.v[e] : top.v[e]) : 0.f;
  if (real) key[e] = rank_key(score, e);
  __syncthreads();
  // next frontier: level 1 -> all K candidates in rank order; later levels -> top-K of the K*K
  if (real) {
    const unsigned long long mine = key[e];
    int rank = 0;
#pragma unroll 8
    for (int j = 0; j < n_cand; ++j) rank += key[j] > mine ? 1 : 0;
    const int tail_slot = (level - 1) * K + rank;
    const uint32_t bit = 1u << (tail_slot & 31);
    const int w = tail_slot >> 5;
    mask.x |= w == 0 ? bit : 0u; mask.y |= w == 1 ? bit : 0u; mask.z |= w == 2 ? bit : 0u; mask.w |= w == 3 ? bit : 0u;
    if (rank == r) {                                     // row r of the next forward (level + 1)
      row_tok = top.t[e];
      row_src = level == 1 ? n_new - 1 : n_new + (level - 2) * K + e / K;
      s.row_slot[r] = kv_base + P + n_new + tail_slot;
      s.row_score[(level + 1) & 1][r] = score;
      *(uint4*)(s.row_mask[(level + 1) & 1] + r * 4) = mask;
    }
    if (r == 0) {
      write_pool(s, base + e, level, top.i[e], par, score);
      if (rank < K) s.frontier[(level - 1) * K + rank] = base + e;
    }
  }
  if (r == 0 && threadIdx.x == 0) {
    if (level == 1) write_root(s);
    s.seq[0].kv_base = kv_base;
    s.seq[0].n_prefix = P + n_new;
    s.seq[0].n_tail = level * K;
    s.seq[0].order = 0;
  }
  __syncthreads();
  draft_input_row(in, r, row_tok, feat + (size_t)row_src * in.k, gains, sums);
}

constexpr int MAX_POOL = DRAFT_MAX_POOL;

// After the last forward: its candidates, then the global rerank, in one workgroup.  (Merge, bookkeeping and rerank as three launches:
// 4.6 + 4.9 + 12.3 us, 8B width, K = 10, 711 entries.)  The last level's entries stay in LDS; everything of the levels before that the tree
// may need is requested at the start, two entries to a thread.
// 13.1 us.
template <int NR, int KM>                              // pool <= 64 NR
__global__ __launch_bounds__(1024) void draft_finish_kernel(DraftState s, Candidates c, const int32_t* __restrict__ d2t,
                                                           const int32_t* __restrict__ tok_new, int n_new, int level, int K, int pool,
                                                           int n_nodes, int32_t* __restrict__ tree_tok,
                                                           int32_t* __restrict__ parent, int32_t* __restrict__ node_depth,
                                                           float* __restrict__ cum_logprob,
                                                           int32_t* __restrict__ chosen_dbg) {
  constexpr int PER = NR > 16 ? 2 : 1;        // pool entries of a thread
  __shared__ int16_t node_of[MAX_POOL];       // node id of a kept pool entry, -1 otherwise
  __shared__ Top top;                         // of the last level; v becomes the cumulative scores
  __shared__ int parent_of[256];
  const int tid = threadIdx.x, lane = tid & 63, keep = n_nodes - 1;
  const int n_rows = level == 1 ? 1 : K, n_cand = n_rows * K, base = level_base(level, K), cand = candidate_of_thread(n_rows, n_cand);
  const bool real = cand >= 0 && cand < n_cand;
  int par = 0, old_tok[PER], old_par[PER], old_depth[PER];
  float before = 0.f, older[NR], old_score[PER];
  if (level > 1 && real) { par = s.frontier[(level - 2) * K + cand / K]; before = s.row_score[level & 1][cand / K]; }
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int e = tid + 1024 * i;
    old_tok[i] = old_par[i] = old_depth[i] = 0;
    old_score[i] = 0.f;
    if (e > 0 && e < base) { old_tok[i] = s.pool_tok[e]; old_par[i] = s.pool_parent[e]; old_depth[i] = s.pool_depth[e]; old_score[i] = s.pool_score[e]; }
  }
  // the last wavefront reranks: scores of the levels before
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const int e = 64 * i + lane;
    older[i] = tid >= 960 && e > 0 && e < base ? s.pool_score[e] : 0.f;
  }
  merge_rows<KM>(c, d2t, n_rows, K, top);
#pragma unroll
  for (int i = 0; i < PER; ++i)
    if (tid + 1024 * i > 0 && tid + 1024 * i < base) old_tok[i] = d2t[old_tok[i]];
  __syncthreads();
  if (real) {
    const float score = level > 1 ? before + top.v[cand] : top.v[cand];
    top.v[cand] = score;
    parent_of[cand] = par;
    write_pool(s, base + cand, level, top.i[cand], par, score);
  }
  if (level == 1 && tid == 0) write_root(s);
  __syncthreads();
  // This wavefront holds all scores (entry 64 i + lane in register i, as unsigned numbers in the order of the scores) and
  // finds the keep-th best bit by bit, counting with ballots; ties go to the smaller pool ids.  Node ids follow from bit
  // counts: the kept entries in ascending pool id (the order they were drafted in), after the root.  711 entries, 60 nodes:
  // 10.4 us in a profile (6.4 replayed from a graph), 28.7 us by ranking the survivors of a bound against each other (with a drafted tree nearly all survive).
  if (tid >= 960) {
    uint32_t u[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int e = 64 * i + lane;
      const float score = e >= base && e < pool ? top.v[e - base] : older[i];
      // 0 stands for no entry, below every score (the key of the one NaN with all bits set would be 0 as well)
      u[i] = e > 0 && e < pool ? max((uint32_t)(rank_key(score, e) >> 32), 1u) : 0u;
    }
    uint32_t thr = 0;
    for (int bit = 31; bit >= 0; --bit) {
      const uint32_t next = thr | 1u << bit;
      int n = 0;
#pragma unroll
      for (int i = 0; i < NR; ++i) n += __popcll(__ballot(u[i] >= next));
      if (n >= keep) thr = next;
      if (n == keep) break;
    }
    int ties = keep;                          // entries equal to thr that are kept
#pragma unroll
    for (int i = 0; i < NR; ++i) ties -= __popcll(__ballot(u[i] > thr));
    const unsigned long long below = (1ull << lane) - 1;
    int node = 1;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const unsigned long long eq = __ballot(u[i] == thr);
      const bool kept = u[i] > thr || (u[i] == thr && __popcll(eq & below) < ties);
      const unsigned long long all = __ballot(kept);
      const int e = 64 * i + lane;
      if (e < pool) node_of[e] = kept ? (int16_t)(node + __popcll(all & below)) : e == 0 ? (int16_t)0 : (int16_t)-1;
      ties -= min(ties, (int)__popcll(eq));
      node += __popcll(all);
    }
  }
  __syncthreads();
  if (tid == 0) {
    tree_tok[0] = tok_new[n_new - 1];
    parent[0] = -1;
    node_depth[0] = 0;
    cum_logprob[0] = 0.f;
  }
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int e = tid + 1024 * i;
    if (e == 0 || e >= pool) continue;
    const int nid = node_of[e];
    if (nid < 0) continue;
    const bool last = e >= base;
    tree_tok[nid] = last ? top.t[e - base] : old_tok[i];
    parent[nid] = node_of[last ? parent_of[e - base] : old_par[i]];
    node_depth[nid] = last ? level : old_depth[i];
    cum_logprob[nid] = last ? top.v[e - base] : old_score[i];
    if (chosen_dbg) chosen_dbg[nid - 1] = e;
  }
}

// ---------------------------------------------------------------------------------------------- batched chains
// Chain drafting for a batch (top-1 per level, no tree): forward 1 runs rows1 rows per sequence (the n_new[b] <= rows1
// positions accepted by the previous step, the rest padding), every later forward one row per sequence.

// Rows of forward 1: row (b, j) sits at position P_b + j, cache slot base_b + P_b + j, and sees the draft context plus
// rows 0..j of its own sequence.  Padding rows (j >= n_new[b]) see the same (their results are never used; their
// cache rows land in slots that later forwards overwrite or that stay invisible).
__global__ __launch_bounds__(64) void chain_prep1_kernel(const int32_t* __restrict__ kv_indptr,
                                                        const int32_t* __restrict__ prefix_len, int B, int rows1,
                                                        int32_t* __restrict__ pos, int32_t* __restrict__ slot,
                                                        uint32_t* __restrict__ mask, SeqInfo* __restrict__ seq) {
  const int b = blockIdx.x, j = threadIdx.x;
  const int P = prefix_len[b], base = kv_indptr[b];
  if (j < rows1) {
    const int r = b * rows1 + j;
    pos[r] = P + j;
    slot[r] = base + P + j;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int lo = 32 * w;
      mask[r * 4 + w] = j < lo ? 0u : (j - lo >= 31 ? 0xFFFFFFFFu : ((2u << (j - lo)) - 1u));
    }
  }
  if (j == 0) { seq[b].kv_base = base; seq[b].n_prefix = P; seq[b].n_tail = rows1; seq[b].order = b; }
}

// After forward `level` (1-based) of a chain batch, one workgroup per sequence: the top-1 token of the sequence's last row extends its chain;
// when level < length, its row of the next forward is written, bookkeeping and input (three launches before: see draft_level_kernel).
template <bool BF16, int VPT, int KM>
__global__ __launch_bounds__(1024) void chain_level_kernel(ChainState s, Candidates c, const int32_t* __restrict__ d2t,
                                                          const int32_t* __restrict__ kv_indptr, const int32_t* __restrict__ prefix_len,
                                                          const int32_t* __restrict__ n_new, const int32_t* __restrict__ tok_new, int B,
                                                          int rows1, int level, int length, int32_t* __restrict__ chain_tok,
                                                          float* __restrict__ chain_logp, DraftInput<BF16> in,
                                                          const float* __restrict__ feat) {
  __shared__ RowSums sums;
  __shared__ int row_tok;
  const int b = row_of_workgroup<BF16>(blockIdx.x), tid = threadIdx.x;
  if (b >= B) return;
  const int n = min(max(n_new[b], 1), rows1), P = prefix_len[b], base = kv_indptr[b], at = b * (length + 1);
  DraftGains<BF16, VPT> gains;
  if (level < length) load_gains(in, gains);
  if (tid < 64) {
    float lp;
    int id, tok;
    const float before = level == 1 ? 0.f : chain_logp[at + level - 1];
    merge_row<KM>(c, d2t, b, 1, tid, lp, id, tok);
    if (tid == 0) {
      if (level == 1) {                              // entry 0 of a chain: its root, the last sampled token
        chain_tok[at] = tok_new[b * rows1 + n - 1];
        chain_logp[at] = 0.f;
      }
      chain_tok[at + level] = tok;
      chain_logp[at + level] = before + lp;
      row_tok = tok;
    }
  }
  if (level >= length) return;
  // rows of the next forward: the chain's earlier rows and itself are visible
  if (tid >= (int)blockDim.x - 64)
    for (int i = tid & 63; i < in.head_dim / 2; i += 64) rope_entry(in.cs, b, i, in.head_dim, P + n - 1 + level, in.theta);
  if (tid < 4) {
    const int lo = 32 * tid;
    s.row_mask[b * 4 + tid] = level <= lo ? 0u : (level - lo >= 32 ? 0xFFFFFFFFu : ((1u << (level - lo)) - 1u));
  }
  if (tid == 0) {
    s.row_slot[b] = base + P + n + (level - 1);
    s.seq[b].kv_base = base;
    s.seq[b].n_prefix = P + n;
    s.seq[b].n_tail = level;
    s.seq[b].order = b;
  }
  __syncthreads();
  draft_input_row(in, b, row_tok, feat + (size_t)b * in.k, gains, sums);
}

// x_out[b] = x[b * rows1 + n_new[b] - 1]: the output row of every sequence's last real position.
__global__ __launch_bounds__(256) void chain_gather_kernel(const float* __restrict__ x, const int32_t* __restrict__ n_new,
                                                          int rows1, int k, float* __restrict__ x_out) {
  const int b = blockIdx.x;
  const int n = min(max(n_new[b], 1), rows1);
  const float4* src = (const float4*)(x + ((size_t)b * rows1 + n - 1) * k);
  float4* dst = (float4*)(x_out + (size_t)b * k);
  for (int c = threadIdx.x; c < k / 4; c += 256) dst[c] = src[c];
}

}  // namespace

hipError_t launch_chain_prep1(const int32_t* kv_indptr, const int32_t* prefix_len, int B, int rows1, int32_t* pos,
                              int32_t* slot, uint32_t* mask, SeqInfo* seq, hipStream_t st) {
  if (rows1 < 1 || rows1 > 64) return hipErrorInvalidValue;
  hipLaunchKernelGGL(chain_prep1_kernel, dim3(B), dim3(64), 0, st, kv_indptr, prefix_len, B, rows1, pos, slot, mask, seq);
  return hipGetLastError();
}
hipError_t launch_chain_gather(const float* x, const int32_t* n_new, int B, int rows1, int k, float* x_out, hipStream_t st) {
  hipLaunchKernelGGL(chain_gather_kernel, dim3(B), dim3(256), 0, st, x, n_new, rows1, k, x_out);
  return hipGetLastError();
}

size_t topk_scratch_floats(int n_rows, int V, int K) {
  const size_t n_spans = (size_t)(V + TOPK_SPAN - 1) / TOPK_SPAN;
  return (size_t)n_rows * n_spans * (2 * (size_t)K + 2);
}

namespace {

// The candidates of n_rows rows, merged as well where there are more spans than a wavefront has lanes.
hipError_t launch_candidates(const DraftLogits& zl, int n_rows, int K, float* top_val, int32_t* top_idx, Candidates& c, hipStream_t st) {
  if (n_rows <= 0 || zl.V <= 0 || K <= 0 || K > TOPK_MAX_K) return hipErrorInvalidValue;
  const int n_spans = (zl.V + TOPK_SPAN - 1) / TOPK_SPAN;
  if (n_spans > TOPK_MAX_SPANS) return hipErrorInvalidValue;
  float* cand_val = zl.scratch;
  int32_t* cand_idx = (int32_t*)(zl.scratch + (size_t)n_rows * n_spans * K);
  float* span_stat = zl.scratch + 2 * (size_t)n_rows * n_spans * K;
  c = {cand_val, cand_idx, span_stat, n_spans, top_val, top_idx};
  hipLaunchKernelGGL(topk_spans_kernel, dim3((n_spans + 3) / 4, n_rows), dim3(256), 0, st, zl.z, zl.V, zl.row0, zl.V, K, n_spans,
                     cand_val, cand_idx, span_stat);
  if (n_spans > 64)
    hipLaunchKernelGGL(topk_merge_kernel, dim3(n_rows), dim3(64), 0, st, cand_val, cand_idx, span_stat, n_spans, K, top_val, top_idx);
  return hipGetLastError();
}

// The candidates are registers, and those beyond K cost 0.05-0.1 us each, so there are three sizes: 10 rows of 32000, spans and
// merge, K = 4: 6.3 us with 4, 6.6 with 10, 6.9 with 16; K = 10: 9.5 with 10, 10.0 with 16.
template <typename F>
hipError_t with_candidates(const Candidates& c, int K, F f) {
  if (c.n_spans > 64) f(Int<0>());
  else if (K <= 4) f(Int<4>());
  else if (K <= 10) f(Int<10>());
  else f(Int<16>());
  return hipGetLastError();
}

// A thread per four columns of a row, and at least a wavefront for each row that is merged and one more.
int level_threads(int k, int rows) { return std::min(1024, std::max((k / 4 + 63) / 64, rows + 1) * 64); }

}  // namespace

hipError_t launch_draft_level(bool bf16, const DraftState& s, const DraftLogits& zl, const int32_t* d2t, const int32_t* kv_indptr,
                              const int32_t* prefix_len, int level, int K, int n_new, const DraftInputArgs& in, const float* feat,
                              hipStream_t st) {
  Candidates c;
  if (!draft_input_ok(in)) return hipErrorInvalidValue;
  if (hipError_t e = launch_candidates(zl, level == 1 ? 1 : K, K, s.top_val, s.top_idx, c, st)) return e;
  const int threads = level_threads(in.k, K);
  return with_candidates(c, K, [&](auto km) {
    (void)with_input(bf16, in.k, threads, [&](auto type, auto passes) {
      hipLaunchKernelGGL((draft_level_kernel<type.value, passes.value, km.value>), dim3(bf16 ? rows_grid(K) : K), dim3(threads), 0, st, s, c,
                         d2t, kv_indptr, prefix_len, level, K, n_new, draft_input<type.value>(in), feat);
    });
  });
}

hipError_t launch_draft_finish(const DraftState& s, const DraftLogits& zl, const int32_t* d2t, const int32_t* tok_new, int n_new, int depth,
                               int K, int n_nodes, int32_t* tree_tok, int32_t* parent, int32_t* node_depth, float* cum_logprob,
                               int32_t* chosen_dbg, hipStream_t st) {
  const int pool = 1 + K + (depth - 1) * K * K;
  if (pool > MAX_POOL || n_nodes - 1 > pool - 1 || n_nodes > 64) return hipErrorInvalidValue;   // a tree has at most 64 nodes
  Candidates c;
  if (hipError_t e = launch_candidates(zl, depth == 1 ? 1 : K, K, s.top_val, s.top_idx, c, st)) return e;
  // A register per 64 entries, and each costs 0.2-0.25 us whether it is used or not, so there are three sizes: 201 entries 3.3 us with
  // 4 registers, 5.3 with 12, 10.8 with 32; 711 entries 6.4 with 12, 12.3 with 32 (the rerank alone).
  return with_candidates(c, K, [&](auto km) {
    auto finish = pool <= 256 ? draft_finish_kernel<4, km.value> : pool <= 768 ? draft_finish_kernel<12, km.value>
                                                                               : draft_finish_kernel<MAX_POOL / 64, km.value>;
    hipLaunchKernelGGL(finish, dim3(1), dim3(1024), 0, st, s, c, d2t, tok_new, n_new, depth, K, pool, n_nodes, tree_tok, parent, node_depth,
                       cum_logprob, chosen_dbg);
  });
}

hipError_t launch_chain_level(bool bf16, const ChainState& s, const DraftLogits& zl, const int32_t* d2t, const int32_t* kv_indptr,
                              const int32_t* prefix_len, const int32_t* n_new, const int32_t* tok_new, int B, int rows1, int level,
                              int length, int32_t* chain_tok, float* chain_logp, const DraftInputArgs& in, const float* feat,
                              hipStream_t st) {
  Candidates c;
  if (length > 120 || !draft_input_ok(in)) return hipErrorInvalidValue;
  if (hipError_t e = launch_candidates(zl, B, 1, s.top_val, s.top_idx, c, st)) return e;
  const int threads = level_threads(in.k, 1);
  auto launch = [&](auto km) {
    return with_input(bf16, in.k, threads, [&](auto type, auto passes) {
      hipLaunchKernelGGL((chain_level_kernel<type.value, passes.value, km.value>), dim3(bf16 ? rows_grid(B) : B), dim3(threads), 0, st, s, c,
                         d2t, kv_indptr, prefix_len, n_new, tok_new, B, rows1, level, length, chain_tok, chain_logp,
                         draft_input<type.value>(in), feat);
    });
  };
  return c.n_spans > 64 ? launch(Int<0>()) : launch(Int<1>());
}
