// Host-side launch interface of the gfx950 kernels (one definition per .hip file).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

typedef uint16_t bf16_t;

// ---------------------------------------------------------------- GEMM (gemm_skinny.hip, gemm_f32.hip)
// Weight operand: up to three [rows_i, K] row-major matrices.
//   mode 0: their rows are concatenated (q|k|v projections run as one GEMM);
//   mode 1: tiles interleave rows of w[0] (gate) with the same rows of w[1] (up), 32 at a time or, in tiles of 192 and 224
//           weight rows, 8, so that the SwiGLU product can be formed in the epilogue.
struct GemmWeights {
  const void* w[3];
  int rows[3];
  int nmat;
  int mode;
};
enum { GEMM_EPI_PARTIAL = 0, GEMM_EPI_SWIGLU = 1, GEMM_EPI_RESIDUAL = 2, GEMM_EPI_ROPE = 3 };   // the last two: fp32 only

// Y = X W^T for few rows (M <= a few hundred) streaming the weights once: bf16 inputs, fp32 accumulate.
//   x      fragment-major bf16 [ceil64(M), K] (see xf_offset)
//   out    epi PARTIAL: fp32 [S, M, N] (split-K partial sums, S = splits); the consumer adds them
//          epi SWIGLU : fragment-major bf16 [ceil64(M), N/2] = silu(gate) * up   (requires S == 1)
// Requires K % (128*S) == 0.  N = total weight rows.  ev_start / ev_stop (optional): events attached to the dispatch.
hipError_t launch_gemm_skinny(const bf16_t* x, const GemmWeights& W, int M, int N, int K, int S, int epi,
                              void* out, hipStream_t st, hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr);

// The same product for many rows (M > 64): MFMA-bound tiling, see gemm_wide.hip.  Chooses tile shape and split-K
// itself (S <= what fits into out_capacity_floats; 0 forces S = 1) and reports S.
hipError_t launch_gemm_wide(const bf16_t* x, const GemmWeights& W, int M, int N, int K, int epi, void* out,
                            size_t out_capacity_floats, int* S_out, hipStream_t st, hipEvent_t ev_start = nullptr,
                            hipEvent_t ev_stop = nullptr);

// q/k/v (W: their three matrices, head size 128) rotated, k and v in the cache rows slot[m]; where wide_rope_fits says so.
struct WideRope {
  const float* cs = nullptr;            // rotary tables, cs_step from one row's to the next one's
  int cs_step = 0;
  const int32_t* slot = nullptr;
  int H = 0, Hkv = 0;
  bf16_t* q = nullptr;                  // [M, H, 128]
  bf16_t* kc = nullptr;
  bf16_t* vc = nullptr;
};
bool wide_rope_fits(int M, int N, int K, size_t out_capacity_floats);
hipError_t launch_gemm_wide_rope(const bf16_t* x, const GemmWeights& W, int M, int N, int K, const WideRope& rope, size_t out_capacity_floats,
                                 hipStream_t st, hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr);

// The same for at most 64 rows in tiles of 64 x cols (128 or 256), in S ranges of K.  Weights at multiples of 16 bytes.
hipError_t launch_gemm_wide64(const bf16_t* x, const GemmWeights& W, int M, int N, int K, int cols, int S, int epi, void* out,
                              hipStream_t st, hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr);

// fp32 GEMM, exact arithmetic: x [M, K], weights [N, K] stacked.  epi PARTIAL: out [M, N]; SWIGLU (mode 1): out [M, N / 2];
// RESIDUAL: out [M, N] += , and copies of the sum to each non-null copies[i]; ROPE: the rows are q|k|v heads, out = q [M, H, d]
// rotated, k rotated and v to the cache rows slot[m].
struct F32Fuse {
  const float* gain = nullptr;          // x is the RMSNorm of the rows given, with this gain
  float eps = 0.f;
  float* copies[4] = {nullptr, nullptr, nullptr, nullptr};
  const float* cs = nullptr;            // rotary tables, cs_step from one row's to the next one's
  int cs_step = 0;
  const int32_t* slot = nullptr;
  float* kc = nullptr;
  float* vc = nullptr;
  int H = 0, Hkv = 0, d = 0;
};
hipError_t launch_gemm_f32(const float* x, const GemmWeights& W, int M, int N, int K, int epi, float* out, hipStream_t st,
                           const F32Fuse& fuse = F32Fuse());

// ---------------------------------------------------------------- elementwise (elementwise.hip)
struct SeqInfo {           // one per sequence, device resident
  int32_t kv_base;         // first cache slot of the sequence
  int32_t n_prefix;        // slots visible to every row
  int32_t n_tail;          // following slots, visible according to the per-row bit mask
  int32_t order;           // entry i: the sequence that attention workgroup group i works on (longest first)
};

// The first launch of a pass over R rows: bookkeeping, and the rows' residual.
struct BeginRows {
  const void* embed;                    // x = embed[tok], or null: x holds the rows
  const int32_t* tok;
  int vocab;
  const int32_t* parent;                // B trees of N nodes: 128-bit ancestor masks; null: a prefill chunk, causal masks in blocks of 64 rows
  int B, N;
  const int32_t* kv_indptr;
  const int32_t* prefix_len;
  int head_dim;
  float theta;
  int32_t* slot;                        // [R] cache slots
  uint32_t* mask;                       // [R][4]
  float* cs;                            // [R][head_dim] rotary tables
  SeqInfo* seq;                         // one per tree, or block
};
// copies x to each non-null copy_out; with a gain: act = RMSNorm(x; gain) in the activation layout
hipError_t launch_begin_rows(bool bf16, const BeginRows& b, float* x, int R, int k, const void* gain, float eps, void* act,
                             float* const copy_out[4], hipStream_t st);
// cs[0] = the rotary table of position prefix_len[0] + at.
hipError_t launch_rope_table(float* cs, const int32_t* prefix_len, int at, int head_dim, float theta, hipStream_t st);
// After a prefill chunk: len[0] += n, draft_len[0] += m.
hipError_t launch_end_prefill(int32_t* len, int n, int32_t* draft_len, int m, hipStream_t st);
// x += sum_s partial[s]; copies x to each non-null copy_out; act = RMSNorm(x; gain) in the activation layout.
hipError_t launch_add_norm(bool bf16, float* x, const float* partial, int S, int R, int k, const void* gain, float eps,
                           void* act, float* const copy_out[4], hipStream_t st);
// bf16: sums the q|k|v split-K partials, rotates q and k, writes q [R,H,d] and the cache rows.  cs_step: from a row's rotary table to the
// next one's (0: all rows at one position).
hipError_t launch_rope_kv_write(const float* qkv_partial, int S, int R, int H, int Hkv, int d, const float* cs, int cs_step,
                                const int32_t* slot, void* q, void* kcache, void* vcache, hipStream_t st);
hipError_t launch_pack3(bool bf16, const float* a, const float* b, const float* c, int M, int k, void* act, hipStream_t st);
hipError_t launch_reduce_partials(const float* partial, int S, int M, int N, float* out, hipStream_t st);
// Draft layer input: act[r] = [RMSNorm(E[tok[r]]; g_embed) ; RMSNorm(f_r; g_feat)], y[r] = f_r, and the rotary table cs[r] of the
// row's position.
struct DraftInputArgs {
  const void* embed;
  const void* g_embed;
  const void* g_feat;
  void* act;
  float* y;
  float* cs;
  int vocab, k, head_dim;
  float eps, theta;
};
// f_r = feat[r], positions already on the device
hipError_t launch_draft_input(bool bf16, const DraftInputArgs& a, const int32_t* tok, const float* feat, const int32_t* pos, int M,
                              hipStream_t st);
// The same for draft forward 1 of a tree (the n_new positions behind the context), with slots, causal masks, sequence info, and the
// rotary tables of the later forwards: cs[n_new + l - 2] is that of forward l.  Without mask and seq: any number of rows.
hipError_t launch_draft_first(bool bf16, const DraftInputArgs& a, const int32_t* tok, const float* feat, const int32_t* kv_indptr,
                              const int32_t* prefix_len, int n_new, int depth, int32_t* slot, uint32_t* mask, SeqInfo* seq,
                              hipStream_t st);

// ---------------------------------------------------------------- attention (attention.hip)
// Tree-masked attention of rows [B * rows_per_seq] against a (ragged) cache.
//   bf16: q [R,H,d] bf16, cache bf16, out = fragment-major bf16 [R, H*d]; d must be 128.
//   fp32: q fp32, cache fp32, out row-major fp32.
// scratch: fp32 workspace of attention_scratch_floats(...) elements.
size_t attention_scratch_floats(int R, int H, int d, int max_splits);
int attention_pick_splits(int B, int rows_per_seq, int H, int Hkv, int max_len);
hipError_t launch_tree_attention(bool bf16, const void* q, const void* kcache, const void* vcache, const SeqInfo* seq,
                                 const uint32_t* mask, int B, int rows_per_seq, int H, int Hkv, int d, int max_len,
                                 int n_splits, float* scratch, void* out, hipStream_t st);

// ---------------------------------------------------------------- draft tree (select.hip)
#define DRAFT_MAX_POOL 2048   /* candidates the final rerank can hold: 1 + K + (D-1) K^2 must not exceed it */
struct DraftState {          // device arrays owned by the workspace
  int32_t* pool_tok;         // [pool] draft ids
  int32_t* pool_parent;      // [pool]
  int32_t* pool_depth;       // [pool]
  float* pool_score;         // [pool]
  int32_t* frontier;         // [D][K] pool ids expanded by forward l+1 (row 0 = level-1 candidates)
  float* top_val;            // [max_rows][K] log-probabilities of the per-row top-K
  int32_t* top_idx;          // [max_rows][K]
  // rows of the next forward; those of forward l at l & 1, as a launch reads one set while it writes the other
  int32_t* row_slot;         // [K]
  uint32_t* row_mask[2];     // [K][4]
  float* row_score[2];       // [K] cumulative log-probability
  SeqInfo* seq;              // [1]
};
// scratch: topk_scratch_floats(n_rows, V, K) floats.
size_t topk_scratch_floats(int n_rows, int V, int K);
// What a draft forward left: logits z[rows, V] and where their top K go through.
struct DraftLogits {
  const float* z;
  int row0, V;
  float* scratch;
};
// After forward `level` < depth (1-based): per-row log-softmax and top-K (value desc, id asc), the new pool entries, the next frontier,
// and the next forward's rows: bookkeeping and input (f_r = feat[row of the parent's output]), but for the rotary table.
hipError_t launch_draft_level(bool bf16, const DraftState& s, const DraftLogits& zl, const int32_t* d2t, const int32_t* kv_indptr,
                              const int32_t* prefix_len, int level, int K, int n_new, const DraftInputArgs& in, const float* feat,
                              hipStream_t st);
// After the last forward: its pool entries, then the global rerank and the tree.
hipError_t launch_draft_finish(const DraftState& s, const DraftLogits& zl, const int32_t* d2t, const int32_t* tok_new, int n_new, int depth,
                               int K, int n_nodes, int32_t* tree_tok, int32_t* parent, int32_t* node_depth, float* cum_logprob,
                               int32_t* chosen_dbg, hipStream_t st);

// Batched chain drafting: per-sequence state of the next forward (one row per sequence), device arrays.
struct ChainState {
  float* top_val;            // [B] log-probability of the top-1 token of every sequence's last row
  int32_t* top_idx;          // [B] its draft id
  int32_t* row_slot;         // [B]
  uint32_t* row_mask;        // [B][4]
  SeqInfo* seq;              // [B]
};
hipError_t launch_chain_prep1(const int32_t* kv_indptr, const int32_t* prefix_len, int B, int rows1, int32_t* pos,
                              int32_t* slot, uint32_t* mask, SeqInfo* seq, hipStream_t st);
// After forward `level` (1-based) of a chain batch: the top-1 token of every sequence's last row extends its chain; when level < length, the
// next forward's rows (one per sequence, f_r = feat[sequence]) are written.
hipError_t launch_chain_level(bool bf16, const ChainState& s, const DraftLogits& zl, const int32_t* d2t, const int32_t* kv_indptr,
                              const int32_t* prefix_len, const int32_t* n_new, const int32_t* tok_new, int B, int rows1, int level,
                              int length, int32_t* chain_tok, float* chain_logp, const DraftInputArgs& in, const float* feat,
                              hipStream_t st);
hipError_t launch_chain_gather(const float* x, const int32_t* n_new, int B, int rows1, int k, float* x_out, hipStream_t st);

// ---------------------------------------------------------------- acceptance (accept.hip)
#define ACCEPT_CHUNK 2048
size_t accept_scratch_floats(int R, int V);
hipError_t launch_accept(const float* logits, const int32_t* tree_tok, const int32_t* parent, int B, int N, int V,
                         float temperature, const float* uniforms, float* scratch, int32_t* accept_len, int32_t* path,
                         int32_t* bonus, hipStream_t st);

// ---------------------------------------------------------------- commit (commit.hip)
// Moves the accepted nodes' cache rows to the front of the tree slots (every layer, in place), gathers their
// features and following tokens, advances the prefix lengths.  k_layers / v_layers: host arrays of device pointers.
hipError_t launch_commit(void* const* k_layers, void* const* v_layers, int n_layers, const int32_t* kv_indptr,
                         int32_t* prefix_len, const int32_t* tree_tok, const int32_t* path, const int32_t* accept_len,
                         const int32_t* bonus, const float* taps, int B, int N, int hidden, int row_bytes, int rows,
                         float* taps_new, int32_t* tok_new, int32_t* n_new, int32_t* draft_prefix_len, int draft_rows,
                         hipStream_t st);

// ---------------------------------------------------------------- training-time-test attention (causal_attention.hip)
// q [T,H,d], k / v [s+1,T,Hkv,d] (bf16 with d == 128, or fp32), out fp32 [T,H,d].
hipError_t launch_ttt_attention(bool bf16, const void* q, const void* k, const void* v, int T, int H, int Hkv, int d, int s,
                                float* out, hipStream_t st);
// Causal attention of a prefill chunk (bf16, d == 128): rows 0..n-1 at positions seq[0].n_prefix + row of one sequence, whose
// cache rows, the chunk's own included, are written.  q [n, H, d] bf16, out fragment-major bf16 [n, H * d].
hipError_t launch_prefill_attention(const void* q, const void* kcache, const void* vcache, const SeqInfo* seq, int n, int H, int Hkv,
                                    int d, void* out, hipStream_t st);
