// C ABI (include/eagle3.h): argument checks, workspace carving and the launch sequences of the four
// step calls.  No arithmetic of the method happens on the host.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

#include "../../include/eagle3.h"
#include "../../include/eagle3_measure.h"
#include "causal_rules.hpp"
#include "common.hpp"
#include "kernels.hpp"
#include "wide_tiles.hpp"

namespace {

thread_local char g_err[512] = "";

int fail_hip(hipError_t e, const char* what) {
  snprintf(g_err, sizeof(g_err), "%s: %s", what, hipGetErrorString(e));
  return EAGLE3_E_HIP;
}
#define CK(expr)                                             \
  do {                                                       \
    hipError_t _e = (expr);                                  \
    if (_e != hipSuccess) return fail_hip(_e, #expr);        \
  } while (0)

size_t align_up(size_t v, size_t a = 256) { return (v + a - 1) / a * a; }

// Rows of a prefill chunk, as far as the workspace that the caller hands over holds them.  bf16: one pass over the weights serves
// the whole chunk, and from about 2048 rows on the products run at the matrix cores' rate and more rows no longer help
// (an 8B-shaped prompt of 2048 tokens, 32 layers: 139.6 ms in chunks of 64).  fp32 (small models, exact kernels): enough rows
// to amortise the launches.
constexpr int PREFILL_ROWS_BF16 = 2048, PREFILL_ROWS_FP32 = 256;

struct Carver {          // first pass (base == nullptr) measures, second pass hands out pointers
  char* base;
  size_t off = 0;
  explicit Carver(void* b) : base((char*)b) {}
  template <typename T> T* take(size_t n) {
    T* p = base ? (T*)(base + off) : nullptr;
    off += align_up(n * sizeof(T));
    return p;
  }
};

}  // namespace

struct eagle3_ctx {
  eagle3_config cfg;
  bool bf16;
  size_t act_size;                      // bytes per activation element
  std::vector<eagle3_layer_weights> layers;
  eagle3_target_weights tw;
  eagle3_draft_weights dw;
  bool has_target = false, has_draft = false;
  void* ws = nullptr;
  size_t ws_bytes = 0, ws_full = 0;     // ws_full: with prefill chunks of full length
  size_t ws_need = 0;                   // ws_need: of the present sizes (size_for)

  // optional per-launch timing of the GEMMs
  bool profiling = false;
  struct Stamp { hipEvent_t a, b; double bytes; int kind; };
  std::vector<Stamp> stamps;
  size_t stamps_used = 0;

  int R_max, Md_max, Rall, a_rows, pool_max;     // Rall: rows of the widest launch
  size_t part_floats, attn_floats;
  // workspace
  float* x; void* act_k; void* act_attn; void* act_h; void* q; float* part; float* attn_scratch;
  uint32_t* mask; int32_t* slot; float* cs; SeqInfo* seq;
  float* accept_stats;
  float* z; float* a_buf; int32_t* pos1; float* topk_scratch; DraftState ds;
  int chunk_max;                        // rows per prefill chunk: a multiple of 64, or fewer than 64
  float* chunk_taps; float* chunk_g;
  int rows1_max;                        // rows per sequence of a chain batch's forward 1
  ChainState cs_chain;

  int chunk_full() const { return bf16 ? PREFILL_ROWS_BF16 : PREFILL_ROWS_FP32; }
  int chunk_least() const { return std::min(cfg.max_nodes, cfg.max_new); }      // prefill adds no rows to those of the step calls

  // Sizes of everything when prefill runs in chunks of `chunk` rows.
  void size_for(int chunk) {
    const eagle3_config& c = cfg;
    chunk_max = chunk;
    const int R_step = std::max(R_max, Md_max);
    Rall = std::max(R_step, chunk);
    const size_t widest = std::max<size_t>((size_t)(c.n_heads + 2 * c.n_kv_heads) * c.head_dim, c.hidden);
    // split-K partial sums: up to 4 slices of the widest projection, 8 of a hidden-sized one; 2 for a prefill chunk, whose
    // many rows fill the chip without more
    part_floats = bf16 ? std::max<size_t>({1024 * widest, 4 * (size_t)R_step * widest, 8 * (size_t)R_step * c.hidden, 2 * (size_t)chunk * widest}) : 1;
    size_t af = 0;
    auto attention = [&](int batch, int rows) {
      const int s = attention_pick_splits(batch, rows, c.n_heads, c.n_kv_heads, 1 << 30);
      af = std::max(af, attention_scratch_floats(batch * rows, c.n_heads, c.head_dim, s));
    };
    for (int b = 1; b <= c.max_batch; ++b) attention(b, c.max_nodes);
    attention(1, Md_max);
    // prefill: blocks of 64 rows, as long as their number can be one that the unsplit kernel does not take at every length
    for (int b = 1; 64 * b <= chunk && !prefill_attention_fits(64 * (b - 1) + 1, c.n_heads, c.n_kv_heads, 1 << 30); ++b) attention(b, 64);
    attn_floats = bf16 ? af : 1;
    carve(nullptr);
  }

  void carve(void* base) {
    const eagle3_config& c = cfg;
    Carver cv(base);
    const size_t k = c.hidden, I = c.intermediate, Hd = (size_t)c.n_heads * c.head_dim;
    const size_t Rpad = (size_t)(Rall + 63) / 64 * 64;
    x = cv.take<float>((size_t)Rall * k);
    act_k = cv.take<char>(Rpad * 3 * k * act_size);
    act_attn = cv.take<char>(Rpad * Hd * act_size);
    act_h = cv.take<char>(Rpad * I * act_size);
    q = cv.take<char>((size_t)Rall * Hd * act_size);
    part = cv.take<float>(part_floats);
    attn_scratch = cv.take<float>(attn_floats);
    mask = cv.take<uint32_t>((size_t)Rall * 4);
    slot = cv.take<int32_t>(Rall);
    cs = cv.take<float>((size_t)Rall * c.head_dim);
    seq = cv.take<SeqInfo>(std::max(c.max_batch, (chunk_max + 63) / 64));
    accept_stats = cv.take<float>(accept_scratch_floats(R_max, c.vocab));
    const int mb = std::max(c.max_batch, 1);
    z = cv.take<float>((size_t)std::max(Md_max, mb) * c.draft_vocab);
    a_buf = cv.take<float>((size_t)std::max(a_rows, mb * rows1_max) * k);
    pos1 = cv.take<int32_t>(Rall);
    topk_scratch = cv.take<float>(std::max(topk_scratch_floats(c.max_topk, c.draft_vocab, c.max_topk),
                                           topk_scratch_floats(mb, c.draft_vocab, 1)));
    cs_chain.top_val = cv.take<float>(mb);
    cs_chain.top_idx = cv.take<int32_t>(mb);
    cs_chain.row_slot = cv.take<int32_t>(mb);
    cs_chain.row_mask = cv.take<uint32_t>((size_t)mb * 4);
    cs_chain.seq = cv.take<SeqInfo>(mb);
    ds.pool_tok = cv.take<int32_t>(pool_max);
    ds.pool_parent = cv.take<int32_t>(pool_max);
    ds.pool_depth = cv.take<int32_t>(pool_max);
    ds.pool_score = cv.take<float>(pool_max);
    ds.frontier = cv.take<int32_t>((size_t)c.max_depth * c.max_topk);
    ds.top_val = cv.take<float>((size_t)Md_max * c.max_topk);
    ds.top_idx = cv.take<int32_t>((size_t)Md_max * c.max_topk);
    ds.row_slot = cv.take<int32_t>(c.max_topk);
    for (int i = 0; i < 2; ++i) {
      ds.row_mask[i] = cv.take<uint32_t>((size_t)c.max_topk * 4);
      ds.row_score[i] = cv.take<float>(c.max_topk);
    }
    ds.seq = cv.take<SeqInfo>(1);
    chunk_taps = cv.take<float>((size_t)3 * chunk_max * k);
    chunk_g = cv.take<float>((size_t)chunk_max * k);
    ws_need = cv.off;
  }

  Stamp* stamp(double bytes, int kind) {               // of the next GEMM launch, where launches are timed
    if (!profiling || stamps_used >= stamps.size()) return nullptr;
    Stamp* sp = &stamps[stamps_used++];
    sp->bytes = bytes;
    sp->kind = kind;
    return sp;
  }

  DraftInputArgs draft_input_args() const {
    return {tw.embed, dw.norm_embed, dw.norm_feat, act_k, x, cs, cfg.vocab, cfg.hidden, cfg.head_dim, cfg.rms_eps, cfg.rope_theta};
  }

  // One projection Y = act W^T.  epi PARTIAL: result (S partial sums) in `part`; *S_out = S.
  // epi SWIGLU: silu(gate)*up lands in act_h.  fp32: to direct_out only (a layer's products are fused with what follows them).
  int project(const void* act_in, const GemmWeights& W, int M, int N, int K, int epi, int* S_out, hipStream_t st,
              float* direct_out = nullptr) {
    if (bf16 && M > 64) {
      Stamp* sp = stamp(2.0 * N * K, EAGLE3_GEMM_MANY_ROWS);
      int S = 1;
      // A result that goes straight to its place is not split, except where more inputs than outputs leave CUs idle (the fusion
      // of a prompt's features, K = 3 N: the partial sums are small against the weights then).  8B width, us, unsplit / split and
      // summed: 77 rows 136 / 28 + 6, 512 rows 139 / 56 + 15, 1024 rows 145 / 95 + 17.
      const bool split = direct_out && N < K && ((N + 127) / 128) * ((M + 127) / 128) <= 256 &&
                         many_tiles(M, N, K, false, part_floats).S > 1;
      void* out = epi == GEMM_EPI_SWIGLU ? act_h : (direct_out && !split ? (void*)direct_out : (void*)part);
      CK(launch_gemm_wide((const bf16_t*)act_in, W, M, N, K, epi, out, direct_out && !split ? 0 : part_floats, &S, st,
                          sp ? sp->a : nullptr, sp ? sp->b : nullptr));
      if (split) CK(launch_reduce_partials(part, S, M, N, direct_out, st));
      if (S_out) *S_out = S;
      return EAGLE3_OK;
    }
    if (bf16) {
      // what the direct loads of the wider tiles need
      bool wide_ok = W.mode == 0 || N % 8 == 0;
      for (int i = 0; i < W.nmat; ++i) wide_ok = wide_ok && (uintptr_t)W.w[i] % 16 == 0 && (W.nmat == 1 || W.rows[i] % 8 == 0);
      const FewRows t = few_rows(M, N, K, epi == GEMM_EPI_SWIGLU, direct_out != nullptr, part_floats, wide_ok);
      const int S = t.S;
      if (epi == GEMM_EPI_PARTIAL && direct_out == nullptr && (size_t)S * M * N > part_floats) return EAGLE3_E_STATE;
      void* out = epi == GEMM_EPI_SWIGLU ? act_h : (direct_out && S == 1 ? (void*)direct_out : (void*)part);
      Stamp* sp = stamp(2.0 * N * K, M <= 32 ? EAGLE3_GEMM_FEW_ROWS : t.cols == 64 ? EAGLE3_GEMM_TILE64 : EAGLE3_GEMM_TILE128);
      if (t.cols == 64)
        CK(launch_gemm_skinny((const bf16_t*)act_in, W, M, N, K, S, epi, out, st, sp ? sp->a : nullptr, sp ? sp->b : nullptr));
      else
        CK(launch_gemm_wide64((const bf16_t*)act_in, W, M, N, K, t.cols, S, epi, out, st, sp ? sp->a : nullptr, sp ? sp->b : nullptr));
      if (direct_out && S > 1) CK(launch_reduce_partials(part, S, M, N, direct_out, st));
      if (S_out) *S_out = S;
      return EAGLE3_OK;
    }
    CK(launch_gemm_f32((const float*)act_in, W, M, N, K, epi, direct_out, st));
    if (S_out) *S_out = 1;
    return EAGLE3_OK;
  }
};

#define TRY(expr)                  \
  do {                             \
    int _rc = (expr);              \
    if (_rc != EAGLE3_OK) return _rc; \
  } while (0)

extern "C" {

const char* eagle3_strerror(int code) {
  switch (code) {
    case EAGLE3_OK: return "ok";
    case EAGLE3_E_NULL: return "a required pointer is NULL";
    case EAGLE3_E_SHAPE: return "a size is outside what the configuration or the kernels support";
    case EAGLE3_E_STATE: return "weights or workspace not set, or workspace too small";
    case EAGLE3_E_HIP: return "a HIP call failed (see eagle3_last_error)";
    default: return "unknown error code";
  }
}
const char* eagle3_last_error(void) { return g_err; }

int eagle3_create(const eagle3_config* cfg, eagle3_ctx** out) {
  if (!cfg || !out) return EAGLE3_E_NULL;
  const eagle3_config& c = *cfg;
  if (c.hidden <= 0 || c.n_heads <= 0 || c.n_kv_heads <= 0 || c.head_dim <= 0 || c.intermediate <= 0 || c.vocab <= 0 ||
      c.draft_vocab <= 0 || c.draft_vocab > 512 * 1024 || c.n_layers <= 0 || c.n_heads % c.n_kv_heads != 0)
    return EAGLE3_E_SHAPE;
  if (c.dtype != EAGLE3_BF16 && c.dtype != EAGLE3_FP32) return EAGLE3_E_SHAPE;
  if (c.max_batch < 1 || c.max_nodes < 1 || c.max_nodes > 64 || c.max_depth < 1 || c.max_topk < 1 || c.max_topk > 16 ||
      c.max_new < 1 || c.max_new > 64 || (c.max_depth - 1) * c.max_topk > 128 ||
      1 + c.max_topk + (c.max_depth - 1) * c.max_topk * c.max_topk > DRAFT_MAX_POOL)
    return EAGLE3_E_SHAPE;
  for (int t = 0; t < 3; ++t)
    if (c.tap_layers[t] < 0 || c.tap_layers[t] >= c.n_layers) return EAGLE3_E_SHAPE;
  if (c.dtype == EAGLE3_BF16) {
    if (c.head_dim != 128 || c.hidden % 128 || c.intermediate % 128 || (c.n_heads * c.head_dim) % 128)
      return EAGLE3_E_SHAPE;
    // launches of more than 64 rows go through the many-row GEMM, which stores four outputs at a time
    const long many = std::max((long)c.max_batch * c.max_nodes, (long)c.max_batch * c.max_new);
    if (many > 64 && (c.vocab % 4 || c.draft_vocab % 4)) return EAGLE3_E_SHAPE;
  } else {
    if (c.head_dim % 2 || c.head_dim > 256) return EAGLE3_E_SHAPE;
  }
  if (!(c.rope_theta > 0.f) || !(c.rms_eps >= 0.f)) return EAGLE3_E_SHAPE;
  eagle3_ctx* ctx = new (std::nothrow) eagle3_ctx();
  if (!ctx) return EAGLE3_E_STATE;
  ctx->cfg = c;
  ctx->bf16 = c.dtype == EAGLE3_BF16;
  ctx->act_size = ctx->bf16 ? 2 : 4;
  ctx->R_max = c.max_batch * c.max_nodes;
  ctx->Md_max = std::max(c.max_new, c.max_topk);
  ctx->a_rows = c.max_new + (c.max_depth - 1) * c.max_topk;
  ctx->rows1_max = std::min(c.max_nodes, c.max_new);
  ctx->pool_max = 1 + c.max_topk + (c.max_depth - 1) * c.max_topk * c.max_topk;
  ctx->size_for(ctx->chunk_full());
  ctx->ws_full = ctx->ws_need;
  *out = ctx;
  return EAGLE3_OK;
}

int eagle3_destroy(eagle3_ctx* ctx) {
  if (ctx)
    for (auto& s : ctx->stamps) {
      (void)hipEventDestroy(s.a);
      (void)hipEventDestroy(s.b);
    }
  delete ctx;
  return EAGLE3_OK;
}

int eagle3_workspace_bytes(const eagle3_ctx* ctx, size_t* out) {
  if (!ctx || !out) return EAGLE3_E_NULL;
  *out = ctx->ws_full;
  return EAGLE3_OK;
}

int eagle3_set_workspace(eagle3_ctx* ctx, void* dev, size_t bytes) {
  if (!ctx || !dev) return EAGLE3_E_NULL;
  if ((uintptr_t)dev & 255) return EAGLE3_E_STATE;
  // the longest prefill chunks that fit
  const int before = ctx->chunk_max, least = ctx->chunk_least();
  for (int chunk = ctx->chunk_full(); chunk >= least; chunk = chunk > 64 ? chunk - 64 : chunk > least ? least : 0) {
    ctx->size_for(chunk);
    if (ctx->ws_need > bytes) continue;
    ctx->ws = dev;
    ctx->ws_bytes = bytes;
    ctx->carve(dev);
    return EAGLE3_OK;
  }
  ctx->size_for(before);
  ctx->carve(ctx->ws);
  return EAGLE3_E_STATE;
}

int eagle3_set_weights(eagle3_ctx* ctx, const eagle3_target_weights* t, const eagle3_draft_weights* d) {
  if (!ctx) return EAGLE3_E_NULL;
  if (t) {
    if (!t->layers || !t->embed || !t->final_norm || !t->lm_head) return EAGLE3_E_NULL;
    for (int l = 0; l < ctx->cfg.n_layers; ++l) {
      const eagle3_layer_weights& w = t->layers[l];
      if (!w.wq || !w.wk || !w.wv || !w.wo || !w.w_gate || !w.w_up || !w.w_down || !w.norm_attn || !w.norm_mlp)
        return EAGLE3_E_NULL;
    }
    ctx->layers.assign(t->layers, t->layers + ctx->cfg.n_layers);
    ctx->tw = *t;
    ctx->tw.layers = ctx->layers.data();
    ctx->has_target = true;
  }
  if (d) {
    const eagle3_layer_weights& w = d->layer;
    if (!d->w_fc || !d->norm_embed || !d->norm_feat || !d->final_norm || !d->lm_head || !d->d2t || !w.wq || !w.wk ||
        !w.wv || !w.wo || !w.w_gate || !w.w_up || !w.w_down || !w.norm_mlp)
      return EAGLE3_E_NULL;
    ctx->dw = *d;
    ctx->has_draft = true;
  }
  return EAGLE3_OK;
}

int eagle3_profile_begin(eagle3_ctx* ctx) {
  if (!ctx) return EAGLE3_E_NULL;
  if (ctx->stamps.empty()) {
    ctx->stamps.resize(8192);
    for (auto& s : ctx->stamps) {
      CK(hipEventCreate(&s.a));
      CK(hipEventCreate(&s.b));
    }
  }
  ctx->stamps_used = 0;
  ctx->profiling = true;
  return EAGLE3_OK;
}

int eagle3_profile_read(eagle3_ctx* ctx, int kind, double* ms_total, int64_t* launches, double* weight_bytes) {
  if (!ctx || !ms_total || !launches || !weight_bytes) return EAGLE3_E_NULL;
  double ms = 0, bytes = 0;
  int64_t n = 0;
  for (size_t i = 0; i < ctx->stamps_used; ++i) {
    auto& s = ctx->stamps[i];
    if (s.kind != kind) continue;
    CK(hipEventSynchronize(s.b));
    float t = 0.f;
    CK(hipEventElapsedTime(&t, s.a, s.b));
    ms += t; bytes += s.bytes; ++n;
  }
  *ms_total = ms; *launches = n; *weight_bytes = bytes;
  return EAGLE3_OK;
}

int eagle3_profile_end(eagle3_ctx* ctx) {
  if (!ctx) return EAGLE3_E_NULL;
  ctx->profiling = false;
  ctx->stamps_used = 0;
  return EAGLE3_OK;
}

static int fuse_rows(eagle3_ctx* ctx, const float* low, const float* mid, const float* high, int M, float* g_out,
                     hipStream_t st);

int eagle3_fuse_features(eagle3_ctx* ctx, const float* low, const float* mid, const float* high, int32_t M,
                         float* g_out, eagle3_stream stream) {
  if (!ctx || !low || !mid || !high || !g_out) return EAGLE3_E_NULL;
  if (!ctx->ws || !ctx->has_draft) return EAGLE3_E_STATE;
  if (M < 1 || M > ctx->cfg.max_new) return EAGLE3_E_SHAPE;
  return fuse_rows(ctx, low, mid, high, M, g_out, (hipStream_t)stream);
}

static int fuse_rows(eagle3_ctx* ctx, const float* low, const float* mid, const float* high, int M, float* g_out,
                     hipStream_t st) {
  const int k = ctx->cfg.hidden;
  CK(launch_pack3(ctx->bf16, low, mid, high, M, k, ctx->act_k, st));
  GemmWeights W = {{ctx->dw.w_fc, nullptr, nullptr}, {k, 0, 0}, 1, 0};
  return ctx->project(ctx->act_k, W, M, k, 3 * k, GEMM_EPI_PARTIAL, nullptr, st, g_out);
}

// fp32: the operand of the product over N weight rows (pairs: see f32_norm_inside) that takes the RMSNorm of R rows of x: the rows
// themselves, with the gain in f, or the normed ones.
static int norm_operand(eagle3_ctx* ctx, float* x, const void* gain, int R, int N, int K, bool pairs, F32Fuse& f, const float** in,
                        hipStream_t st) {
  f.gain = (const float*)gain; f.eps = ctx->cfg.rms_eps;
  *in = x;
  if (!gain || f32_norm_inside(R, N, K, pairs)) return EAGLE3_OK;
  CK(launch_add_norm(false, x, nullptr, 0, R, K, gain, f.eps, ctx->act_k, nullptr, st));
  f.gain = nullptr;
  *in = (const float*)ctx->act_k;
  return EAGLE3_OK;
}

// q/k/v projection of R rows, rotated (cs, cs_step: their rotary tables), k and v in their cache slots.  in: the projection's operand, K wide; fp32 with a gain: the
// rows whose RMSNorm is that operand.
static int project_qkv(eagle3_ctx* ctx, const eagle3_layer_weights& w, void* in, const void* gain, int K, int R, const int32_t* slot,
                       const float* cs, int cs_step, void* kc, void* vc, hipStream_t st) {
  const eagle3_config& c = ctx->cfg;
  const int H = c.n_heads, Hkv = c.n_kv_heads, d = c.head_dim;
  GemmWeights Wqkv = {{w.wq, w.wk, w.wv}, {H * d, Hkv * d, Hkv * d}, 3, 0};
  if (!ctx->bf16) {
    F32Fuse f;
    const float* rows;
    TRY(norm_operand(ctx, (float*)in, gain, R, (H + 2 * Hkv) * d, K, true, f, &rows, st));
    f.cs = cs; f.cs_step = cs_step; f.slot = slot; f.kc = (float*)kc; f.vc = (float*)vc; f.H = H; f.Hkv = Hkv; f.d = d;
    CK(launch_gemm_f32(rows, Wqkv, R, (H + 2 * Hkv) * d, K, GEMM_EPI_ROPE, (float*)ctx->q, st, f));
    return EAGLE3_OK;
  }
  const int N = (H + 2 * Hkv) * d;
  if (wide_rope_fits(R, N, K, ctx->part_floats)) {
    const WideRope rope = {cs, cs_step, slot, H, Hkv, (bf16_t*)ctx->q, (bf16_t*)kc, (bf16_t*)vc};
    eagle3_ctx::Stamp* sp = ctx->stamp(2.0 * N * K, EAGLE3_GEMM_MANY_ROWS);
    CK(launch_gemm_wide_rope((const bf16_t*)in, Wqkv, R, N, K, rope, ctx->part_floats, st, sp ? sp->a : nullptr, sp ? sp->b : nullptr));
    return EAGLE3_OK;
  }
  int S = 1;
  TRY(ctx->project(in, Wqkv, R, (H + 2 * Hkv) * d, K, GEMM_EPI_PARTIAL, &S, st));
  CK(launch_rope_kv_write(ctx->part, S, R, H, Hkv, d, cs, cs_step, slot, ctx->q, kc, vc, st));
  return EAGLE3_OK;
}

static int project_head(eagle3_ctx* ctx, int R, const void* head, int V, float* out, hipStream_t st) {
  GemmWeights W = {{head, nullptr, nullptr}, {V, 0, 0}, 1, 0};
  return ctx->project(ctx->act_k, W, R, V, ctx->cfg.hidden, GEMM_EPI_PARTIAL, nullptr, st, out);
}

// RMSNorm and LM head of R rows, to which S partial sums in `part` are added first; copies: see launch_add_norm.
static int norm_head(eagle3_ctx* ctx, float* x, int S, int R, const void* gain, float* const copies[4], const void* head, int V, float* out,
                     hipStream_t st) {
  const int k = ctx->cfg.hidden;
  GemmWeights W = {{head, nullptr, nullptr}, {V, 0, 0}, 1, 0};
  if (!ctx->bf16) {
    F32Fuse f;
    const float* rows;
    TRY(norm_operand(ctx, x, gain, R, V, k, false, f, &rows, st));
    CK(launch_gemm_f32(rows, W, R, V, k, GEMM_EPI_PARTIAL, out, st, f));
    return EAGLE3_OK;
  }
  CK(launch_add_norm(true, x, S ? ctx->part : nullptr, S, R, k, gain, ctx->cfg.rms_eps, ctx->act_k, copies, st));
  return project_head(ctx, R, head, V, out, st);
}

// attention + output projection + MLP of one layer, shared by the target stack and the draft layer.
// On entry: q, and the cache rows of k and v, are written (project_qkv); x holds the residual rows.
// On exit: bf16: `part` holds S_down partial sums of the MLP output (to be added to x by the caller); fp32: x holds the layer's
// output, and so does each non-null copy; S_down = 0.
// R rows exist, B * rows_per_seq of them (and up to 63 more in a prefill chunk's last block) go through attention.
// prefill: the rows are R consecutive positions of one sequence.
// last_row: of the rows only the last one goes on behind its keys and values (its residual row stays where it is).
static int layer_tail(eagle3_ctx* ctx, const eagle3_layer_weights& w, int B, int rows_per_seq, int R, bool prefill, const uint32_t* mask,
                      const SeqInfo* seq, void* kc, void* vc, int max_len, float* const copies[4], int* S_down, hipStream_t st,
                      bool last_row = false) {
  const eagle3_config& c = ctx->cfg;
  const int k = c.hidden, H = c.n_heads, Hkv = c.n_kv_heads, d = c.head_dim, I = c.intermediate;
  const char* q = (const char*)ctx->q;
  float* x = ctx->x;
  if (last_row) {                                   // the block that row R - 1 is in, as a sequence of that row alone
    q += (size_t)(R - 1) * H * d * ctx->act_size;
    x += (size_t)(R - 1) * k;
    seq += (R - 1) / 64;
    mask += (size_t)(R - 1) * 4;
    B = rows_per_seq = R = 1;
  }
  if (!last_row && prefill && ctx->bf16 && prefill_attention_fits(R, H, Hkv, max_len)) {
    CK(launch_prefill_attention(q, kc, vc, seq, R, H, Hkv, d, ctx->act_attn, st));
  } else {
    int ns = 1;
    if (ctx->bf16) {
      ns = attention_pick_splits(B, rows_per_seq, H, Hkv, max_len);
      while (ns > 1 && attention_scratch_floats(B * rows_per_seq, H, d, ns) > ctx->attn_floats) --ns;
    }
    CK(launch_tree_attention(ctx->bf16, q, kc, vc, seq, mask, B, rows_per_seq, H, Hkv, d, max_len, ns,
                             ctx->attn_scratch, ctx->act_attn, st));
  }
  int S_o = 1;
  GemmWeights Wo = {{w.wo, nullptr, nullptr}, {k, 0, 0}, 1, 0};
  GemmWeights Wgu = {{w.w_gate, w.w_up, nullptr}, {I, I, 0}, 2, 1};
  GemmWeights Wd = {{w.w_down, nullptr, nullptr}, {k, 0, 0}, 1, 0};
  if (!ctx->bf16) {
    F32Fuse norm, out;
    const float* rows;
    for (int i = 0; copies && i < 4; ++i) out.copies[i] = copies[i];
    CK(launch_gemm_f32((const float*)ctx->act_attn, Wo, R, k, H * d, GEMM_EPI_RESIDUAL, x, st));
    TRY(norm_operand(ctx, x, w.norm_mlp, R, 2 * I, k, true, norm, &rows, st));
    CK(launch_gemm_f32(rows, Wgu, R, 2 * I, k, GEMM_EPI_SWIGLU, (float*)ctx->act_h, st, norm));
    CK(launch_gemm_f32((const float*)ctx->act_h, Wd, R, k, I, GEMM_EPI_RESIDUAL, x, st, out));
    *S_down = 0;
    return EAGLE3_OK;
  }
  TRY(ctx->project(ctx->act_attn, Wo, R, k, H * d, GEMM_EPI_PARTIAL, &S_o, st));
  CK(launch_add_norm(true, x, ctx->part, S_o, R, k, w.norm_mlp, c.rms_eps, ctx->act_k, nullptr, st));
  TRY(ctx->project(ctx->act_k, Wgu, R, 2 * I, k, GEMM_EPI_SWIGLU, nullptr, st));
  TRY(ctx->project(ctx->act_h, Wd, R, k, I, GEMM_EPI_PARTIAL, S_down, st));
  return EAGLE3_OK;
}

// Layers [l0, l1) of the target stack over R rows, from what `begin` says; attention sees them as B sequences of N rows.
// logits != nullptr: finish with the final norm and the
// LM head (requires l1 == n_layers).  norm_out: finish with the norm in front of layer l1.  x_out (optional) receives the residual stream after layer l1 - 1.
static int run_layers(eagle3_ctx* ctx, const BeginRows& begin, int B, int N, int R, bool prefill, const eagle3_kv* kv, int max_len, int l0, int l1,
                      float* x_out, float* logits, float* taps, float* dbg_hidden, hipStream_t st, bool norm_out = false) {
  const eagle3_config& c = ctx->cfg;
  const int k = c.hidden;
  const size_t Rk = (size_t)R * k;
  // what receives the residual stream in front of layer l, the output of layer l - 1
  struct Copies { float* p[4]; };
  auto copies_at = [&](int l) {
    Copies co = {};
    if (l > 0 && taps)
      for (int t = 0; t < 3; ++t)
        if (c.tap_layers[t] == l - 1) co.p[t] = taps + (size_t)t * Rk;
    if (dbg_hidden) co.p[3] = dbg_hidden + (size_t)l * Rk;
    if (l == l1 && x_out) co.p[3] = x_out;
    return co;
  };
  int S_prev = 0;                                   // bf16: partial sums of the previous layer's MLP still to be added
  for (int l = l0; l <= l1; ++l) {
    // bf16: x becomes the output of layer l-1 here, is copied, and normed for what follows.  fp32: x is complete, layer l-1 has
    // made the copies, and the norm comes with the product that follows (norm_operand).  l0: x is formed here.
    const Copies co = copies_at(l);
    const bool head = l == c.n_layers && l == l1 && logits, norm = head || l < l1 || norm_out;
    const void* gain = head ? ctx->tw.final_norm : norm ? ctx->layers[l].norm_attn : nullptr;
    if (l == l0)
      CK(launch_begin_rows(ctx->bf16, begin, ctx->x, R, k, ctx->bf16 ? gain : nullptr, c.rms_eps, ctx->act_k, co.p, st));
    else if (ctx->bf16)
      CK(launch_add_norm(true, ctx->x, ctx->part, S_prev, R, k, gain, c.rms_eps, norm ? ctx->act_k : nullptr, co.p, st));
    if (head) return ctx->bf16 ? project_head(ctx, R, ctx->tw.lm_head, c.vocab, logits, st)
                               : norm_head(ctx, ctx->x, 0, R, gain, nullptr, ctx->tw.lm_head, c.vocab, logits, st);
    if (l == l1) break;
    const eagle3_layer_weights& w = ctx->layers[l];
    TRY(project_qkv(ctx, w, ctx->bf16 ? ctx->act_k : ctx->x, w.norm_attn, k, R, ctx->slot, ctx->cs, c.head_dim, kv->k[l], kv->v[l], st));
    const Copies next = copies_at(l + 1);
    TRY(layer_tail(ctx, w, B, N, R, prefill, ctx->mask, ctx->seq, kv->k[l], kv->v[l], max_len, next.p, &S_prev, st));
  }
  return EAGLE3_OK;
}

// The same over the node rows of B trees, from the token embeddings (x_in == nullptr, requires l0 == 0) or from x_in.
static int verify_layers(eagle3_ctx* ctx, int B, int N, const int32_t* tree_tok, const int32_t* parent,
                         const eagle3_kv* kv, const float* x_in, int l0, int l1, float* x_out, float* logits, float* taps,
                         float* dbg_hidden, hipStream_t st) {
  const eagle3_config& c = ctx->cfg;
  const int R = B * N;
  // by the runtime: x_in may lie in memory that no kernel of this GPU can read (another GPU's, without peer access)
  if (x_in) CK(hipMemcpyAsync(ctx->x, x_in, (size_t)R * c.hidden * sizeof(float), hipMemcpyDeviceToDevice, st));
  const BeginRows begin = {x_in ? nullptr : ctx->tw.embed, tree_tok, c.vocab, parent, B, N, kv->kv_indptr, kv->prefix_len, (int)c.head_dim, c.rope_theta,
                           ctx->slot, ctx->mask, ctx->cs, ctx->seq};
  return run_layers(ctx, begin, B, N, R, false, kv, kv->max_prefix_len + N, l0, l1, x_out, logits, taps, dbg_hidden, st);
}

static int check_verify_args(eagle3_ctx* ctx, int B, int N, const int32_t* tree_tok, const int32_t* parent,
                             const eagle3_kv* kv, int l0, int l1) {
  if (!ctx || !tree_tok || !parent || !kv) return EAGLE3_E_NULL;
  if (!kv->k || !kv->v || !kv->kv_indptr || !kv->prefix_len) return EAGLE3_E_NULL;
  if (!ctx->ws || !ctx->has_target) return EAGLE3_E_STATE;
  const eagle3_config& c = ctx->cfg;
  if (B < 1 || B > c.max_batch || N < 1 || N > c.max_nodes || kv->max_prefix_len < 0) return EAGLE3_E_SHAPE;
  if (l0 < 0 || l1 < l0 || l1 > c.n_layers) return EAGLE3_E_SHAPE;
  for (int l = l0; l < l1; ++l)
    if (!kv->k[l] || !kv->v[l]) return EAGLE3_E_NULL;
  return EAGLE3_OK;
}

int eagle3_tree_verify(eagle3_ctx* ctx, int32_t B, int32_t N, const int32_t* tree_tok, const int32_t* parent,
                       const eagle3_kv* kv, float* logits, float* taps, float* dbg_hidden, eagle3_stream stream) {
  if (!logits || !taps) return EAGLE3_E_NULL;
  TRY(check_verify_args(ctx, B, N, tree_tok, parent, kv, 0, ctx ? ctx->cfg.n_layers : 0));
  return verify_layers(ctx, B, N, tree_tok, parent, kv, nullptr, 0, ctx->cfg.n_layers, nullptr, logits, taps, dbg_hidden,
                       (hipStream_t)stream);
}

int eagle3_tree_verify_layers(eagle3_ctx* ctx, int32_t B, int32_t N, const int32_t* tree_tok, const int32_t* parent,
                              const eagle3_kv* kv, const float* x_in, int32_t layer_begin, int32_t layer_end,
                              float* x_out, float* logits, eagle3_stream stream) {
  TRY(check_verify_args(ctx, B, N, tree_tok, parent, kv, layer_begin, layer_end));
  if (!x_in && layer_begin != 0) return EAGLE3_E_NULL;
  if (!x_out && !logits) return EAGLE3_E_NULL;
  if (logits && layer_end != ctx->cfg.n_layers) return EAGLE3_E_SHAPE;
  return verify_layers(ctx, B, N, tree_tok, parent, kv, x_in, layer_begin, layer_end, x_out, logits, nullptr, nullptr,
                       (hipStream_t)stream);
}

int eagle3_draft_expand(eagle3_ctx* ctx, const float* g_new, const int32_t* tok_new, int32_t n_new,
                        const eagle3_kv* dkv, int32_t depth, int32_t topk, int32_t n_nodes, int32_t* tree_tok,
                        int32_t* parent, int32_t* node_depth, float* cum_logprob, const eagle3_draft_debug* dbg,
                        eagle3_stream stream) {
  if (!ctx || !g_new || !tok_new || !dkv || !tree_tok || !parent || !node_depth || !cum_logprob) return EAGLE3_E_NULL;
  if (!dkv->k || !dkv->v || !dkv->k[0] || !dkv->v[0] || !dkv->kv_indptr || !dkv->prefix_len) return EAGLE3_E_NULL;
  if (!ctx->ws || !ctx->has_draft || !ctx->has_target) return EAGLE3_E_STATE;    // the target's embedding table is used
  const eagle3_config& c = ctx->cfg;
  const int pool = 1 + topk + (depth - 1) * topk * topk;
  if (n_new < 1 || n_new > c.max_new || depth < 1 || depth > c.max_depth || topk < 1 || topk > c.max_topk ||
      n_nodes < 2 || n_nodes > c.max_nodes || n_nodes > pool || dkv->max_prefix_len < 0)
    return EAGLE3_E_SHAPE;
  hipStream_t st = (hipStream_t)stream;
  const int k = c.hidden, H = c.n_heads, Hkv = c.n_kv_heads, d = c.head_dim, Vd = c.draft_vocab, K = topk;
  const eagle3_layer_weights& w = ctx->dw.layer;
  const DraftState& ds = ctx->ds;
  void* kc = dkv->k[0];
  void* vc = dkv->v[0];

  const DraftInputArgs in = ctx->draft_input_args();
  // the rotary tables of all forwards at once, or, in the smallest workspaces, one after the other
  const bool all_tables = n_new + depth - 1 <= ctx->Rall;
  CK(launch_draft_first(ctx->bf16, in, tok_new, g_new, dkv->kv_indptr, dkv->prefix_len, n_new, all_tables ? depth : 1, ctx->slot, ctx->mask,
                        ctx->seq, st));
  for (int level = 1; level <= depth; ++level) {
    const int M = level == 1 ? n_new : K;
    const int a_row0 = level == 1 ? 0 : n_new + (level - 2) * K;
    const bool first = level == 1;
    const int max_len = dkv->max_prefix_len + n_new + (level - 1) * K;
    if (!first && !all_tables) CK(launch_rope_table(ctx->cs, dkv->prefix_len, n_new + level - 2, d, c.rope_theta, st));
    TRY(project_qkv(ctx, w, ctx->act_k, nullptr, 2 * k, M, first ? ctx->slot : ds.row_slot,
                    first || !all_tables ? ctx->cs : ctx->cs + (size_t)(n_new + level - 2) * d, first ? d : 0, kc, vc, st));
    // a = y1 + MLP(...): keep it for the children, and norm it for the LM head
    float* copies[4] = {ctx->a_buf + (size_t)a_row0 * k, nullptr, nullptr, nullptr};
    int S_down = 1;
    TRY(layer_tail(ctx, w, 1, M, M, false, first ? ctx->mask : ds.row_mask[level & 1], first ? ctx->seq : ds.seq, kc, vc, max_len, copies, &S_down, st));
    TRY(norm_head(ctx, ctx->x, S_down, M, ctx->dw.final_norm, copies, ctx->dw.lm_head, Vd, ctx->z, st));
    const DraftLogits zl = {ctx->z, first ? n_new - 1 : 0, Vd, ctx->topk_scratch};
    if (level < depth)
      CK(launch_draft_level(ctx->bf16, ds, zl, ctx->dw.d2t, dkv->kv_indptr, dkv->prefix_len, level, K, n_new, in, ctx->a_buf, st));
    else
      CK(launch_draft_finish(ds, zl, ctx->dw.d2t, tok_new, n_new, depth, K, n_nodes, tree_tok, parent, node_depth, cum_logprob,
                             dbg ? dbg->chosen : nullptr, st));
  }
  if (dbg) {
    const size_t pb = (size_t)pool * 4;
    if (dbg->pool_tok) CK(hipMemcpyAsync(dbg->pool_tok, ds.pool_tok, pb, hipMemcpyDeviceToDevice, st));
    if (dbg->pool_parent) CK(hipMemcpyAsync(dbg->pool_parent, ds.pool_parent, pb, hipMemcpyDeviceToDevice, st));
    if (dbg->pool_score) CK(hipMemcpyAsync(dbg->pool_score, ds.pool_score, pb, hipMemcpyDeviceToDevice, st));
    if (dbg->frontier && depth > 1)
      CK(hipMemcpyAsync(dbg->frontier, ds.frontier, (size_t)(depth - 1) * K * 4, hipMemcpyDeviceToDevice, st));
  }
  return EAGLE3_OK;
}

int eagle3_accept(eagle3_ctx* ctx, int32_t B, int32_t N, const float* logits, const int32_t* tree_tok,
                  const int32_t* parent, float temperature, const float* uniforms, int32_t* accept_len, int32_t* path,
                  int32_t* bonus_tok, eagle3_stream stream) {
  if (!ctx || !logits || !tree_tok || !parent || !accept_len || !path || !bonus_tok) return EAGLE3_E_NULL;
  if (temperature > 0.f && !uniforms) return EAGLE3_E_NULL;
  if (!ctx->ws) return EAGLE3_E_STATE;
  if (B < 1 || B > ctx->cfg.max_batch || N < 1 || N > ctx->cfg.max_nodes || !(temperature >= 0.f)) return EAGLE3_E_SHAPE;
  CK(launch_accept(logits, tree_tok, parent, B, N, ctx->cfg.vocab, temperature, uniforms, ctx->accept_stats, accept_len,
                   path, bonus_tok, (hipStream_t)stream));
  return EAGLE3_OK;
}

int eagle3_draft_chain(eagle3_ctx* ctx, int32_t B, const float* g_new, const int32_t* tok_new, const int32_t* n_new,
                       int32_t rows1, const eagle3_kv* dkv, int32_t length, int32_t* chain_tok, float* chain_logp,
                       eagle3_stream stream) {
  if (!ctx || !g_new || !tok_new || !n_new || !dkv || !chain_tok || !chain_logp) return EAGLE3_E_NULL;
  if (!dkv->k || !dkv->v || !dkv->k[0] || !dkv->v[0] || !dkv->kv_indptr || !dkv->prefix_len) return EAGLE3_E_NULL;
  if (!ctx->ws || !ctx->has_draft || !ctx->has_target) return EAGLE3_E_STATE;
  const eagle3_config& c = ctx->cfg;
  if (B < 1 || B > c.max_batch || rows1 < 1 || rows1 > ctx->rows1_max || length < 1 || length > c.max_depth ||
      dkv->max_prefix_len < 0)
    return EAGLE3_E_SHAPE;
  hipStream_t st = (hipStream_t)stream;
  const int k = c.hidden, H = c.n_heads, Hkv = c.n_kv_heads, d = c.head_dim, Vd = c.draft_vocab;
  const eagle3_layer_weights& w = ctx->dw.layer;
  const ChainState& cs = ctx->cs_chain;
  void* kc = dkv->k[0];
  void* vc = dkv->v[0];
  const DraftInputArgs in = ctx->draft_input_args();
  CK(launch_chain_prep1(dkv->kv_indptr, dkv->prefix_len, B, rows1, ctx->pos1, ctx->slot, ctx->mask, ctx->seq, st));
  CK(launch_draft_input(ctx->bf16, in, tok_new, g_new, ctx->pos1, B * rows1, st));
  for (int level = 1; level <= length; ++level) {
    const int rps = level == 1 ? rows1 : 1, M = B * rps;
    const bool first = level == 1;
    const int32_t* slot = first ? ctx->slot : cs.row_slot;
    const uint32_t* mask = first ? ctx->mask : cs.row_mask;
    const SeqInfo* seq = first ? ctx->seq : cs.seq;
    const int max_len = dkv->max_prefix_len + rows1 + level;
    TRY(project_qkv(ctx, w, ctx->act_k, nullptr, 2 * k, M, slot, ctx->cs, d, kc, vc, st));
    const bool gather = level == 1 && rows1 > 1;
    float* copies[4] = {gather ? nullptr : ctx->a_buf, nullptr, nullptr, nullptr};
    int S_down = 1;
    TRY(layer_tail(ctx, w, B, rps, M, false, mask, seq, kc, vc, max_len, copies, &S_down, st));
    if (gather) {
      // a = y1 + MLP(...) for every row, then the row of each sequence's last real position moves to row b
      if (ctx->bf16) CK(launch_add_norm(true, ctx->x, ctx->part, S_down, M, k, nullptr, c.rms_eps, nullptr, nullptr, st));
      CK(launch_chain_gather(ctx->x, n_new, B, rows1, k, ctx->a_buf, st));
      S_down = 0;
    }
    TRY(norm_head(ctx, gather ? ctx->a_buf : ctx->x, S_down, B, ctx->dw.final_norm, copies, ctx->dw.lm_head, Vd, ctx->z, st));
    CK(launch_chain_level(ctx->bf16, cs, {ctx->z, 0, Vd, ctx->topk_scratch}, ctx->dw.d2t, dkv->kv_indptr, dkv->prefix_len, n_new, tok_new, B,
                          rows1, level, length, chain_tok, chain_logp, in, ctx->a_buf, st));
  }
  return EAGLE3_OK;
}

int eagle3_prefill(eagle3_ctx* ctx, const int32_t* tokens, int32_t T, const eagle3_kv* kv, const eagle3_kv* dkv,
                   float* g_last, float* logits_last, eagle3_stream stream) {
  if (!ctx || !tokens || !kv || !dkv || !g_last || !logits_last) return EAGLE3_E_NULL;
  if (!kv->k || !kv->v || !kv->kv_indptr || !kv->prefix_len) return EAGLE3_E_NULL;
  if (!dkv->k || !dkv->v || !dkv->k[0] || !dkv->v[0] || !dkv->kv_indptr || !dkv->prefix_len) return EAGLE3_E_NULL;
  if (!ctx->ws || !ctx->has_target || !ctx->has_draft) return EAGLE3_E_STATE;
  const eagle3_config& c = ctx->cfg;
  if (T < 1 || kv->max_prefix_len < 0 || dkv->max_prefix_len < 0) return EAGLE3_E_SHAPE;
  for (int l = 0; l < c.n_layers; ++l)
    if (!kv->k[l] || !kv->v[l]) return EAGLE3_E_NULL;
  hipStream_t st = (hipStream_t)stream;
  const int k = c.hidden, H = c.n_heads, Hkv = c.n_kv_heads, d = c.head_dim;
  const eagle3_layer_weights& w = ctx->dw.layer;
  // Behind the last layer only the last position is read, unless that layer's output is one of the three features: the others need
  // no more of it than their keys and values.  8B width, 32 layers: 2048 tokens 27.8 -> 27.2 ms.
  bool tail_row = true;
  for (int t = 0; t < 3; ++t) tail_row = tail_row && c.tap_layers[t] != c.n_layers - 1;
  // chunks of equal length (whole 64-row blocks): a short last chunk would stream all weights for a few rows
  const int n_chunks = (T + ctx->chunk_max - 1) / ctx->chunk_max;
  const int C = std::min(ctx->chunk_max, ((T + n_chunks - 1) / n_chunks + 63) / 64 * 64);
  for (int c0 = 0; c0 < T; c0 += C) {
    const int n = std::min(C, T - c0), blocks = (n + 63) / 64;
    const bool last = c0 + n == T;
    // target: the chunk on top of everything cached so far; features of every position recorded
    const size_t nk = (size_t)n * k;
    const BeginRows begin = {ctx->tw.embed, tokens + c0, c.vocab, nullptr, 1, 0, kv->kv_indptr, kv->prefix_len, d, c.rope_theta,
                             ctx->slot, ctx->mask, ctx->cs, ctx->seq};
    const int max_len = kv->max_prefix_len + c0 + n, L = c.n_layers;
    int S_tail = 0;
    if (tail_row) {
      TRY(run_layers(ctx, begin, blocks, blocks == 1 ? n : 64, n, true, kv, max_len, 0, L - 1, nullptr, nullptr, ctx->chunk_taps, nullptr, st, true));
      const eagle3_layer_weights& wl = ctx->layers[L - 1];
      TRY(project_qkv(ctx, wl, ctx->bf16 ? ctx->act_k : ctx->x, wl.norm_attn, k, n, ctx->slot, ctx->cs, d, kv->k[L - 1], kv->v[L - 1], st));
      if (last) TRY(layer_tail(ctx, wl, 1, 1, n, true, ctx->mask, ctx->seq, kv->k[L - 1], kv->v[L - 1], max_len, nullptr, &S_tail, st, true));
    } else {
      TRY(run_layers(ctx, begin, blocks, blocks == 1 ? n : 64, n, true, kv, max_len, 0, L, nullptr, nullptr, ctx->chunk_taps, nullptr, st));
    }
    if (last) {                                       // next-token logits of the last position only
      TRY(norm_head(ctx, ctx->x + (size_t)(n - 1) * k, S_tail, 1, ctx->tw.final_norm, nullptr, ctx->tw.lm_head, c.vocab, logits_last, st));
    }
    // fused features of the chunk's positions; the draft cache rows of those whose next token is known
    TRY(fuse_rows(ctx, ctx->chunk_taps, ctx->chunk_taps + nk, ctx->chunk_taps + 2 * nk, n, ctx->chunk_g, st));
    // by the runtime, as x_in comes: g_last may lie where no kernel of this GPU can write
    if (last) CK(hipMemcpyAsync(g_last, ctx->chunk_g + (size_t)(n - 1) * k, (size_t)k * sizeof(float), hipMemcpyDeviceToDevice, st));
    const int m = last ? n - 1 : n;
    if (m > 0) {
      CK(launch_draft_first(ctx->bf16, ctx->draft_input_args(), tokens + c0 + 1, ctx->chunk_g, dkv->kv_indptr, dkv->prefix_len, m, 1, ctx->slot,
                            nullptr, nullptr, st));
      TRY(project_qkv(ctx, w, ctx->act_k, nullptr, 2 * k, m, ctx->slot, ctx->cs, d, dkv->k[0], dkv->v[0], st));
    }
    CK(launch_end_prefill((int32_t*)kv->prefix_len, n, (int32_t*)dkv->prefix_len, m, st));
  }
  return EAGLE3_OK;
}

int eagle3_ttt_attention(int32_t dtype, int32_t T, int32_t n_heads, int32_t n_kv_heads, int32_t head_dim, int32_t step,
                         const void* q, const void* k_steps, const void* v_steps, float* out, eagle3_stream stream) {
  if (!q || !k_steps || !v_steps || !out) return EAGLE3_E_NULL;
  if (dtype != EAGLE3_BF16 && dtype != EAGLE3_FP32) return EAGLE3_E_SHAPE;
  if (T < 1 || n_heads < 1 || n_kv_heads < 1 || n_heads % n_kv_heads || step < 0 || head_dim < 1) return EAGLE3_E_SHAPE;
  if (dtype == EAGLE3_BF16 ? head_dim != 128 : (head_dim > 1024 || (size_t)(T + step) * 4 > 60 * 1024)) return EAGLE3_E_SHAPE;
  CK(launch_ttt_attention(dtype == EAGLE3_BF16, q, k_steps, v_steps, T, n_heads, n_kv_heads, head_dim, step, out,
                          (hipStream_t)stream));
  return EAGLE3_OK;
}

int eagle3_commit(eagle3_ctx* ctx, int32_t B, int32_t N, const int32_t* tree_tok, const int32_t* path,
                  const int32_t* accept_len, const int32_t* bonus_tok, const eagle3_kv* kv, int32_t* prefix_len,
                  const float* taps, int32_t rows, float* taps_new, int32_t* tok_new, int32_t* n_new,
                  int32_t* draft_prefix_len, int32_t draft_rows, eagle3_stream stream) {
  if (!ctx || !tree_tok || !path || !accept_len || !bonus_tok || !kv || !prefix_len || !taps || !tok_new || !n_new)
    return EAGLE3_E_NULL;
  if (!kv->k || !kv->v || !kv->kv_indptr) return EAGLE3_E_NULL;
  const eagle3_config& c = ctx->cfg;
  if (B < 1 || B > c.max_batch || N < 1 || N > c.max_nodes || rows < 1 || draft_rows < 0) return EAGLE3_E_SHAPE;
  for (int l = 0; l < c.n_layers; ++l)
    if (!kv->k[l] || !kv->v[l]) return EAGLE3_E_NULL;
  CK(launch_commit(kv->k, kv->v, c.n_layers, kv->kv_indptr, prefix_len, tree_tok, path, accept_len, bonus_tok, taps, B, N,
                   c.hidden, (int)(c.n_kv_heads * c.head_dim * ctx->act_size), rows, taps_new, tok_new, n_new,
                   draft_prefix_len, draft_rows, (hipStream_t)stream));
  return EAGLE3_OK;
}

}  // extern "C"
