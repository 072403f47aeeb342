// Row-wise kernels between the GEMMs: embedding gather, residual add + RMSNorm, rotary embedding and
// cache write, tree bookkeeping, feature packing.  All are tiny next to the weight
// streams; they exist to hand the next GEMM its operand in the layout it reads.
#include <algorithm>

#include "common.hpp"
#include "draft_row.hpp"
#include "kernels.hpp"

namespace {

// One pass; VEC: four consecutive columns per thread, where k is a multiple of 4 and the table is 16-byte aligned.
template <typename TW, bool VEC>
__global__ __launch_bounds__(256) void embed_rows_kernel(const TW* __restrict__ embed, const int32_t* __restrict__ tok,
                                                        int k, int vocab, float* __restrict__ x) {
  const int r = blockIdx.x, c = (VEC ? 4 : 1) * (blockIdx.y * 256 + threadIdx.x);
  if (c >= k) return;
  const size_t t = (size_t)min(max(tok[r], 0), vocab - 1) * k + c;
  if constexpr (VEC) *(float4*)(x + (size_t)r * k + c) = load4_f32(embed, t);
  else x[(size_t)r * k + c] = load_f32(embed, t);
}

struct CopyOut { float* p[4]; };

// One workgroup per row, four consecutive columns per thread (two such groups when k > 4096): the row stays
// in registers between the partial-sum reduction and the normalised store.
template <bool BF16>
__global__ __launch_bounds__(1024) void add_norm_kernel(float* __restrict__ x, const float* __restrict__ partial, int S,
                                                       int R, int k, const typename Act<BF16>::type* __restrict__ gain,
                                                       float eps, typename Act<BF16>::type* __restrict__ act, CopyOut co) {
  __shared__ float red[17];
  const int r = row_of_workgroup<BF16>(blockIdx.x), nvec = k >> 2, bd = blockDim.x;
  if (r >= R) return;
  constexpr int VPT = 2;
  float4 val[VPT];
  float ss = 0.f;
#pragma unroll
  for (int j = 0; j < VPT; ++j) {
    const int v = threadIdx.x + j * bd;
    if (v < nvec) {
      float4 a = *(const float4*)(x + (size_t)r * k + 4 * v);
      // four partial sums per round, all requested before the first is added (one memory round trip per round
      // instead of one per partial sum); the order of the additions stays s = 0, 1, 2, ...
      for (int s0 = 0; s0 < S; s0 += 4) {
        float4 p[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = *(const float4*)(partial + ((size_t)min(s0 + i, S - 1) * R + r) * k + 4 * v);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (s0 + i < S) { a.x += p[i].x; a.y += p[i].y; a.z += p[i].z; a.w += p[i].w; }
      }
      *(float4*)(x + (size_t)r * k + 4 * v) = a;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (co.p[i]) *(float4*)(co.p[i] + (size_t)r * k + 4 * v) = a;
      ss += a.x * a.x + a.y * a.y + a.z * a.z + a.w * a.w;
      val[j] = a;
    }
  }
  float4 g[VPT];                                      // requested before the reduction, used after it
  if (act != nullptr) {
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
      const int v = threadIdx.x + j * bd;
      if (v < nvec) g[j] = load4_f32(gain, 4 * v);
    }
  }
  ss = block_sum(ss, red);
  if (act == nullptr) return;
  const float inv = 1.0f / sqrtf(ss / (float)k + eps);
#pragma unroll
  for (int j = 0; j < VPT; ++j) {
    const int v = threadIdx.x + j * bd;
    if (v < nvec)
      Act<BF16>::store4(act, r, 4 * v, k, val[j].x * inv * g[j].x, val[j].y * inv * g[j].y, val[j].z * inv * g[j].z,
                        val[j].w * inv * g[j].w);
  }
}

__global__ __launch_bounds__(256) void tree_prep_kernel(const int32_t* __restrict__ parent,
                                                       const int32_t* __restrict__ kv_indptr,
                                                       const int32_t* __restrict__ prefix_len, int N, int d, float theta,
                                                       int32_t* __restrict__ depth, uint32_t* __restrict__ mask,
                                                       int32_t* __restrict__ slot, float* __restrict__ cs,
                                                       SeqInfo* __restrict__ seq) {
  // Workgroup (b, y): every y walks sequence b's tree (parents staged in LDS: one memory round trip, then the walks
  // stay on chip) and fills its share of the rotary table, whose sines and cosines are the bulk of the work; y = 0
  // also writes the masks, depths, slots and the sequence record.
  __shared__ int sdepth[64], spar[64];
  __shared__ int rank;
  const int b = blockIdx.x, y = blockIdx.y, i = threadIdx.x, B = gridDim.x;
  const int P = prefix_len[b], base = kv_indptr[b];
  if (i < N) spar[i] = parent[b * N + i];
  if (i == 0) rank = 0;
  __syncthreads();
  if (y == 0) {
    // rank of this sequence by prefix length, longest first (ties: smaller index first): attention hands out its
    // workgroups in that order, so that the long sequences start first and the short ones fill the tail
    int longer = 0;
    for (int o = i; o < B; o += 256) {
      const int Po = prefix_len[o];
      longer += (Po > P || (Po == P && o < b)) ? 1 : 0;
    }
    if (longer) atomicAdd(&rank, longer);
  }
  if (i < N) {
    uint32_t m[4] = {0u, 0u, 0u, 0u};
    int cur = i, dep = 0;
    for (int it = 0; it < N; ++it) {                     // bounded walk: malformed parents cannot loop
      m[cur >> 5] |= 1u << (cur & 31);
      const int p = spar[cur];
      if (p < 0 || p >= cur) break;
      cur = p;
      ++dep;
    }
    sdepth[i] = dep;
    if (y == 0) {
      const int r = b * N + i;
      depth[r] = dep;
      slot[r] = base + P + i;
#pragma unroll
      for (int w = 0; w < 4; ++w) mask[r * 4 + w] = m[w];
    }
  }
  __syncthreads();
  if (y == 0 && i == 0) {
    seq[rank].order = b;
    seq[b].kv_base = base; seq[b].n_prefix = P; seq[b].n_tail = N;
  }
  const int half = d / 2;
  for (int e = y * 256 + i; e < N * half; e += 256 * gridDim.y) {
    const int row = e / half, f = e % half;
    rope_entry(cs, b * N + row, f, d, P + sdepth[row], theta);
  }
}

// One workgroup per row; a thread handles four consecutive rotary pairs (i..i+3, i+d/2..i+d/2+3) of one head.  (fp32: gemm_f32.hip.)
__global__ __launch_bounds__(1024) void rope_kv_write_kernel(const float* __restrict__ qkv, int S, int R, int H, int Hkv,
                                                            int d, const float* __restrict__ cs, int cs_step,
                                                            const int32_t* __restrict__ slot, bf16_t* __restrict__ q,
                                                            bf16_t* __restrict__ kc, bf16_t* __restrict__ vc) {
  const int r = blockIdx.x, half = d / 2, NT = (H + 2 * Hkv) * d, q4 = half / 4;
  const size_t sl = (size_t)slot[r];
  for (int e = threadIdx.x; e < (H + 2 * Hkv) * q4; e += blockDim.x) {
    const int h = e / q4, i = (e % q4) * 4;
    float4 x1 = make_float4(0.f, 0.f, 0.f, 0.f), x2 = x1;
    for (int s0 = 0; s0 < S; s0 += 4) {                 // four partial sums per memory round trip, added in order
      float4 a[4], b[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float* row = qkv + ((size_t)min(s0 + j, S - 1) * R + r) * NT + h * d;
        a[j] = *(const float4*)(row + i);
        b[j] = *(const float4*)(row + i + half);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (s0 + j < S) {
          x1.x += a[j].x; x1.y += a[j].y; x1.z += a[j].z; x1.w += a[j].w;
          x2.x += b[j].x; x2.y += b[j].y; x2.z += b[j].z; x2.w += b[j].w;
        }
    }
    bf16_t* dst;
    if (h < H + Hkv) {
      const float4 c = *(const float4*)(cs + (size_t)r * cs_step + i), sn = *(const float4*)(cs + (size_t)r * cs_step + half + i);
      const float4 o1 = make_float4(x1.x * c.x - x2.x * sn.x, x1.y * c.y - x2.y * sn.y, x1.z * c.z - x2.z * sn.z,
                                    x1.w * c.w - x2.w * sn.w);
      const float4 o2 = make_float4(x2.x * c.x + x1.x * sn.x, x2.y * c.y + x1.y * sn.y, x2.z * c.z + x1.z * sn.z,
                                    x2.w * c.w + x1.w * sn.w);
      x1 = o1; x2 = o2;
      dst = h < H ? q + ((size_t)r * H + h) * d : kc + (sl * Hkv + (h - H)) * d;
    } else {
      dst = vc + (sl * Hkv + (h - H - Hkv)) * d;
    }
    store4_plain(dst, i, x1.x, x1.y, x1.z, x1.w);
    store4_plain(dst, i + half, x2.x, x2.y, x2.z, x2.w);
  }
}

// The fusion's input row [a; b; c], one pass.  VEC: four consecutive columns per thread, where k is a multiple of 4 and the
// three inputs, which are the caller's, are 16-byte aligned (64 rows of 3 x 4096: 5.4 us; 10.8 us with one column per thread, whose
// bf16 stores are 2 bytes each).
template <bool BF16, bool VEC>
__global__ __launch_bounds__(256) void pack3_kernel(const float* __restrict__ a, const float* __restrict__ b,
                                                   const float* __restrict__ c, int M, int k,
                                                   typename Act<BF16>::type* __restrict__ act) {
  const int r = row_of_workgroup<BF16>(blockIdx.x), col = (VEC ? 4 : 1) * (blockIdx.y * 256 + threadIdx.x);
  if (r >= M || col >= 3 * k) return;
  const int part = col / k;
  const float* src = (part == 0 ? a : part == 1 ? b : c) + (size_t)r * k + col - part * k;
  if constexpr (VEC) {
    const float4 v = *(const float4*)src;
    Act<BF16>::store4(act, r, col, 3 * k, v.x, v.y, v.z, v.w);
  } else {
    Act<BF16>::store(act, r, col, 3 * k, *src);
  }
}

__global__ __launch_bounds__(256) void reduce_partials_kernel(const float* __restrict__ partial, int S, size_t MN,
                                                             float* __restrict__ out) {
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < MN; e += (size_t)gridDim.x * 256) {
    float v = 0.f;
    for (int s = 0; s < S; ++s) v += partial[(size_t)s * MN + e];
    out[e] = v;
  }
}

template <bool BF16, int VPT>
__global__ __launch_bounds__(1024) void draft_input_kernel(DraftInput<BF16> p, const int32_t* __restrict__ tok, const float* __restrict__ feat,
                                                          const int32_t* __restrict__ pos, int M) {
  __shared__ RowSums sums;
  const int r = row_of_workgroup<BF16>(blockIdx.x);
  if (r >= M) return;
  DraftGains<BF16, VPT> gains;
  load_gains(p, gains);
  draft_input_row(p, r, tok[r], feat + (size_t)r * p.k, gains, sums);
  // the row's rotary table, for the q/k rotation that follows the projection
  for (int i = threadIdx.x; i < p.head_dim / 2; i += blockDim.x) rope_entry(p.cs, r, i, p.head_dim, pos[r], p.theta);
}

// Draft forward 1 of a tree: n_new rows behind the context, causal among themselves; their bookkeeping comes with their input
// (a launch of its own cost 4.7 us).  Further workgroups form the rotary tables of the later forwards, whose rows share one position each.
template <bool BF16, int VPT>
__global__ __launch_bounds__(1024) void draft_first_kernel(DraftInput<BF16> p, const int32_t* __restrict__ tok, const float* __restrict__ feat,
                                                          const int32_t* __restrict__ kv_indptr, const int32_t* __restrict__ prefix_len,
                                                          int n_new, int depth, int32_t* __restrict__ slot, uint32_t* __restrict__ mask,
                                                          SeqInfo* __restrict__ seq) {
  __shared__ RowSums sums;
  const int r = row_of_workgroup<BF16>(blockIdx.x), tid = threadIdx.x;
  if (r >= n_new + depth - 1) return;
  const int P = prefix_len[0], base = kv_indptr[0];
  if (r < n_new) {
    if (tid < 4) {
      const int lo = 32 * tid;
      mask[r * 4 + tid] = r < lo ? 0u : (r - lo >= 31 ? 0xFFFFFFFFu : ((2u << (r - lo)) - 1u));     // bits 0..r
    }
    if (tid == 0) {
      slot[r] = base + P + r;
      if (r == 0) { seq[0].kv_base = base; seq[0].n_prefix = P; seq[0].n_tail = n_new; seq[0].order = 0; }
    }
    DraftGains<BF16, VPT> gains;
    load_gains(p, gains);
    draft_input_row(p, r, tok[r], feat + (size_t)r * p.k, gains, sums);
  }
  for (int i = tid; i < p.head_dim / 2; i += blockDim.x) rope_entry(p.cs, r, i, p.head_dim, P + r, p.theta);
}

// Rows of a prefill chunk, four per workgroup: row r continues the sequence at position P + r.  For attention the chunk is
// cut into blocks of 64 rows: block b sees the context and every earlier block unconditionally (n_prefix = P + 64 b) and its
// own rows causally through the row masks, so the tree kernels run a chunk of any length as a batch of "sequences" that
// share one cache.  The last block has the most keys, so it is handed out first.
__global__ __launch_bounds__(256) void prefill_prep_kernel(const int32_t* __restrict__ kv_indptr,
                                                          const int32_t* __restrict__ prefix_len, int n, int d, float theta,
                                                          int32_t* __restrict__ pos, int32_t* __restrict__ slot,
                                                          uint32_t* __restrict__ mask, float* __restrict__ cs,
                                                          SeqInfo* __restrict__ seq) {
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (r >= n) return;
  const int P = prefix_len[0], base = kv_indptr[0], j = r & 63, b = r >> 6;
  if (lane < 4) {                                        // causal inside the block: bits 0..j
    const int lo = 32 * lane;
    mask[r * 4 + lane] = j < lo ? 0u : (j - lo >= 31 ? 0xFFFFFFFFu : ((2u << (j - lo)) - 1u));
  }
  if (lane == 0) {
    pos[r] = P + r;
    slot[r] = base + P + r;
    if (j == 0) {
      seq[b].kv_base = base; seq[b].n_prefix = P + r; seq[b].n_tail = min(64, n - r);
      seq[b].order = (n + 63) / 64 - 1 - b;
    }
  }
  if (cs)
    for (int i = lane; i < d / 2; i += 64) rope_entry(cs, r, i, d, P + r, theta);
}

__global__ __launch_bounds__(64) void advance_lengths_kernel(int32_t* __restrict__ len, int B, int by) {
  const int b = blockIdx.x * 64 + threadIdx.x;
  if (b < B) len[b] += by;
}

}  // namespace

hipError_t launch_prefill_prep(const int32_t* kv_indptr, const int32_t* prefix_len, int n, int head_dim, float theta,
                               int32_t* pos, int32_t* slot, uint32_t* mask, float* cs, SeqInfo* seq, hipStream_t st) {
  if (n < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(prefill_prep_kernel, dim3((n + 3) / 4), dim3(256), 0, st, kv_indptr, prefix_len, n, head_dim, theta, pos,
                     slot, mask, cs, seq);
  return hipGetLastError();
}
hipError_t launch_advance_lengths(int32_t* len, int B, int by, hipStream_t st) {
  hipLaunchKernelGGL(advance_lengths_kernel, dim3((B + 63) / 64), dim3(64), 0, st, len, B, by);
  return hipGetLastError();
}

#define DISPATCH_BF16(flag, KERNEL, grid, block, st, ...)                                       \
  do {                                                                                          \
    if (flag) hipLaunchKernelGGL(KERNEL<true>, grid, block, 0, st, __VA_ARGS__);               \
    else hipLaunchKernelGGL(KERNEL<false>, grid, block, 0, st, __VA_ARGS__);                   \
  } while (0)

hipError_t launch_embed_rows(bool bf16, const void* embed, const int32_t* tok, int R, int k, int vocab, float* x,
                             hipStream_t st) {
  const bool vec = k % 4 == 0 && ((uintptr_t)embed & 15) == 0;
  const dim3 grid(R, ((vec ? k / 4 : k) + 255) / 256);
  if (bf16) {
    auto kernel = vec ? embed_rows_kernel<bf16_t, true> : embed_rows_kernel<bf16_t, false>;
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, (const bf16_t*)embed, tok, k, vocab, x);
  } else {
    auto kernel = vec ? embed_rows_kernel<float, true> : embed_rows_kernel<float, false>;
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, (const float*)embed, tok, k, vocab, x);
  }
  return hipGetLastError();
}

hipError_t launch_add_norm(bool bf16, float* x, const float* partial, int S, int R, int k, const void* gain, float eps,
                           void* act, float* const copy_out[4], hipStream_t st) {
  CopyOut co;
  for (int i = 0; i < 4; ++i) co.p[i] = copy_out ? copy_out[i] : nullptr;
  if (k % 4 || k > 8192) return hipErrorInvalidValue;
  const int bd = std::min(1024, (k / 4 + 63) / 64 * 64);
  if (bf16)
    hipLaunchKernelGGL(add_norm_kernel<true>, dim3(rows_grid(R)), dim3(bd), 0, st, x, partial, S, R, k, (const bf16_t*)gain, eps,
                       (bf16_t*)act, co);
  else
    hipLaunchKernelGGL(add_norm_kernel<false>, dim3(R), dim3(bd), 0, st, x, partial, S, R, k, (const float*)gain, eps,
                       (float*)act, co);
  return hipGetLastError();
}

hipError_t launch_tree_prep(const int32_t* parent, const int32_t* kv_indptr, const int32_t* prefix_len, int B, int N,
                            int head_dim, float theta, int32_t* depth, uint32_t* mask, int32_t* slot, float* cs,
                            SeqInfo* seq, hipStream_t st) {
  if (N > 64) return hipErrorInvalidValue;
  // enough workgroups that each thread computes one or two table entries, no more than ~1024 workgroups in all
  const int per_seq = std::max(1, std::min((N * (head_dim / 2) + 511) / 512, std::max(1, 1024 / B)));
  hipLaunchKernelGGL(tree_prep_kernel, dim3(B, per_seq), dim3(256), 0, st, parent, kv_indptr, prefix_len, N, head_dim, theta, depth,
                     mask, slot, cs, seq);
  return hipGetLastError();
}

hipError_t launch_rope_kv_write(const float* qkv_partial, int S, int R, int H, int Hkv, int d, const float* cs, int cs_step,
                                const int32_t* slot, void* q, void* kcache, void* vcache, hipStream_t st) {
  if (d % 8) return hipErrorInvalidValue;
  const int bd = std::min(1024, ((H + 2 * Hkv) * d / 8 + 63) / 64 * 64);
  hipLaunchKernelGGL(rope_kv_write_kernel, dim3(R), dim3(bd), 0, st, qkv_partial, S, R, H, Hkv, d, cs, cs_step, slot, (bf16_t*)q,
                     (bf16_t*)kcache, (bf16_t*)vcache);
  return hipGetLastError();
}

hipError_t launch_pack3(bool bf16, const float* a, const float* b, const float* c, int M, int k, void* act, hipStream_t st) {
  const bool vec = k % 4 == 0 && (((uintptr_t)a | (uintptr_t)b | (uintptr_t)c) & 15) == 0;
  const int cols = vec ? 3 * k / 4 : 3 * k;
  const dim3 grid(bf16 ? rows_grid(M) : M, (cols + 255) / 256);
  if (bf16) {
    auto kernel = vec ? pack3_kernel<true, true> : pack3_kernel<true, false>;
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, a, b, c, M, k, (bf16_t*)act);
  } else {
    auto kernel = vec ? pack3_kernel<false, true> : pack3_kernel<false, false>;
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, a, b, c, M, k, (float*)act);
  }
  return hipGetLastError();
}

hipError_t launch_reduce_partials(const float* partial, int S, int M, int N, float* out, hipStream_t st) {
  const size_t MN = (size_t)M * N;
  const int blocks = (int)((MN + 255) / 256 < 1024 ? (MN + 255) / 256 : 1024);
  hipLaunchKernelGGL(reduce_partials_kernel, dim3(blocks), dim3(256), 0, st, partial, S, MN, out);
  return hipGetLastError();
}

namespace {
int draft_input_threads(int k) { return std::min(1024, ((k / 4 + 63) / 64) * 64); }
}  // namespace

hipError_t launch_draft_input(bool bf16, const DraftInputArgs& a, const int32_t* tok, const float* feat, const int32_t* pos, int M,
                              hipStream_t st) {
  if (!draft_input_ok(a)) return hipErrorInvalidValue;
  const int threads = draft_input_threads(a.k);
  return with_input(bf16, a.k, threads, [&](auto type, auto passes) {
    hipLaunchKernelGGL((draft_input_kernel<type.value, passes.value>), dim3(bf16 ? rows_grid(M) : M), dim3(threads), 0, st,
                       draft_input<type.value>(a), tok, feat, pos, M);
  });
}

hipError_t launch_draft_first(bool bf16, const DraftInputArgs& a, const int32_t* tok, const float* feat, const int32_t* kv_indptr,
                              const int32_t* prefix_len, int n_new, int depth, int32_t* slot, uint32_t* mask, SeqInfo* seq,
                              hipStream_t st) {
  if (!draft_input_ok(a) || n_new < 1 || n_new > 64 || depth < 1) return hipErrorInvalidValue;
  const int threads = draft_input_threads(a.k), rows = n_new + depth - 1;
  return with_input(bf16, a.k, threads, [&](auto type, auto passes) {
    hipLaunchKernelGGL((draft_first_kernel<type.value, passes.value>), dim3(bf16 ? rows_grid(rows) : rows), dim3(threads), 0, st,
                       draft_input<type.value>(a), tok, feat, kv_indptr, prefix_len, n_new, depth, slot, mask, seq);
  });
}
