// Row-wise kernels between the GEMMs: embedding gather, residual add + RMSNorm, rotary embedding and
// cache write, tree bookkeeping, feature packing.  All are tiny next to the weight
// streams; they exist to hand the next GEMM its operand in the layout it reads.
#include <algorithm>

#include "common.hpp"
#include "draft_row.hpp"
#include "kernels.hpp"

namespace {

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

// Part y of n_parts of sequence b's tree: every part walks the tree (parents staged in LDS: one memory round trip, then the walks
// stay on chip) and fills its share of the rotary table, whose sines and cosines are the bulk of the work; part 0
// also writes the masks, slots and the sequence record.
__device__ __forceinline__ void tree_prep(const BeginRows& p, int b, int y, int n_parts) {
  __shared__ int sdepth[64], spar[64];
  __shared__ int rank;
  const int i = threadIdx.x, threads = blockDim.x, B = p.B, N = p.N, d = p.head_dim;
  const int P = p.prefix_len[b], base = p.kv_indptr[b];
  if (i < N) spar[i] = p.parent[b * N + i];
  if (i == 0) rank = 0;
  __syncthreads();
  if (y == 0) {
    // rank of this sequence by prefix length, longest first (ties: smaller index first): attention hands out its
    // workgroups in that order, so that the long sequences start first and the short ones fill the tail
    int longer = 0;
    for (int o = i; o < B; o += threads) {
      const int Po = p.prefix_len[o];
      longer += (Po > P || (Po == P && o < b)) ? 1 : 0;
    }
    if (longer) atomicAdd(&rank, longer);
  }
  if (i < N) {
    uint32_t m[4] = {0u, 0u, 0u, 0u};
    int cur = i, dep = 0;
    for (int it = 0; it < N; ++it) {                     // bounded walk: malformed parents cannot loop
      m[cur >> 5] |= 1u << (cur & 31);
      const int q = spar[cur];
      if (q < 0 || q >= cur) break;
      cur = q;
      ++dep;
    }
    sdepth[i] = dep;
    if (y == 0) {
      const int r = b * N + i;
      p.slot[r] = base + P + i;
#pragma unroll
      for (int w = 0; w < 4; ++w) p.mask[r * 4 + w] = m[w];
    }
  }
  __syncthreads();
  if (y == 0 && i == 0) {
    p.seq[rank].order = b;
    p.seq[b].kv_base = base; p.seq[b].n_prefix = P; p.seq[b].n_tail = N;
  }
  const int half = d / 2;
  for (int e = y * threads + i; e < N * half; e += threads * n_parts) {
    const int row = e / half, f = e % half;
    rope_entry(p.cs, b * N + row, f, d, P + sdepth[row], p.theta);
  }
}

// Rows of a prefill chunk of n, one per wavefront: row r continues the sequence at position P + r.  For attention the chunk is
// cut into blocks of 64 rows: block b sees the context and every earlier block unconditionally (n_prefix = P + 64 b) and its
// own rows causally through the row masks, so the tree kernels run a chunk of any length as a batch of "sequences" that
// share one cache.  The last block has the most keys, so it is handed out first.
__device__ __forceinline__ void prefill_prep(const BeginRows& p, int r, int n) {
  const int lane = threadIdx.x & 63;
  if (r >= n) return;
  const int P = p.prefix_len[0], base = p.kv_indptr[0], j = r & 63, b = r >> 6;
  if (lane < 4) {                                        // causal inside the block: bits 0..j
    const int lo = 32 * lane;
    p.mask[r * 4 + lane] = j < lo ? 0u : (j - lo >= 31 ? 0xFFFFFFFFu : ((2u << (j - lo)) - 1u));
  }
  if (lane == 0) {
    p.slot[r] = base + P + r;
    if (j == 0) {
      p.seq[b].kv_base = base; p.seq[b].n_prefix = P + r; p.seq[b].n_tail = min(64, n - r);
      p.seq[b].order = (n + 63) / 64 - 1 - b;
    }
  }
  for (int i = lane; i < p.head_dim / 2; i += 64) rope_entry(p.cs, r, i, p.head_dim, P + r, p.theta);
}

// How a pass over R rows begins: bookkeeping by the first prep_wgs workgroups (a multiple of 8: see row_of_workgroup), and each row's
// residual, from the embedding table or as it lies in x, with its copies and, with a gain, the RMSNorm that the first projection reads.  None needs
// another: as three launches (bookkeeping, embedding, norm: 5.7 + 4.8 + 4.9 us for 60 rows of 4096) each waited for the one before;
// 6.0 here (8.0 with half as many, twice as large workgroups for the rotary table).  It is there for the two launches it takes out of every pass, which
// the host hands over too; of a bf16 pass those 9 us are less than two runs differ (77 tokens 4665 -> 4665 us, 4 trees of 29 nodes 1555 -> 1548).
// The rotary table's fp64 beside the row work takes 96 registers, so a CU holds one workgroup of 1024 threads.
template <bool BF16>
__global__ __launch_bounds__(1024) void begin_rows_kernel(BeginRows p, int prep_wgs, int parts, float* __restrict__ x, int R, int k,
                                                         const typename Act<BF16>::type* __restrict__ gain, float eps,
                                                         typename Act<BF16>::type* __restrict__ act, CopyOut co) {
  __shared__ float red[17];
  if ((int)blockIdx.x < prep_wgs) {
    if (!p.parent) prefill_prep(p, blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6), R);
    else if ((int)blockIdx.x < p.B * parts) tree_prep(p, blockIdx.x / parts, blockIdx.x % parts, parts);
    return;
  }
  const int r = row_of_workgroup<BF16>(blockIdx.x - prep_wgs), nvec = k >> 2, bd = blockDim.x;
  if (r >= R) return;
  constexpr int VPT = 2;
  typedef typename Act<BF16>::type T;
  const T* table = (const T*)p.embed;
  const size_t from = table ? (size_t)min(max(p.tok[r], 0), p.vocab - 1) * k : 0;
  const bool whole = ((uintptr_t)table & 15) == 0;       // the caller's table may start anywhere
  float4 val[VPT], g[VPT];
  float ss = 0.f;
#pragma unroll
  for (int j = 0; j < VPT; ++j) {
    const int v = threadIdx.x + j * bd;
    if (v < nvec) {
      if (gain) g[j] = load4_f32(gain, 4 * v);
      float4 a;
      if (!table) a = *(const float4*)(x + (size_t)r * k + 4 * v);
      else if (whole) a = load4_f32(table, from + 4 * v);
      else a = make_float4(load_f32(table, from + 4 * v), load_f32(table, from + 4 * v + 1), load_f32(table, from + 4 * v + 2), load_f32(table, from + 4 * v + 3));
      if (table) *(float4*)(x + (size_t)r * k + 4 * v) = a;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (co.p[i]) *(float4*)(co.p[i] + (size_t)r * k + 4 * v) = a;
      ss += a.x * a.x + a.y * a.y + a.z * a.z + a.w * a.w;
      val[j] = a;
    }
  }
  if (!gain) return;
  ss = block_sum(ss, red);
  const float inv = 1.0f / sqrtf(ss / (float)k + eps);
#pragma unroll
  for (int j = 0; j < VPT; ++j) {
    const int v = threadIdx.x + j * bd;
    if (v < nvec)
      Act<BF16>::store4(act, r, 4 * v, k, val[j].x * inv * g[j].x, val[j].y * inv * g[j].y, val[j].z * inv * g[j].z,
                        val[j].w * inv * g[j].w);
  }
}

// One workgroup per row; a thread handles four consecutive rotary pairs (i..i+3, i+d/2..i+d/2+3) of one head of d = 128.  (fp32: gemm_f32.hip.)
__global__ __launch_bounds__(1024) void rope_kv_write_kernel(const float* __restrict__ qkv, int S, int R, int H, int Hkv,
                                                            const float* __restrict__ cs, int cs_step,
                                                            const int32_t* __restrict__ slot, bf16_t* __restrict__ q,
                                                            bf16_t* __restrict__ kc, bf16_t* __restrict__ vc) {
  constexpr int d = 128, half = d / 2, q4 = half / 4;
  const int r = blockIdx.x, NT = (H + 2 * Hkv) * d;
  const size_t sl = (size_t)slot[r];
  for (int e = threadIdx.x; e < (H + 2 * Hkv) * q4; e += blockDim.x) {
    const int h = (unsigned)e / q4, i = (unsigned)e % q4 * 4;
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

// Draft forward 1 of a tree: n_new rows behind the context, causal among themselves (or, without mask and seq, rows of which only the keys and
// values are wanted); their bookkeeping comes with their input
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
    if (mask && tid < 4) {
      const int lo = 32 * tid;
      mask[r * 4 + tid] = r < lo ? 0u : (r - lo >= 31 ? 0xFFFFFFFFu : ((2u << (r - lo)) - 1u));     // bits 0..r
    }
    if (tid == 0) {
      slot[r] = base + P + r;
      if (seq && r == 0) { seq[0].kv_base = base; seq[0].n_prefix = P; seq[0].n_tail = n_new; seq[0].order = 0; }
    }
    DraftGains<BF16, VPT> gains;
    load_gains(p, gains);
    draft_input_row(p, r, tok[r], feat + (size_t)r * p.k, gains, sums);
  }
  for (int i = tid; i < p.head_dim / 2; i += blockDim.x) rope_entry(p.cs, r, i, p.head_dim, P + r, p.theta);
}

__global__ __launch_bounds__(128) void rope_table_kernel(float* __restrict__ cs, const int32_t* __restrict__ prefix_len, int at, int d,
                                                        float theta) {
  for (int i = threadIdx.x; i < d / 2; i += 128) rope_entry(cs, 0, i, d, prefix_len[0] + at, theta);
}

// The end of a prefill chunk: n positions are in the target's cache and m in the draft's.
__global__ __launch_bounds__(64) void end_prefill_kernel(int32_t* len, int n, int32_t* draft_len, int m) {
  if (threadIdx.x == 0) { len[0] += n; draft_len[0] += m; }
}

}  // namespace

hipError_t launch_rope_table(float* cs, const int32_t* prefix_len, int at, int head_dim, float theta, hipStream_t st) {
  hipLaunchKernelGGL(rope_table_kernel, dim3(1), dim3(128), 0, st, cs, prefix_len, at, head_dim, theta);
  return hipGetLastError();
}

hipError_t launch_end_prefill(int32_t* len, int n, int32_t* draft_len, int m, hipStream_t st) {
  hipLaunchKernelGGL(end_prefill_kernel, dim3(1), dim3(64), 0, st, len, n, draft_len, m);
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

hipError_t launch_begin_rows(bool bf16, const BeginRows& b, float* x, int R, int k, const void* gain, float eps, void* act,
                             float* const copy_out[4], hipStream_t st) {
  if (k % 4 || k > 8192 || (b.parent && b.N > 64)) return hipErrorInvalidValue;
  CopyOut co;
  for (int i = 0; i < 4; ++i) co.p[i] = copy_out ? copy_out[i] : nullptr;
  const int threads = std::min(1024, std::max((k / 4 + 63) / 64, 4) * 64);
  // trees: 512 entries of the rotary table (fp64 sines and cosines) to a workgroup, no more than ~1024 workgroups in all; prefill: a wavefront per row
  const int parts = std::max(1, std::min((b.N * (b.head_dim / 2) + 511) / 512, std::max(1, 1024 / std::max(1, b.B))));
  const int prep = b.parent ? b.B * parts : (R + threads / 64 - 1) / (threads / 64), prep_wgs = (prep + 7) / 8 * 8;
  const dim3 grid(prep_wgs + (bf16 ? rows_grid(R) : R));
  if (bf16)
    hipLaunchKernelGGL(begin_rows_kernel<true>, grid, dim3(threads), 0, st, b, prep_wgs, parts, x, R, k, (const bf16_t*)gain, eps, (bf16_t*)act, co);
  else
    hipLaunchKernelGGL(begin_rows_kernel<false>, grid, dim3(threads), 0, st, b, prep_wgs, parts, x, R, k, (const float*)gain, eps, (float*)act, co);
  return hipGetLastError();
}

hipError_t launch_rope_kv_write(const float* qkv_partial, int S, int R, int H, int Hkv, int d, const float* cs, int cs_step,
                                const int32_t* slot, void* q, void* kcache, void* vcache, hipStream_t st) {
  if (d != 128) return hipErrorInvalidValue;
  const int bd = std::min(1024, ((H + 2 * Hkv) * d / 8 + 63) / 64 * 64);
  hipLaunchKernelGGL(rope_kv_write_kernel, dim3(R), dim3(bd), 0, st, qkv_partial, S, R, H, Hkv, cs, cs_step, slot, (bf16_t*)q,
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
  if (!draft_input_ok(a) || n_new < 1 || (mask && n_new > 64) || depth < 1) return hipErrorInvalidValue;
  const int threads = draft_input_threads(a.k), rows = n_new + depth - 1;
  return with_input(bf16, a.k, threads, [&](auto type, auto passes) {
    hipLaunchKernelGGL((draft_first_kernel<type.value, passes.value>), dim3(bf16 ? rows_grid(rows) : rows), dim3(threads), 0, st,
                       draft_input<type.value>(a), tok, feat, kv_indptr, prefix_len, n_new, depth, slot, mask, seq);
  });
}
