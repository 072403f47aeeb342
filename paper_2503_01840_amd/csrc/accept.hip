// Acceptance walk over the verified tree.
//
// Pass 1 (whole chip): per (row, chunk of ACCEPT_CHUNK vocabulary entries) the maximum, its first index and (sampled
// walk) the sum of exp(z - chunk max) of z = logits / T.  Pass 2: ONE wavefront per sequence walks from the root:
//   greedy     follow the child whose token is the row argmax (ties -> smaller id), else stop with it;
//   stochastic test the children in ascending node id against the running residual distribution, and on
//              failure draw the bonus token by inverse CDF of the residual in vocabulary order.
// The walk's workgroup reduces the statistics of all rows of its tree first; the bonus draw reads one chunk of logits.
#include <limits.h>

#include <algorithm>
#include <mutex>

#include "../../include/eagle3.h"
#include "common.hpp"
#include "kernels.hpp"

namespace {

constexpr int CH = ACCEPT_CHUNK;

// One wavefront per (row, chunk of 2048 logits): the chunk is read once (eight 16-byte loads per lane, all requested first)
// as four pieces of 512 entries; each piece gives (max, first arg-max, sum of exp relative to that max), the four are
// combined in order.  Bound: the stream of logits; what has to be kept out of its way is vector work, so the arg-max
// is not carried through the reduction but found afterwards from the lanes that hold the max (compares and scalar bit
// operations), and the greedy walk, which never looks at them, forms no sums.
// 512 rows of 128256 logits (263 MB): 50.6 us as one workgroup per chunk with (value, index) reductions.
template <bool SUMS>
__global__ __launch_bounds__(256) void accept_stats_kernel(const float* __restrict__ logits, int V, int n_chunks, bool vec4,
                                                          float inv_t, float* __restrict__ stats) {
  const int c = blockIdx.x * 4 + (threadIdx.x >> 6), r = blockIdx.y, lane = threadIdx.x & 63;
  if (c >= n_chunks) return;
  const float* z = logits + (size_t)r * V;
  const int lo = c * CH;
  float x[4][8];
  if (vec4) {                                            // V % 4 == 0: a lane's four entries exist or do not
#pragma unroll
    for (int w = 0; w < 4; ++w)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int v = lo + w * 512 + h * 256 + 4 * lane;
        float4 q = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
        if (v < V) q = *(const float4*)(z + v);
        x[w][4 * h] = q.x; x[w][4 * h + 1] = q.y; x[w][4 * h + 2] = q.z; x[w][4 * h + 3] = q.w;
      }
  } else {
#pragma unroll
    for (int w = 0; w < 4; ++w)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int v = lo + w * 512 + (j >> 2) * 256 + 4 * lane + (j & 3);
        x[w][j] = v < V ? z[v] : -INFINITY;
      }
  }
  float pm[4], ps[4];
  int pi[4];
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    float mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      x[w][j] *= inv_t;
      mx = fmaxf(mx, x[w][j]);
    }
    mx = wave_max(mx);
    pm[w] = mx;
    // first entry equal to the max: entries run over h, then lanes, then e = j & 3
    int first = INT_MAX;
#pragma unroll
    for (int h = 1; h >= 0; --h) {
      unsigned long long eq[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) eq[e] = __ballot(x[w][4 * h + e] == mx);
      const unsigned long long any = eq[0] | eq[1] | eq[2] | eq[3];
      if (any) {
        const int l = __ffsll((long long)any) - 1;
        const int e = (eq[0] >> l) & 1 ? 0 : (eq[1] >> l) & 1 ? 1 : (eq[2] >> l) & 1 ? 2 : 3;
        first = lo + w * 512 + h * 256 + 4 * l + e;
      }
    }
    pi[w] = mx > -INFINITY ? first : INT_MAX;
    ps[w] = 0.f;
    if constexpr (SUMS) {
      float sum = 0.f;
      if (mx > -INFINITY) {
#pragma unroll
        for (int j = 0; j < 8; ++j) sum += expf(x[w][j] - mx);   // exp(-inf) = 0 for the padding
      }
      ps[w] = wave_sum_butterfly(sum);
    }
  }
  float M = pm[0];
  int A = pi[0];
#pragma unroll
  for (int w = 1; w < 4; ++w)
    if (pm[w] > M || (pm[w] == M && pi[w] < A)) { M = pm[w]; A = pi[w]; }
  float S = 0.f;
  if constexpr (SUMS) {
#pragma unroll
    for (int w = 0; w < 4; ++w)
      if (pm[w] > -INFINITY) S += ps[w] * expf(pm[w] - M);
  }
  if (lane == 0) *(float4*)(stats + ((size_t)r * n_chunks + c) * 4) = make_float4(M, __int_as_float(A), S, 0.f);
}

// Maxima over the wavefront of four values per lane: lanes 16 g .. 16 g + 15 end with that of a, c, b, d for g = 0..3.
__device__ __forceinline__ float wave_max4(float a, float b, float c, float d) {
  auto fold32 = [](float x, float y) {         // lanes 0..31: x over the two halves, lanes 32..63: y
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  };
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(fold32(a, b)), __float_as_uint(fold32(c, d)), false, false);
  float m = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  m = xlane_max_step<0>(m); m = xlane_max_step<1>(m); m = xlane_max_step<2>(m); m = xlane_max_step<3>(m);
  return m;
}

__device__ __forceinline__ float wave_incl_scan(float v, int lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const float t = __shfl_up(v, o, 64);
    if (lane >= o) v += t;
  }
  return v;
}

// One workgroup per sequence.  Its wavefronts first reduce the chunk statistics of all N rows side by side (one memory
// round trip instead of one per step of the walk); then the first wavefront walks on values in LDS, and only the bonus draw
// goes back to memory.  Sampled walk over 64 8-node trees: 17.4 us when each step fetched its row's statistics, 9.6 us now.  A big
// tree of which nothing is accepted uses one row of the 60: the loads of all rows and of the nodes are requested together, and
// the maxima of a wavefront's four rows reduced together (60 nodes, 32000 logits, greedy, both kernels: 6.5 us with a fetch per
// step, 8.2 us when each row was loaded and reduced by itself, 6.0 us now; some nodes accepted: 11.0, 9.4 and 7.0 us).
constexpr int ROWS_PER_WAVE = 4;               // up to 64 nodes on up to 16 wavefronts
__global__ __launch_bounds__(1024) void accept_walk_kernel(const float* __restrict__ logits,
                                                        const int32_t* __restrict__ tree_tok,
                                                        const int32_t* __restrict__ parent, int N, int V, int n_chunks, bool vec4,
                                                        float inv_t, bool greedy, const float* __restrict__ uniforms,
                                                        const float* __restrict__ stats, int32_t* __restrict__ accept_len,
                                                        int32_t* __restrict__ path, int32_t* __restrict__ bonus_tok) {
  __shared__ float row_max[64], row_tot[64];
  __shared__ int row_arg[64];
  const int b = blockIdx.x, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n_waves = blockDim.x >> 6;
  const int my_par = lane < N ? parent[b * N + lane] : INT_MIN;
  const int my_tok = lane < N ? tree_tok[b * N + lane] : -1;
  float4 first[ROWS_PER_WAVE];                 // this lane's first chunk of the wavefront's rows
#pragma unroll
  for (int j = 0; j < ROWS_PER_WAVE; ++j) {
    const int r = wave + j * n_waves;
    first[j] = make_float4(-INFINITY, __int_as_float(INT_MAX), 0.f, 0.f);
    if (r < N && lane < n_chunks) first[j] = *(const float4*)(stats + ((size_t)(b * N + r) * n_chunks + lane) * 4);
  }
  auto arg_at = [&](int j, float mx) -> int {  // lane = chunk: the first lane that holds the max has the smallest index
    const unsigned long long at = __ballot(first[j].x == mx);
    return __builtin_amdgcn_readlane(__float_as_int(first[j].y), at ? __ffsll((long long)at) - 1 : 0);
  };
  auto finish = [&](int j, float mx, int am) {
    const int r = wave + j * n_waves;
    float tot = 0.f;
    if (!greedy) {
      if (lane < n_chunks) tot = first[j].z * expf(first[j].x - mx);
      for (int c = lane + 64; c < n_chunks; c += 64) {
        const float* st = stats + ((size_t)(b * N + r) * n_chunks + c) * 4;
        tot += st[2] * expf(st[0] - mx);
      }
      tot = wave_sum_butterfly(tot);
    }
    if (lane == 0) { row_max[r] = mx; row_arg[r] = am; row_tot[r] = tot; }
  };
  if (n_chunks > 64) {
#pragma unroll
    for (int j = 0; j < ROWS_PER_WAVE; ++j)
      if (wave + j * n_waves < N) {
        const float* st = stats + (size_t)(b * N + wave + j * n_waves) * n_chunks * 4;
        float mx = first[j].x;
        int am = __float_as_int(first[j].y);
        for (int c = lane + 64; c < n_chunks; c += 64) {
          const float2 s = *(const float2*)(st + c * 4);
          const int i = __float_as_int(s.y);
          if (s.x > mx || (s.x == mx && i < am)) { mx = s.x; am = i; }
        }
        wave_best_pair(mx, am);
        finish(j, mx, am);
      }
  } else if (wave + n_waves >= N) {
    const float mx = wave_max(first[0].x);
    if (wave < N) finish(0, mx, arg_at(0, mx));
  } else {                                     // the maxima of four rows together: a quarter of the steps, which up to four
    float mx = wave_max4(first[0].x, first[1].x, first[2].x, first[3].x);      // wavefronts share on each SIMD
#pragma unroll
    for (int j = 0; j < ROWS_PER_WAVE; ++j)
      if (wave + j * n_waves < N) {
        const float m = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(mx), 16 * ((j & 1) << 1 | j >> 1)));
        finish(j, m, arg_at(j, m));
      }
  }
  __syncthreads();
  if (wave > 0) return;
  if (lane < N) path[b * N + lane] = lane == 0 ? 0 : -1;
  // what the child tests of the stochastic walk read, fetched for every node at once: the target's logit of the node's
  // own token at its parent's row, and the node's uniform (one memory round trip instead of one per tested child)
  float my_z = 0.f, my_u = 0.f, my_bonus_u = 0.f;
  if (!greedy && lane < N) my_bonus_u = uniforms[(size_t)b * 2 * N + 2 * lane + 1];
  if (!greedy && lane > 0 && lane < N && my_par >= 0 && my_par < lane) {
    my_z = logits[((size_t)b * N + my_par) * V + min(max(my_tok, 0), V - 1)];
    my_u = uniforms[(size_t)b * 2 * N + 2 * lane];
  }
  int cur = 0, len = 0, bonus = 0;
  for (int step = 0; step < N; ++step) {
    const int row = b * N + cur;
    const float* st = stats + (size_t)row * n_chunks * 4;
    const float mx = row_max[cur];
    const int am = row_arg[cur];
    const unsigned long long kids = __ballot(lane < N && lane > cur && my_par == cur);
    if (greedy) {
      const unsigned long long hit = __ballot(lane < N && lane > cur && my_par == cur && my_tok == am);
      if (hit) {
        cur = __ffsll((long long)hit) - 1;
        ++len;
        if (lane == 0) path[b * N + len] = cur;
        continue;
      }
      bonus = am;
      break;
    }
    // ---- stochastic
    const float tot = row_tot[cur];
    const float* z = logits + (size_t)row * V;
    float rej = 0.f;
    int n_struck = 0, accepted = -1, struck = -1;      // lane j < n_struck holds the j-th rejected token
    unsigned long long rest = kids;
    while (rest) {
      const int c = __ffsll((long long)rest) - 1;
      rest &= rest - 1;
      const int t = min(max(__shfl(my_tok, c, 64), 0), V - 1);
      const bool is_struck = __any(lane < n_struck && struck == t);
      const float pt = expf(__shfl(my_z, c, 64) * inv_t - mx) / tot;
      const float thr = is_struck ? 0.f : pt / (1.f - rej);
      const float u = __shfl(my_u, c, 64);
      if (u < thr) { accepted = c; break; }
      if (!is_struck) {
        rej += pt;
        if (lane == n_struck) struck = t;
        ++n_struck;
      }
    }
    if (accepted >= 0) {
      cur = accepted;
      ++len;
      if (lane == 0) path[b * N + len] = cur;
      continue;
    }
    // bonus token: first v (vocabulary order) whose residual CDF reaches u * (1 - rej), in un-normalised units
    const float target = __shfl(my_bonus_u, cur, 64) * (1.f - rej) * tot;
    float carry = 0.f;
    int chunk = -1, last_pos_chunk = -1;
    float before = 0.f;
    for (int c0 = 0; c0 < n_chunks && chunk < 0; c0 += 64) {
      const int c = c0 + lane;
      float sc = c < n_chunks ? st[c * 4 + 2] * expf(st[c * 4] - mx) : 0.f;
      for (int j = 0; j < n_struck; ++j) {
        const int t = __shfl(struck, j, 64);
        if (t / CH == c) sc -= expf(z[t] * inv_t - mx);
      }
      sc = fmaxf(sc, 0.f);
      const float incl = wave_incl_scan(sc, lane) + carry;
      const unsigned long long pos = __ballot(sc > 0.f);
      const unsigned long long cross = __ballot(sc > 0.f && incl >= target);
      if (pos) last_pos_chunk = c0 + 63 - __clzll((long long)pos);
      if (cross) {
        const int l = __ffsll((long long)cross) - 1;
        chunk = c0 + l;
        before = __shfl(incl - sc, l, 64);
      }
      carry = __shfl(incl, 63, 64);
    }
    bool take_last = false;
    if (chunk < 0) { chunk = max(last_pos_chunk, 0); take_last = true; }   // rounding left the total short of the target
    // inside the chunk: 32 consecutive entries per lane
    const int v0 = chunk * CH + lane * (CH / 64);
    float e[CH / 64];
    if (vec4 && (chunk + 1) * CH <= V) {
#pragma unroll
      for (int i = 0; i < CH / 64; i += 4) {
        const float4 q = *(const float4*)(z + v0 + i);
        e[i] = q.x; e[i + 1] = q.y; e[i + 2] = q.z; e[i + 3] = q.w;
      }
    } else {
#pragma unroll
      for (int i = 0; i < CH / 64; ++i) e[i] = v0 + i < V ? z[v0 + i] : -INFINITY;
    }
    float ltot = 0.f;
#pragma unroll
    for (int i = 0; i < CH / 64; ++i) e[i] = v0 + i < V ? expf(e[i] * inv_t - mx) : 0.f;
    for (int j = 0; j < n_struck; ++j) {
      const int t = __shfl(struck, j, 64) - v0;
#pragma unroll
      for (int i = 0; i < CH / 64; ++i)
        if (t == i) e[i] = 0.f;
    }
#pragma unroll
    for (int i = 0; i < CH / 64; ++i) ltot += e[i];
    const float lincl = wave_incl_scan(ltot, lane) + before;
    const unsigned long long lpos = __ballot(ltot > 0.f);
    unsigned long long lcross = take_last ? 0ull : __ballot(ltot > 0.f && lincl >= target);
    int win_lane;
    bool last_in_lane = false;
    if (lcross) win_lane = __ffsll((long long)lcross) - 1;
    else { win_lane = lpos ? 63 - __clzll((long long)lpos) : 0; last_in_lane = true; }
    int found = -1;
    if (lane == win_lane) {
      float run = lincl - ltot;
      int last = -1;
#pragma unroll
      for (int i = 0; i < CH / 64; ++i) {
        if (e[i] > 0.f) {
          run += e[i];
          last = v0 + i;
          if (!last_in_lane && found < 0 && run >= target) found = v0 + i;
        }
      }
      if (found < 0) found = last;
    }
    bonus = __shfl(found, win_lane, 64);
    break;
  }
  if (lane == 0) {
    accept_len[b] = len;
    bonus_tok[b] = bonus;
  }
}

}  // namespace

size_t accept_scratch_floats(int R, int V) { return (size_t)R * ((V + CH - 1) / CH) * 4; }

hipError_t launch_accept(const float* logits, const int32_t* tree_tok, const int32_t* parent, int B, int N, int V,
                         float temperature, const float* uniforms, float* scratch, int32_t* accept_len, int32_t* path,
                         int32_t* bonus, hipStream_t st) {
  const int n_chunks = (V + CH - 1) / CH;
  const bool greedy = temperature <= 0.f;
  const float inv_t = greedy ? 1.f : 1.f / temperature;
  const bool vec4 = V % 4 == 0 && ((uintptr_t)logits & 15) == 0;       // whole 16-byte loads in every row
  const dim3 grid((n_chunks + 3) / 4, B * N);
  if (greedy) hipLaunchKernelGGL(accept_stats_kernel<false>, grid, dim3(256), 0, st, logits, V, n_chunks, vec4, inv_t, scratch);
  else hipLaunchKernelGGL(accept_stats_kernel<true>, grid, dim3(256), 0, st, logits, V, n_chunks, vec4, inv_t, scratch);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(accept_walk_kernel, dim3(B), dim3(64 * std::min(N, 64 / ROWS_PER_WAVE)), 0, st, logits, tree_tok, parent, N, V, n_chunks, vec4, inv_t, greedy,
                     uniforms, scratch, accept_len, path, bonus);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------------------------
// The same walk for callers that cannot allocate and hold no context (code under HIP graph capture, tight serving
// loops): the per-(row, chunk) statistics live in a fixed device array of this library instead of a workspace.
// Each GPU holds its own copy of the array at its own address; the address is looked up once per device, with that
// device current, and only that pointer (never the array's name) is handed to the kernels.
#define ACCEPT_STATIC_FLOATS (256 * 1024)                    /* 1 MiB: rows * chunks <= 65536 */
static __device__ __align__(256) float scratch[ACCEPT_STATIC_FLOATS];

namespace {
constexpr int MAX_DEVICES = 64;
std::mutex g_static_mu;
float* g_static_ptr[MAX_DEVICES] = {};

// Device address of `scratch` on the current device (looked up on the first call per device).
hipError_t static_scratch(float** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_static_mu);
  if (!g_static_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_static_ptr[dev] = (float*)p;
  }
  *out = g_static_ptr[dev];
  return hipSuccess;
}
}  // namespace

extern "C" int eagle3_accept_static(int32_t B, int32_t N, int32_t vocab, const float* logits, const int32_t* tree_tok,
                                    const int32_t* parent, float temperature, const float* uniforms, int32_t* accept_len,
                                    int32_t* path, int32_t* bonus_tok, eagle3_stream stream) {
  if (!logits || !tree_tok || !parent || !accept_len || !path || !bonus_tok) return EAGLE3_E_NULL;
  if (temperature > 0.f && !uniforms) return EAGLE3_E_NULL;
  if (B < 1 || N < 1 || N > 64 || vocab < 1 || !(temperature >= 0.f)) return EAGLE3_E_SHAPE;
  if ((size_t)B * N > (size_t)ACCEPT_STATIC_FLOATS) return EAGLE3_E_SHAPE;
  if (accept_scratch_floats(B * N, vocab) > (size_t)ACCEPT_STATIC_FLOATS) return EAGLE3_E_SHAPE;
  float* ptr = nullptr;
  if (static_scratch(&ptr) != hipSuccess) return EAGLE3_E_HIP;
  // every (row, chunk) entry the walk reads is written by the statistics pass of the same call: nothing to clear
  if (launch_accept(logits, tree_tok, parent, B, N, vocab, temperature, uniforms, ptr, accept_len, path, bonus_tok,
                    (hipStream_t)stream) != hipSuccess)
    return EAGLE3_E_HIP;
  return EAGLE3_OK;
}
