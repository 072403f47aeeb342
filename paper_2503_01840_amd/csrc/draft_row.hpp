// Input rows of the draft layer, formed by every kernel that starts a draft forward.
#pragma once
#include "common.hpp"
#include "kernels.hpp"

// cos/sin of pos * theta^(-2i/d) in fp64, stored fp32: cs[r][i] = cos, cs[r][d/2 + i] = sin
__device__ __forceinline__ void rope_entry(float* cs, int r, int i, int d, int pos, float theta) {
  const double inv = pow((double)theta, -2.0 * (double)i / (double)d);
  double s, c;
  sincos((double)pos * inv, &s, &c);
  cs[(size_t)r * d + i] = (float)c;
  cs[(size_t)r * d + d / 2 + i] = (float)s;
}

template <bool BF16>
struct DraftInput {
  typedef typename Act<BF16>::type T;
  const T* embed;
  const T* g_embed;
  const T* g_feat;
  T* act;                // [rows, 2 k]
  float* y;              // [rows, k]
  float* cs;             // [rows, head_dim]
  int vocab, k, head_dim;
  float eps, theta;
};

template <bool BF16>
inline DraftInput<BF16> draft_input(const DraftInputArgs& a) {
  typedef typename Act<BF16>::type T;
  return {(const T*)a.embed, (const T*)a.g_embed, (const T*)a.g_feat, (T*)a.act, a.y, a.cs, a.vocab, a.k, a.head_dim, a.eps, a.theta};
}
inline bool draft_input_ok(const DraftInputArgs& a) { return a.k % 4 == 0 && a.k <= 8192; }   // as the norms that follow
// f(type, passes): the activations' type (1: bf16) and the passes over a row of k columns that `threads` make.  Kernels have no more passes
// than they need: a kernel runs once between two streams of weights, which leave nothing of it in the caches, and its code arrives a line at a time.
template <int N> struct Int { static constexpr int value = N; };
template <typename F>
inline hipError_t with_input(bool bf16, int k, int threads, F f) {
  const bool one = k / 4 <= threads;
  if (bf16) one ? f(Int<1>(), Int<1>()) : f(Int<1>(), Int<2>());
  else one ? f(Int<0>(), Int<1>()) : f(Int<0>(), Int<2>());
  return hipGetLastError();
}

// Four entries of a gain as they lie in memory: requested at the start of a kernel and converted where they are used.
template <bool BF16> struct RawGain { uint2 v; };
template <> struct RawGain<false> { float4 v; };
__device__ __forceinline__ float4 gain_f32(const RawGain<true>& g) {
  return make_float4(__uint_as_float(g.v.x << 16), __uint_as_float(g.v.x & 0xFFFF0000u), __uint_as_float(g.v.y << 16),
                     __uint_as_float(g.v.y & 0xFFFF0000u));
}
__device__ __forceinline__ float4 gain_f32(const RawGain<false>& g) { return g.v; }
template <bool BF16, int VPT> struct DraftGains { RawGain<BF16> e[VPT], f[VPT]; };
template <bool BF16, int VPT>
__device__ __forceinline__ void load_gains(const DraftInput<BF16>& p, DraftGains<BF16, VPT>& g) {
  typedef decltype(RawGain<BF16>::v) Raw;
#pragma unroll
  for (int j = 0; j < VPT; ++j) {
    const int c = 4 * (threadIdx.x + j * blockDim.x);
    if (c < p.k) { g.e[j].v = *(const Raw*)(p.g_embed + c); g.f[j].v = *(const Raw*)(p.g_feat + c); }
  }
}

// act[r] = [RMSNorm(E[token]; g_embed) ; RMSNorm(f; g_feat)], y[r] = f.  One workgroup, four consecutive columns per thread and pass, the
// row kept in registers between the sums of squares and the normalising pass (VPT passes: k <= 4 VPT blockDim.x).  sums: nothing has used them before.
struct RowSums { float e[16], f[16]; };
template <bool BF16, int VPT>
__device__ __forceinline__ void draft_input_row(const DraftInput<BF16>& p, int r, int token, const float* __restrict__ f,
                                                const DraftGains<BF16, VPT>& gains, RowSums& sums) {
  const int k = p.k, t = min(max(token, 0), p.vocab - 1), nw = blockDim.x >> 6;
  float4 e[VPT], v[VPT];
  float se = 0.f, sf = 0.f;
#pragma unroll
  for (int j = 0; j < VPT; ++j) {
    const int c = 4 * (threadIdx.x + j * blockDim.x);
    if (c < k) {
      e[j] = load4_f32(p.embed, (size_t)t * k + c);
      v[j] = *(const float4*)(f + c);
      *(float4*)(p.y + (size_t)r * k + c) = v[j];
      se += e[j].x * e[j].x + e[j].y * e[j].y + e[j].z * e[j].z + e[j].w * e[j].w;
      sf += v[j].x * v[j].x + v[j].y * v[j].y + v[j].z * v[j].z + v[j].w * v[j].w;
    }
  }
  // sums in the order of block_sum, as every norm has them: a last bit of an input can turn over candidates that are all but tied
  se = wave_sum(se);
  sf = wave_sum(sf);
  if ((threadIdx.x & 63) == 0) { sums.e[threadIdx.x >> 6] = se; sums.f[threadIdx.x >> 6] = sf; }
  __syncthreads();
  se = sf = 0.f;
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    se += w < nw ? sums.e[w] : 0.f;
    sf += w < nw ? sums.f[w] : 0.f;
  }
  const float ie = 1.0f / sqrtf(se / (float)k + p.eps), iv = 1.0f / sqrtf(sf / (float)k + p.eps);
#pragma unroll
  for (int j = 0; j < VPT; ++j) {
    const int c = 4 * (threadIdx.x + j * blockDim.x);
    if (c < k) {
      const float4 ge = gain_f32(gains.e[j]), gf = gain_f32(gains.f[j]);
      Act<BF16>::store4(p.act, r, c, 2 * k, e[j].x * ie * ge.x, e[j].y * ie * ge.y, e[j].z * ie * ge.z, e[j].w * ie * ge.w);
      Act<BF16>::store4(p.act, r, k + c, 2 * k, v[j].x * iv * gf.x, v[j].y * iv * gf.y, v[j].z * iv * gf.z, v[j].w * iv * gf.w);
    }
  }
}
