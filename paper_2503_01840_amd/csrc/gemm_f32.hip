// fp32 GEMM for the exact-arithmetic (small model) configuration: out[m, n] = sum_k x[m, k] w[n, k] over up to three
// stacked weight matrices, or h = silu(gate) * up of two.  What stands between two products of a layer is done by them, as a launch
// of its own costs as much as a product does here: the RMSNorm of the input rows (every wavefront sums their squares along with
// its own products; 3.1 us a launch saved, as long as there are few wavefronts: f32_norm_inside), the rotation and cache write of q/k/v, and the residual sum.
//
// One wavefront per (weight row, group of 8 activation rows); the lanes stride over K, four consecutive k at a time.  At
// these sizes (a few hundred rows of a few hundred k, all of it in L2) a launch is bound by its own latency: the loads of
// an iteration are requested together, the eight sums of a wavefront are reduced together (two halving steps leave four
// sums per register, then four DPP steps), and a stacked weight is one launch (16 rows of a 256 x 256 weight: 5.2 us with one
// load per iteration and eight shuffle reductions one after the other, 3.7 us now).
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace {
constexpr int RM = 8;

struct F32Params {
  const float* x;
  const float* w[3];
  int rows[3];
  int nmat, M, N, K;
  Divisor by_half;             // half a head, for rotary pairs
  float* out;
  F32Fuse f;
};
enum { STORE, SWIGLU, RESIDUAL, ROPE };

// acc[r] (r = 0..7) summed over the 64 lanes: on return lane 16 j + i holds row_of(j) of lo and 4 + row_of(j) of hi,
// row_of = 0, 2, 1, 3.
__device__ __forceinline__ void sum8(const float (&acc)[RM], float& lo, float& hi) {
  auto fold32 = [](float a, float b) {       // lanes 0..31: a summed over the two halves, lanes 32..63: b
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  };
  auto fold16 = [](float a, float b) {       // even groups of 16 lanes: a summed over two neighbouring groups, odd: b
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  };
  lo = fold16(fold32(acc[0], acc[1]), fold32(acc[2], acc[3]));
  hi = fold16(fold32(acc[4], acc[5]), fold32(acc[6], acc[7]));
  lo = xlane_sum_step<0>(lo); hi = xlane_sum_step<0>(hi);
  lo = xlane_sum_step<1>(lo); hi = xlane_sum_step<1>(hi);
  lo = xlane_sum_step<2>(lo); hi = xlane_sum_step<2>(hi);
  lo = xlane_sum_step<3>(lo); hi = xlane_sum_step<3>(hi);
}

// NW weight rows per wavefront (2: gate and up, or the two of a rotary pair); VEC: 16-byte loads.  NORM: acc sums gain * x * w, and
// ss the squares of x.
template <int NW, bool NORM, bool VEC>
__device__ __forceinline__ void dot_rows(const F32Params& p, const float* const (&wr)[NW], int m0, int lane, float (&acc)[NW][RM],
                                         float (&ss)[RM]) {
  const float* xr[RM];
#pragma unroll
  for (int r = 0; r < RM; ++r) xr[r] = p.x + (size_t)min(m0 + r, p.M - 1) * p.K;
#pragma unroll
  for (int r = 0; r < RM; ++r) {
    ss[r] = 0.f;
#pragma unroll
    for (int i = 0; i < NW; ++i) acc[i][r] = 0.f;
  }
  if constexpr (VEC) {
    for (int k = 4 * lane; k < p.K; k += 256) {
      float4 w[NW], x[RM], g;
#pragma unroll
      for (int i = 0; i < NW; ++i) w[i] = *(const float4*)(wr[i] + k);
#pragma unroll
      for (int r = 0; r < RM; ++r) x[r] = *(const float4*)(xr[r] + k);
      if constexpr (NORM) {
        g = *(const float4*)(p.f.gain + k);
#pragma unroll
        for (int r = 0; r < RM; ++r) ss[r] = fmaf(x[r].w, x[r].w, fmaf(x[r].z, x[r].z, fmaf(x[r].y, x[r].y, fmaf(x[r].x, x[r].x, ss[r]))));
#pragma unroll
        for (int i = 0; i < NW; ++i) w[i] = make_float4(w[i].x * g.x, w[i].y * g.y, w[i].z * g.z, w[i].w * g.w);
      }
#pragma unroll
      for (int i = 0; i < NW; ++i)
#pragma unroll
        for (int r = 0; r < RM; ++r)
          acc[i][r] = fmaf(x[r].w, w[i].w, fmaf(x[r].z, w[i].z, fmaf(x[r].y, w[i].y, fmaf(x[r].x, w[i].x, acc[i][r]))));
    }
  } else {
    for (int k = lane; k < p.K; k += 64) {
      const float g = NORM ? p.f.gain[k] : 1.f;
#pragma unroll
      for (int r = 0; r < RM; ++r) {
        const float x = xr[r][k];
        if constexpr (NORM) ss[r] = fmaf(x, x, ss[r]);
#pragma unroll
        for (int i = 0; i < NW; ++i) acc[i][r] = fmaf(x, wr[i][k] * g, acc[i][r]);
      }
    }
  }
}

template <int EPI, bool NORM, bool VEC>
__global__ __launch_bounds__(256) void gemm_f32_kernel(F32Params p) {
  constexpr int NW = EPI == SWIGLU || EPI == ROPE ? 2 : 1;
  const int lane = threadIdx.x & 63, n = blockIdx.x * 4 + (threadIdx.x >> 6), m0 = blockIdx.y * RM;
  if (n >= p.N) return;
  const float* wr[NW];
  const F32Fuse& f = p.f;
  const int half = f.d / 2;
  const int head = EPI == ROPE ? n / p.by_half : 0, pair = EPI == ROPE ? n - head * half : 0;
  if constexpr (EPI == SWIGLU) {
    wr[0] = p.w[0] + (size_t)n * p.K;
    wr[1] = p.w[1] + (size_t)n * p.K;
  } else {
    int i = 0, row = EPI == ROPE ? head * f.d + pair : n;
    while (i + 1 < p.nmat && row >= p.rows[i]) { row -= p.rows[i]; ++i; }
    wr[0] = p.w[i] + (size_t)row * p.K;
    if constexpr (EPI == ROPE) wr[1] = wr[0] + (size_t)half * p.K;
  }
  // what the epilogue reads of rows m and m + 4, requested before the products
  const int j = lane >> 4, m = m0 + ((j & 1) << 1 | j >> 1), mc[2] = {min(m, p.M - 1), min(m + 4, p.M - 1)};
  float before[2], cosine[2] = {1.f, 1.f}, sine[2] = {0.f, 0.f};
  int slot[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    if constexpr (EPI == RESIDUAL) before[i] = p.out[(size_t)mc[i] * p.N + n];
    if constexpr (EPI == ROPE) {
      if (head < f.H + f.Hkv) { cosine[i] = f.cs[(size_t)mc[i] * f.cs_step + pair]; sine[i] = f.cs[(size_t)mc[i] * f.cs_step + half + pair]; }
      slot[i] = f.slot[mc[i]];
    }
  }
  float acc[NW][RM], ss[RM], sum[2][NW];
  dot_rows<NW, NORM, VEC>(p, wr, m0, lane, acc, ss);
#pragma unroll
  for (int i = 0; i < NW; ++i) sum8(acc[i], sum[0][i], sum[1][i]);
  if constexpr (NORM) {
    float sq[2];
    sum8(ss, sq[0], sq[1]);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float inv = 1.0f / sqrtf(sq[i] / (float)p.K + f.eps);
#pragma unroll
      for (int w = 0; w < NW; ++w) sum[i][w] *= inv;
    }
  }
  if (lane & 15) return;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = m + 4 * i;
    if (row >= p.M) break;
    const float (&v)[NW] = sum[i];
    const size_t at = (size_t)row * p.N + n;
    if constexpr (EPI == STORE) p.out[at] = v[0];
    if constexpr (EPI == SWIGLU) p.out[at] = v[0] / (1.f + expf(-v[0])) * v[1];
    if constexpr (EPI == RESIDUAL) {
      const float x = before[i] + v[0];
      p.out[at] = x;
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (f.copies[t]) f.copies[t][at] = x;
    }
    if constexpr (EPI == ROPE) {
      float a = v[0], b = v[1];
      if (head < f.H + f.Hkv) { a = v[0] * cosine[i] - v[1] * sine[i]; b = v[1] * cosine[i] + v[0] * sine[i]; }
      float* dst = head < f.H ? p.out + ((size_t)row * f.H + head) * f.d
                              : (head < f.H + f.Hkv ? f.kc + ((size_t)slot[i] * f.Hkv + head - f.H) * f.d
                                                    : f.vc + ((size_t)slot[i] * f.Hkv + head - f.H - f.Hkv) * f.d);
      dst[pair] = a;
      dst[half + pair] = b;
    }
  }
}
}  // namespace

hipError_t launch_gemm_f32(const float* x, const GemmWeights& W, int M, int N, int K, int epi, float* out, hipStream_t st,
                           const F32Fuse& fuse) {
  if (M <= 0 || N <= 0 || K <= 0) return hipErrorInvalidValue;
  if (epi == GEMM_EPI_SWIGLU && (W.mode != 1 || N % 2)) return hipErrorInvalidValue;
  if (epi == GEMM_EPI_ROPE && (fuse.d < 8 || fuse.d % 8 || N != (fuse.H + 2 * fuse.Hkv) * fuse.d)) return hipErrorInvalidValue;
  if (fuse.gain && (K % 4 || K > 8192)) return hipErrorInvalidValue;
  F32Params p;
  p.x = x;
  bool vec = K % 4 == 0 && (((uintptr_t)x | (uintptr_t)fuse.gain) & 15) == 0;        // 16-byte loads in every row
  for (int i = 0; i < 3; ++i) {
    p.w[i] = (const float*)W.w[i];
    p.rows[i] = W.rows[i];
    if (i < W.nmat) vec = vec && ((uintptr_t)W.w[i] & 15) == 0;
  }
  p.nmat = W.nmat; p.M = M; p.N = epi == GEMM_EPI_SWIGLU || epi == GEMM_EPI_ROPE ? N / 2 : N; p.K = K;
  p.out = out;
  p.f = fuse;
  p.by_half = divisor(epi == GEMM_EPI_ROPE ? fuse.d / 2 : 1);
  const dim3 grid((p.N + 3) / 4, (M + RM - 1) / RM);
  auto run = [&](auto e) {
    constexpr int E = decltype(e)::value;
    auto kernel = fuse.gain ? (vec ? gemm_f32_kernel<E, true, true> : gemm_f32_kernel<E, true, false>)
                            : (vec ? gemm_f32_kernel<E, false, true> : gemm_f32_kernel<E, false, false>);
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, p);
  };
  if (epi == GEMM_EPI_SWIGLU) run(std::integral_constant<int, SWIGLU>());
  else if (epi == GEMM_EPI_RESIDUAL) run(std::integral_constant<int, RESIDUAL>());
  else if (epi == GEMM_EPI_ROPE) run(std::integral_constant<int, ROPE>());
  else run(std::integral_constant<int, STORE>());
  return hipGetLastError();
}
