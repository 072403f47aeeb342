// fp32 GEMM for the exact-arithmetic (small model) configuration: out[m, n] = sum_k x[m, k] w[n, k] over up to three
// stacked weight matrices, or h = silu(gate) * up of two.
//
// One wavefront per (weight row, group of 8 activation rows); the lanes stride over K, four consecutive k at a time.  At
// these sizes (a few hundred rows of a few hundred k, all of it in L2) a launch is bound by its own latency: the loads of
// an iteration are requested together, the eight sums of a wavefront are reduced together (two halving steps leave four
// sums per register, then four DPP steps), and a stacked weight is one launch (16 rows of a 256 x 256 weight: 5.2 us with one
// load per iteration and eight shuffle reductions one after the other, 3.7 us now).
#include "common.hpp"
#include "kernels.hpp"

namespace {
constexpr int RM = 8;

struct F32Params {
  const float* x;
  const float* w[3];
  int rows[3];
  int nmat, M, N, K;
  float* out;
};

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

// NW weight rows per wavefront (2: gate and up); VEC: 16-byte loads
template <int NW, bool VEC>
__device__ __forceinline__ void dot_rows(const F32Params& p, const float* const (&wr)[NW], int m0, int lane, float (&acc)[NW][RM]) {
  const float* xr[RM];
#pragma unroll
  for (int r = 0; r < RM; ++r) xr[r] = p.x + (size_t)min(m0 + r, p.M - 1) * p.K;
#pragma unroll
  for (int i = 0; i < NW; ++i)
#pragma unroll
    for (int r = 0; r < RM; ++r) acc[i][r] = 0.f;
  if constexpr (VEC) {
    for (int k = 4 * lane; k < p.K; k += 256) {
      float4 w[NW], x[RM];
#pragma unroll
      for (int i = 0; i < NW; ++i) w[i] = *(const float4*)(wr[i] + k);
#pragma unroll
      for (int r = 0; r < RM; ++r) x[r] = *(const float4*)(xr[r] + k);
#pragma unroll
      for (int i = 0; i < NW; ++i)
#pragma unroll
        for (int r = 0; r < RM; ++r)
          acc[i][r] = fmaf(x[r].w, w[i].w, fmaf(x[r].z, w[i].z, fmaf(x[r].y, w[i].y, fmaf(x[r].x, w[i].x, acc[i][r]))));
    }
  } else {
    for (int k = lane; k < p.K; k += 64)
#pragma unroll
      for (int i = 0; i < NW; ++i) {
        const float w = wr[i][k];
#pragma unroll
        for (int r = 0; r < RM; ++r) acc[i][r] = fmaf(xr[r][k], w, acc[i][r]);
      }
  }
}

template <bool SWIGLU, bool VEC>
__global__ __launch_bounds__(256) void gemm_f32_kernel(F32Params p) {
  constexpr int NW = SWIGLU ? 2 : 1;
  const int lane = threadIdx.x & 63, n = blockIdx.x * 4 + (threadIdx.x >> 6), m0 = blockIdx.y * RM;
  if (n >= p.N) return;
  const float* wr[NW];
  if constexpr (SWIGLU) {
    wr[0] = p.w[0] + (size_t)n * p.K;
    wr[1] = p.w[1] + (size_t)n * p.K;
  } else {
    int i = 0, row = n;
    while (i + 1 < p.nmat && row >= p.rows[i]) { row -= p.rows[i]; ++i; }
    wr[0] = p.w[i] + (size_t)row * p.K;
  }
  float acc[NW][RM], lo[NW], hi[NW];
  dot_rows<NW, VEC>(p, wr, m0, lane, acc);
#pragma unroll
  for (int i = 0; i < NW; ++i) sum8(acc[i], lo[i], hi[i]);
  const int j = lane >> 4, m = m0 + ((j & 1) << 1 | j >> 1);
  if (lane & 15) return;
  auto value = [](const float (&v)[NW]) {
    if constexpr (SWIGLU) return v[0] / (1.f + expf(-v[0])) * v[1];
    else return v[0];
  };
  if (m < p.M) p.out[(size_t)m * p.N + n] = value(lo);
  if (m + 4 < p.M) p.out[(size_t)(m + 4) * p.N + n] = value(hi);
}
}  // namespace

hipError_t launch_gemm_f32(const float* x, const GemmWeights& W, int M, int N, int K, int epi, float* out, hipStream_t st) {
  if (M <= 0 || N <= 0 || K <= 0) return hipErrorInvalidValue;
  if (epi == GEMM_EPI_SWIGLU && (W.mode != 1 || N % 2)) return hipErrorInvalidValue;
  F32Params p;
  p.x = x;
  bool vec = K % 4 == 0 && ((uintptr_t)x & 15) == 0;         // 16-byte loads in every row
  for (int i = 0; i < 3; ++i) {
    p.w[i] = (const float*)W.w[i];
    p.rows[i] = W.rows[i];
    if (i < W.nmat) vec = vec && ((uintptr_t)W.w[i] & 15) == 0;
  }
  p.nmat = W.nmat; p.M = M; p.N = epi == GEMM_EPI_SWIGLU ? N / 2 : N; p.K = K;
  p.out = out;
  auto kernel = epi == GEMM_EPI_SWIGLU ? (vec ? gemm_f32_kernel<true, true> : gemm_f32_kernel<true, false>)
                                       : (vec ? gemm_f32_kernel<false, true> : gemm_f32_kernel<false, false>);
  hipLaunchKernelGGL(kernel, dim3((p.N + 3) / 4, (M + RM - 1) / RM), dim3(256), 0, st, p);
  return hipGetLastError();
}
