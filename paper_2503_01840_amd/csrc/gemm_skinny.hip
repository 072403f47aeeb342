// Weight-streaming bf16 GEMM for few activation rows:  Y[M, N] = X[M, K] * W[N, K]^T, fp32 accumulate.
//
// Every projection of the speculative step (fusion FC, q/k/v, o, gate/up, down, both LM heads) has at
// most a few dozen rows per sequence, so the kernel is bound by reading W once from HBM.  (33..64 rows: the larger matrices
// go through 64-row tiles of gemm_wide.hip.)
//   * one workgroup (4 wavefronts) owns 64 weight rows and one K range (split-K over blockIdx.y);
//   * W is read with 16-byte loads that are contiguous per row (16 lanes = 256 B of one row), staged
//     through registers into a double-buffered, row-padded LDS tile, and read back as MFMA B operands;
//   * X arrives in the fragment-major layout (one 1 KiB block per MFMA A operand), so it is read straight
//     from L2 with perfectly coalesced 16-byte loads and never touches LDS;
//   * the four wavefronts split the K range of a stage (intra-workgroup split-K), each accumulating the
//     whole 64 x 64 tile with v_mfma_f32_32x32x16_bf16; partial tiles are summed through LDS at the end;
//   * PF stages of global loads are kept in flight per wavefront (register prefetch ring).
#include "common.hpp"
#include "kernels.hpp"

namespace {

constexpr int BK = 128;                 // k per stage: 256-byte pieces of a weight row
constexpr int WCH = BK / 32;            // 16-byte weight chunks per thread per stage
constexpr int KSW = BK / 64;            // MFMA k-steps per wavefront per stage
constexpr int CPR = BK / 8;             // 16-byte chunks per weight row per stage
constexpr int BN = 64;                  // weight rows per workgroup
constexpr int WROW = BK * 2 + 16;       // LDS bytes per staged weight row (padded)
constexpr int PF = 4;                   // stages in flight (5 and more spill the prefetch ring to scratch)
constexpr int ROT_MUL = 5;              // stagger of the starting stage from tile to tile
constexpr int RED_LD = 65;              // floats per row of the reduction buffer
constexpr int SMEM_BYTES = 4 * 64 * RED_LD * 4 > 2 * BN * WROW ? 4 * 64 * RED_LD * 4 : 2 * BN * WROW;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// What is behind the arguments that a wavefront has in registers from the start (as one struct with them, behind a memory round trip: together with
// gemm_wide.hip an 8B step 6140 us, 6097 now)
struct GemmParams {
  const bf16_t* w2;
  int rows0, rows1;
  int M, epi;
  float* out_f32;
  bf16_t* out_xf;
};

template <int MH>
__global__ __launch_bounds__(256, 2) void gemm_skinny_kernel(const bf16_t* x, const bf16_t* w0, const bf16_t* w1, int K, int S, int N, int kind, GemmParams p) {
  const int mode = kind & 1, nmat = kind >> 1;         // kind: 2 x matrices + mode
  __shared__ __attribute__((aligned(16))) unsigned char smem[SMEM_BYTES];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int tile = blockIdx.x, split = blockIdx.y, mtile = blockIdx.z;
  const int Kc = K / S, k_begin = split * Kc, KT = Kc / BK;
  auto weight_row = [&](int row) {
    if (mode == 1) {                                   // 32 gate rows | 32 up rows
      const int r = min(tile * 32 + (row & 31), p.rows0 - 1);
      return (row >> 5 ? w1 : w0) + (size_t)r * K;
    }
    int n = min(tile * BN + row, N - 1);
    const bf16_t* w = w0;
    if (nmat > 1 && n >= p.rows0) {
      n -= p.rows0;
      w = w1;
      if (nmat > 2 && n >= p.rows1) { n -= p.rows1; w = p.w2; }
    }
    return w + (size_t)n * K;
  };

  const bf16_t* wptr[WCH];
  int wlds[WCH];
#pragma unroll
  for (int i = 0; i < WCH; ++i) {
    const int c = tid + 256 * i, row = c / CPR, col = c % CPR;
    wptr[i] = weight_row(row) + k_begin + col * 8;
    wlds[i] = row * WROW + col * 16;
  }
  // A-operand blocks of this wavefront: k-steps (k_begin + kt*BK + wave*(BK/4))/16 + {0..KSW-1}, halves 0..MH-1
  const bf16_t* xptr = x + (((size_t)mtile * (K >> 4) + ((k_begin + wave * (BK / 4)) >> 4)) * 2 * 64 + lane) * 8;

  u32x4 wreg[PF][WCH];
  u32x4 xreg[PF][KSW][MH];
  // Workgroups walk their K range from staggered starting stages: with power-of-two row strides, all
  // workgroups reading the same k offset at the same time would hammer the same few HBM channels.
  const int rot = (tile * ROT_MUL + split) % KT;
  auto load_stage = [&](int kt0_, int slot) {
    int kt = kt0_ + rot;
    kt = kt >= KT ? kt - KT : kt;
#pragma unroll
    for (int i = 0; i < WCH; ++i) {
      wreg[slot][i] = *(const u32x4*)(wptr[i] + (size_t)kt * BK);
    }
#pragma unroll
    for (int ks = 0; ks < KSW; ++ks)
#pragma unroll
      for (int mh = 0; mh < MH; ++mh)
        xreg[slot][ks][mh] = *(const u32x4*)(xptr + ((size_t)(kt * (BK / 16) + ks) * 2 + mh) * 512);
  };
  floatx16 acc[MH][2];
#pragma unroll
  for (int mh = 0; mh < MH; ++mh)
#pragma unroll
    for (int nh = 0; nh < 2; ++nh)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mh][nh][r] = 0.f;

  const int b_off = (lane & 31) * WROW + (wave * (BK / 4) + 8 * (lane >> 5)) * 2;
  // One stage: stage `kt`'s weights go from prefetch slot `s` to LDS, its A operands are set aside, the
  // slot is refilled with stage kt + PF (when `refill`), and after the barrier the tile is multiplied.
  auto do_stage = [&](int kt, int s, bool refill) {
    unsigned char* buf = smem + (kt & 1) * (BN * WROW);
#pragma unroll
    for (int i = 0; i < WCH; ++i) *(u32x4*)(buf + wlds[i]) = wreg[s][i];
    u32x4 xc[KSW][MH];
#pragma unroll
    for (int ks = 0; ks < KSW; ++ks)
#pragma unroll
      for (int mh = 0; mh < MH; ++mh) xc[ks][mh] = xreg[s][ks][mh];
    if (refill) load_stage(kt + PF, s);
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < KSW; ++ks)
#pragma unroll
      for (int nh = 0; nh < 2; ++nh) {
        const u32x4 b = *(const u32x4*)(buf + nh * 32 * WROW + b_off + ks * 32);
#pragma unroll
        for (int mh = 0; mh < MH; ++mh)
          acc[mh][nh] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
              __builtin_bit_cast(bf16x8, xc[ks][mh]), __builtin_bit_cast(bf16x8, b), acc[mh][nh], 0, 0, 0);
      }
  };
  // drain: groups whose refills may not all exist (at most the last two groups of a K range)
  auto drain = [&](int kt0) {
    for (; kt0 < KT; kt0 += PF) {
#pragma unroll
      for (int s = 0; s < PF; ++s) {
        const int kt = kt0 + s;
        if (kt < KT) do_stage(kt, s, kt + PF < KT);
      }
    }
  };
  if (KT >= 2 * PF) {
    // Steady state with no branch between the prologue and the loop body, so that the compiler's wait
    // counters stay exact and PF-1 stages of loads remain in flight while one is consumed.
#pragma unroll
    for (int s = 0; s < PF; ++s) {
      load_stage(s, s);
      __builtin_amdgcn_sched_barrier(0);      // keep the issue order: the loop's wait counts depend on it
    }
    int kt0 = 0;
    for (; kt0 + 2 * PF <= KT; kt0 += PF) {
#pragma unroll
      for (int s = 0; s < PF; ++s) do_stage(kt0 + s, s, true);
    }
    drain(kt0);
  } else {
#pragma unroll
    for (int s = 0; s < PF; ++s)
      if (s < KT) load_stage(s, s);
    drain(0);
  }

  // sum the four wavefronts' partial tiles through LDS
  __syncthreads();
  float* red = (float*)smem;
#pragma unroll
  for (int mh = 0; mh < MH; ++mh)
#pragma unroll
    for (int nh = 0; nh < 2; ++nh)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int tok = mh * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        red[(wave * 64 + tok) * RED_LD + nh * 32 + (lane & 31)] = acc[mh][nh][r];
      }
  __syncthreads();
  if (p.epi == GEMM_EPI_PARTIAL) {
#pragma unroll
    for (int e = 0; e < 8 * MH; ++e) {
      const int idx = tid + 256 * e, tok = idx >> 6, f = idx & 63;
      const float v = red[tok * RED_LD + f] + red[(64 + tok) * RED_LD + f] + red[(128 + tok) * RED_LD + f] +
                      red[(192 + tok) * RED_LD + f];
      const int row = mtile * 64 + tok, n = tile * BN + f;
      if (row < p.M && n < N) p.out_f32[((size_t)split * p.M + row) * N + n] = v;
    }
  } else {
    const int I = N >> 1;
#pragma unroll
    for (int e = 0; e < 4 * MH; ++e) {
      const int idx = tid + 256 * e, tok = idx >> 5, f = idx & 31;
      float g = 0.f, u = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        g += red[(w * 64 + tok) * RED_LD + f];
        u += red[(w * 64 + tok) * RED_LD + 32 + f];
      }
      const int row = mtile * 64 + tok, n = tile * 32 + f;
      if (row < p.M && n < I) p.out_xf[xf_offset(row, n, I)] = f32_to_bf16(g / (1.f + expf(-g)) * u);
    }
  }
}

}  // namespace

hipError_t launch_gemm_skinny(const bf16_t* x, const GemmWeights& W, int M, int N, int K, int S, int epi, void* out,
                              hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop) {
  if (M <= 0 || N <= 0 || K <= 0 || S <= 0 || K % (BK * S) != 0) return hipErrorInvalidValue;
  if (epi == GEMM_EPI_SWIGLU && (S != 1 || W.mode != 1)) return hipErrorInvalidValue;
  GemmParams p;
  const bf16_t *w0 = (const bf16_t*)W.w[0], *w1 = (const bf16_t*)W.w[1];
  p.w2 = (const bf16_t*)W.w[2];
  p.rows0 = W.rows[0]; p.rows1 = W.rows[1];
  p.M = M; p.epi = epi;
  const int kind = 2 * W.nmat + W.mode;
  p.out_f32 = (float*)out; p.out_xf = (bf16_t*)out;
  const int tiles = W.mode == 1 ? (N / 2 + 31) / 32 : (N + BN - 1) / BN;
  dim3 grid(tiles, S, (M + 63) / 64);
  if (M <= 32)
    launch_with_events(gemm_skinny_kernel<1>, grid, dim3(256), 0, st, ev_start, ev_stop, x, w0, w1, K, S, N, kind, p);
  else
    launch_with_events(gemm_skinny_kernel<2>, grid, dim3(256), 0, st, ev_start, ev_stop, x, w0, w1, K, S, N, kind, p);
  return hipGetLastError();
}
