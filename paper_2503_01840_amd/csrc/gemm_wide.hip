// bf16 GEMM for MANY activation rows (batched verification: 64 sequences x 8 nodes = 512 rows), and for 33..64 rows where its tiles
// fill the chip:
// Y[M, N] = X[M, K] * W[N, K]^T, fp32 accumulate.  At this width the projections sit at the ridge between weight
// streaming and the MFMA rate, so the kernel is organised around operand reuse and around keeping the loads, the
// LDS reads and the MFMAs of a wavefront all in flight at once:
//   * a workgroup owns a (32 FM WGM) x (16 FB WGN) output tile (FM = 1: the last of its 64-row activation tiles may be half a one); its WGM x WGN wavefronts each hold 2 FM x FB
//     accumulators of v_mfma_f32_16x16x32_bf16 and there is no cross-wavefront reduction.  With many rows the chip is bound by
//     power: products alone sustain 1.88 PFLOP/s as 32x32x16 and 2.14 as 16x16x32 (the sum over 32 k stays inside the matrix
//     unit), with their operands read from LDS 1.64 and 1.86.  With one set of sums they come out bit for bit the same;
//   * both operands reach LDS by direct global-to-LDS loads (global_load_lds_dwordx4: each wavefront
//     instruction deposits 1 KiB contiguously, no staging registers).  A CU accepts roughly one cache line per
//     four clocks whatever its size, so every request is a whole 128-byte line: activations come in 32-k slots
//     (their fragment-major global layout holds every 16-row fragment in one 512-byte run per 16 k, so the copy is verbatim and
//     the LDS reads are linear), weights in BK-wide slots, whole row pieces of 2 BK bytes, and
//     which 16 bytes of its row a lane fetches is XOR-swizzled with the row index so that the MFMA operand reads, 16 rows x
//     one piece, touch every bank once;
//   * one barrier per 32 k.  The barrier of sub-stage h also publishes the data of sub-stage h + 1,
//     so its operand fragments are read into a second set of registers while the products of h run; LDS reads and direct loads
//     are dealt out between the products one by one, so that neither a full load queue nor a burst of reads holds up the matrix
//     pipe (256 x 256 tiles: 2390 cycles per 64 k, of which 2048 are products; 2600 with them in bursts);
//   * the workgroups that share a weight tile (one per 256 activation rows) are launched next to each other on
//     the same XCD, so the tile leaves HBM once; in split products of many activations an XCD has one K range, or two or four, of them all;
//   * the weights are the MFMA's first operand: a lane then holds, for ONE activation row, runs of four
//     consecutive output columns, which is what both epilogues store: fp32 split-K partials (16-byte stores), or
//     SwiGLU (the tile interleaves gate and up rows so that both values of a pair sit in the same lane) written
//     as fragment-major bf16 (8-byte stores).
// 8B width, us, products as 32x32x16 with the reads and loads in bursts / now: 2048 rows gate/up 422 / 368 (1.31 PFLOP/s), down
// 214 / 177, o 77 / 57, q/k/v 100 / 87; 512 rows gate/up 116 / 101, down 73 / 60, q/k/v 39 / 35; 256 rows gate/up 75 / 72 (68
// with 128-k weight stages and staggered walks), 77 rows 61 / 58 (53; 48 in tiles of 96 rows).
// Tiles of 256 x 224 and 256 x 192 (4 x 2 wavefronts of 64 x 112 and 64 x 96) are there for whole rounds of the chip, wide_tiles.hpp says where: 2048
// rows gate/up 371 -> 357 us, q/k/v 92 -> 81, a prompt of 2048 tokens 27.28 -> 26.48 ms; 512 rows gate/up 99.8 -> 98.3 us.
// Measured and not kept: 4 wavefronts of 128 x 128 each (a third fewer LDS reads: loop 4 % shorter, epilogue longer by the same).
//
// SETS: sub-stages add to so many sets of accumulators in turn, so that the sums of a long range of K are as far from 64 bits as with as many
// ranges (28672 x 4096 at 60 rows: 3.95e-7 with one set, 1.88e-7 with four, as in gemm_skinny.hip; 0.1 us a launch).
//
// 33..64 rows stream weights, and of the CU's in-order slots for outstanding lines every activation line takes one like a weight line
// does: tiles of 64 x 128 and 64 x 256 have half and a quarter of an activation line per weight line, where the 64 x 64 tiles of
// gemm_skinny.hip have one.  A workgroup then streams 32 KB of weights in 0.92 us, and 256 of them in 1.44 (5.8 TB/s).
// STAGGER, for them: with a K range of a multiple of 4 KB all workgroups that walk in step ask the same few memory channels, so each
// starts at a stage of its own and goes round.  60 rows, us, 64 x 64 tiles (or 64 x 128 through registers) / in step / staggered:
// gate/up 28672 x 4096 46.4 / 49.5 / 45.9, 57344 x 8192 176 / 176 / 161 (64 x 256), LM head 128256 x 4096 208 / 255 / 194 (64 x 256),
// q/k/v 10240 x 8192 42.9 / 41.6 / 38.6, 5120 x 5120 18.9 / 14.5 / 14.7; but ranges of 7168 and 1024 k: down 8192 x 28672 97.8 / 86.9 /
// 97.9, 12288 x 4096 26.4 / 23.6 / 26.3.
#include <utility>

#include "common.hpp"
#include "kernels.hpp"
#include "wide_places.hpp"
#include "wide_tiles.hpp"

namespace {

// Four neighbours of an output row, which need not start at a multiple of 16 bytes: one store all the same.  So a LM head of any number of
// rows can take the 64-row tiles (128255 x 4096 behind a layer, 60 rows: 342 us, 370 with the workgroups of gemm_skinny.hip).
typedef float row_piece __attribute__((ext_vector_type(4), aligned(4)));

struct WideParams {
  const bf16_t* x;
  const bf16_t* w[3];
  int rows[3];
  int nmat, mode;
  int M, N, K, epi;
  float* out_f32;
  bf16_t* out_xf;
  WideRope rope;
};

// What of it comes behind the arguments that a wavefront has in registers from the start
struct WideRest {
  const bf16_t* w2;
  int rows1, epi;
  float* out_f32;
  bf16_t* out_xf;
  WideRope rope;
};

// Global weight row behind row `row` of workgroup tile `tile` (TN rows per tile).  SwiGLU: every 2 PAIR rows of a tile are PAIR gate
// rows and the PAIR up rows that belong to them.  Rows past the end repeat the last one.
template <int TN, int PAIR, bool ROPE>
__device__ __forceinline__ const bf16_t* weight_row(const WideParams& p, int tile, int row, int& left) {
  if (p.mode == 1) {
    const int r = tile * (TN / 2) + row / (2 * PAIR) * PAIR + row % PAIR, last = p.rows[0] - 1;
    left = max(last - r, 0);
    return ((row & PAIR) ? p.w[1] : p.w[0]) + (size_t)min(r, last) * p.K;
  }
  int n = min(tile * TN + row, p.N - 1);
  left = p.N - 1 - n;
  if (ROPE) {                                          // every 32 rows: 16 of the first half of a head and the 16 they are rotated with
    n = (n & ~127) + (n >> 5 & 3) * 16 + (n & 15) + (n & 16) * 4;
    left = tile * TN + row < p.N ? 7 : 0;              // N is a multiple of 128: a piece's rows (8 or 4) are there, or all of it is behind the end
  }
  const bf16_t* w = p.w[0];
  if (p.nmat > 1 && n >= p.rows[0]) {
    n -= p.rows[0]; w = p.w[1];
    if (p.nmat > 2 && n >= p.rows[1]) { n -= p.rows[1]; w = p.w[2]; }
  }
  return w + (size_t)n * p.K;
}

// One wavefront-wide direct load: lane l's 16 bytes at base + off land at LDS byte address lds_base + AT + 16 l; base is the
// same for the whole wavefront.  The compiler does not see these as memory operations; the kernel counts them itself
// (s_waitcnt vmcnt).
// (m0 carries the LDS address; naming it as clobbered is what is meant, the compiler's remark about reserved
// registers on a clobber list is switched off for this one statement.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int AT>
__device__ __forceinline__ void dma16(const void* base, uint32_t off, uint32_t lds_base) {
  asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_base), "v"(off), "s"(base), "i"(AT)
               : "memory", "m0", "scc");
}
#pragma clang diagnostic pop
// f(0), f(1), ... f(N - 1) with the index as a constant
template <int... I, typename F>
__device__ __forceinline__ void unroll_seq(std::integer_sequence<int, I...>, F f) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, typename F>
__device__ __forceinline__ void unroll(F f) { unroll_seq(std::make_integer_sequence<int, N>{}, f); }
// Own loads but the last n have landed, then everybody's.  No wait for LDS reads: those in flight at a barrier have until
// the next one before their slot is written again, and are used before that.
#define WIDE_WAIT_BARRIER(n) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(n) : "memory")
#define WIDE_PIN() __builtin_amdgcn_sched_barrier(0)

template <int WGM, int WGN, int FM, int FB, int BK, int A_SLOTS, int B_SLOTS, int OCC, bool STAGGER, int SETS, bool ROPE>
__global__ __launch_bounds__(64 * WGM * WGN, OCC) void gemm_wide_kernel(const bf16_t* x, const bf16_t* w0, const bf16_t* w1, int K, int range, int N, int M, int rows0,
                                                                        uint32_t place, uint32_t mblocks_mul, uint32_t stages_mul, WideRest rest) {
  // place: mode, matrices, log2 of the K ranges dealt to XCDs, shifts of the divisors (at most 31): launch_cfg
  const WideParams p = {x, {w0, w1, rest.w2}, {rows0, rest.rows1, 0}, (int)(place >> 1 & 3), (int)(place & 1), M, N, K, rest.epi, rest.out_f32, rest.out_xf, rest.rope};
  constexpr int FA = 2 * FM;                           // 16-row fragments of a wavefront's activation rows; FB: of its weight rows
  constexpr int TM = 32 * FM * WGM, TN = 16 * FB * WGN, NW = WGM * WGN;
  // SwiGLU: gate and up rows in turns of 32, so that both of a pair are accumulators of one lane in two fragments; or, where a wavefront's
  // fragments don't come in fours, in turns of 8, both in one fragment
  constexpr int PAIR = FB % 4 == 0 ? 32 : 8;
  constexpr bool HALF = TM % 64 != 0;                  // the last 64-row activation tile is half a one
  constexpr int SUB = BK / 32;                         // sub-stages of a weight stage
  constexpr int A_SLOT = TM * 64, B_SLOT = TN * BK * 2;              // bytes
  constexpr int B_BASE = A_SLOTS * A_SLOT;
  constexpr int AA = A_SLOTS - 1, BA = B_SLOTS - 1;    // sub-stages and stages that the loads are ahead of the products
  // direct-to-LDS instructions (1 KiB each) per wavefront per activation / weight slot; a weight slot goes out in SUB parts
  // (192 rows over 8 wavefronts: 12 activation pieces; the last four wavefront-instructions repeat pieces, so that every
  // wavefront has the same number of loads in flight)
  constexpr int A_PIECES = A_SLOT / 1024, A_DMA = (A_PIECES + NW - 1) / NW;
  // (224 rows: 28 weight pieces, four for each of the first B_FULL = 4 wavefronts and three for the others; the waits below count the fewer)
  constexpr int B_PIECES = B_SLOT / 1024, B_DMA = (B_PIECES + NW - 1) / NW, B_FULL = B_PIECES - NW * (B_DMA - 1), BP = (B_DMA + SUB - 1) / SUB;
  constexpr int B_LANES = BK / 8, B_ROWS = 64 / B_LANES;           // lanes to a row of a weight piece, rows of a piece
  static_assert((BK == 64 || BK == 128) && B_FULL > 0 && TM % 32 == 0, "1 KiB pieces per wavefront");
  static_assert(FM == 1 || (!HALF && (WGM == 2 || FM == 2)), "a wavefront's 32-row blocks are one, one of every pair, or two neighbours");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;

  const WidePlace at = wide_place(blockIdx.x, blockIdx.y, place >> 3 & 3, Divisor{mblocks_mul, place >> 10 & 31, (int)((unsigned)(M + TM - 1) / TM)});
  const int tile = at.tile, mblock = at.mblock, split = at.split;
  if (tile >= (N + TN - 1) / TN) return;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  const int k_begin = split * range, KT = (unsigned)range / BK;   // KT weight stages = SUB KT sub-stages
  const int MT = (p.M + 63) >> 6;                      // 64-row activation tiles that exist

  // ---- global sources: one address per piece for the wavefront, and the place in K as part of the lanes' offsets.  Piece q of
  // an activation slot is (row tile q / 4, k-step (q / 2) % 2, row half q % 2); piece q of a weight slot is rows
  // B_ROWS q .. B_ROWS (q + 1) - 1.
  constexpr auto swizzle = [](int row) constexpr { return BK == 64 ? (row >> 1) & 7 : row & 15; };   // of the 16-byte pieces of a weight row
  const int b_first = wave < B_FULL ? wave * B_DMA : wave * (B_DMA - 1) + B_FULL;
  const bf16_t* aptr[A_DMA];
  const bf16_t* bptr[B_DMA];
  uint32_t a_off = lane * 16, b_off[B_DMA];
  int a_first = wave * A_DMA;
  if (A_PIECES < A_DMA * NW && a_first >= A_PIECES) a_first -= A_DMA * NW - A_PIECES;
#pragma unroll
  for (int i = 0; i < A_DMA; ++i) {
    const int q = a_first + i, rt = min(mblock * (TM / 64) + (q >> 2), MT - 1);
    const bool half = HALF && q >= TM / 64 * 4;                      // its two pieces are the k-steps of row half 0
    aptr[i] = p.x + (((size_t)rt * (p.K >> 4) + (k_begin >> 4) + (half ? q & 1 : (q >> 1) & 1)) * 2 + (half ? 0 : q & 1)) * 512;
  }
#pragma unroll
  for (int i = 0; i < B_DMA; ++i) {
    const int row = B_ROWS * (b_first + i), r = lane / B_LANES;
    int left;                                          // rows behind this one
    bptr[i] = weight_row<TN, PAIR, ROPE>(p, tile, row, left) + k_begin;
    b_off[i] = (uint32_t)min(r, left) * (uint32_t)p.K * 2 + (((lane % B_LANES) ^ swizzle(row + r)) * 16);
  }
  const uint32_t a_lds = lds0 + a_first * 1024, b_lds = lds0 + B_BASE + b_first * 1024;
  // Each piece of a (sub-)stage, then a step along K.  Past the end of the walk the last one is loaded again, into a
  // slot nobody reads any more, which keeps the number of loads in flight, and with it the waits below, the same in every iteration.
  auto load_a = [&](auto i, uint32_t slot) { dma16<i * 1024>(aptr[i], a_off, a_lds + slot); };
  auto load_b = [&](auto i, uint32_t slot) {
    if (i < B_DMA - 1 || B_FULL == NW || wave < B_FULL) dma16<i * 1024>(bptr[i], b_off[i], b_lds + slot);
  };
  const int rot = STAGGER ? (tile * 5 + split) % Divisor{stages_mul, place >> 5 & 31, KT} : 0;
  if (STAGGER) {
    a_off += rot * SUB * 4096u;
#pragma unroll
    for (int i = 0; i < B_DMA; ++i) b_off[i] += rot * (2u * BK);
  }
  // to sub-stage v (stage t) of the walk, from the one before it
  auto step_a = [&](int v) { a_off += v >= SUB * KT ? 0u : STAGGER && v == SUB * (KT - rot) ? 4096u - SUB * KT * 4096u : 4096u; };
  auto step_b = [&](auto i, int t) { b_off[i] += t >= KT ? 0u : STAGGER && t == KT - rot ? 2u * BK - KT * 2u * BK : 2u * BK; };

  // ---- operand fragments (16 rows x 32 k: lane l holds row l % 16, k 8 (l / 16) .. + 7) inside their slots.  The 32-row
  // blocks of a wavefront: one of every pair (WGM = 2), so that their distances are constants, or two neighbours.
  const int c = lane >> 4;
  const int a_base = (c >> 1) * (HALF && wm == WGM - 1 ? 1024 : 2048) + (c & 1) * 512 + (lane & 15) * 16 +
                     (FM == 1 ? (wm >> 1) * 4096 + (wm & 1) * 1024 : WGM == 2 ? wm * 1024 : wm * 4096);
  constexpr auto a_frag = [](int i) constexpr { return WGM == 2 ? (i >> 1) * 4096 + (i & 1) * 256 : (i >> 1) * 1024 + (i & 1) * 256; };
  // PAIR = 8: a lane's accumulators r = 0, 1 are gate rows and 2, 3 their up rows, so product row 4 a + r is row 2 a + r or 8 + 2 a + r - 2
  const int b_row = PAIR == 8 && p.mode == 1 ? (lane & 2) * 4 + (lane >> 1 & 6) + (lane & 1) : lane & 15;
  int b_base[SUB];
#pragma unroll
  for (int q = 0; q < SUB; ++q) b_base[q] = B_BASE + (wn * 16 * FB + b_row) * (BK * 2) + (((4 * q + c) ^ swizzle(b_row)) * 16);

  floatx4 sums[SETS][FA][FB];                          // sub-stage v adds to set v % SETS
  floatx4(&acc)[FA][FB] = sums[0];

  // Loads complete in issue order.  Sub-stage v = SUB s + q issues every piece of activation sub-stage v + AA, then part q of the
  // pieces of weight stage s + BA; the sub-stages before the first one issue what has begun by then.
  constexpr int LEAD = ((AA > SUB * BA ? AA : SUB * BA) + SUB - 1) / SUB * SUB;
  unroll<LEAD>([&](auto u) {
    constexpr int v = u - LEAD, q = u % SUB, t = u / SUB - LEAD / SUB + BA;
    if constexpr (v + AA >= 0) {
      unroll<A_DMA>([&](auto i) { load_a(i, (v + AA) * A_SLOT); });
      step_a(v + AA + 1);
    }
    if constexpr (t >= 0)
      unroll<BP>([&](auto j) {
        constexpr std::integral_constant<int, q * BP + j> i;
        if constexpr (i < B_DMA) {
          load_b(i, t * B_SLOT);
          step_b(i, t + 1);
        }
      });
  });
#pragma unroll
  for (int j = 0; j < SETS; ++j)
#pragma unroll
    for (int i = 0; i < FA; ++i)
#pragma unroll
      for (int f = 0; f < FB; ++f)
#pragma unroll
        for (int r = 0; r < 4; ++r) sums[j][i][f][r] = 0.f;
  constexpr int PER = A_DMA + BP;                      // loads per sub-stage, at most
  // fewest loads of a wavefront in sub-stage u: weights, and all of sub-stages from .. to - 1
  constexpr auto part = [](int u) constexpr {
    const int q = (u % SUB + SUB) % SUB, rest = B_DMA - (B_FULL < NW ? 1 : 0) - q * BP;
    return rest < 0 ? 0 : rest < BP ? rest : BP;
  };
  constexpr auto loads = [part](int from, int to) constexpr {
    int n = 0;
    for (int u = from; u < to; ++u) n += A_DMA + part(u);
    return n;
  };
  constexpr auto least = [](int x, int y) constexpr { return x < y ? x : y; };
  WIDE_WAIT_BARRIER(least(part(-AA) + loads(1 - AA, 0), loads(-SUB * (BA - 1), 0)));   // A0 and B0 are in LDS
  bf16x8 a0[FA], a1[FA], b0[FB], b1[FB];
#pragma unroll
  for (int i = 0; i < FA; ++i) a0[i] = *(const bf16x8*)(smem + a_base + a_frag(i));
#pragma unroll
  for (int f = 0; f < FB; ++f) b0[f] = *(const bf16x8*)(smem + b_base[0] + f * (32 * BK));

  // One sub-stage: a and b hold its fragments; an and bn receive those of the next.  A fragment of weights stays the first
  // operand of FA products in a row: with the operands the other way round the matrix units draw more power, which costs
  // clock.  The direct loads and LDS reads are dealt out between the products, no two together, so that none of
  // them keeps a product from being issued.
  uint32_t b_slot = 0;                                 // of weight stage s
  auto sub_stage = [&](int s, auto q, auto set, const bf16x8 (&a)[FA], const bf16x8 (&b)[FB], bf16x8 (&an)[FA], bf16x8 (&bn)[FB]) {
    const int h = SUB * s + q;
    // everything up to A(h+1) and, in the last sub-stage, B(s+1) has landed when only the loads issued after it are in
    // flight: what the NEXT sub-stage reads is in LDS from here on, and the slots of sub-stage h - 1 are free
    constexpr int behind_a = part(q + 1 - AA) + loads(q + 2 - AA, q), behind_b = loads(q + 1 - SUB * (BA - 1), q);
    WIDE_WAIT_BARRIER(q < SUB - 1 ? behind_a : least(behind_a, behind_b));
    WIDE_PIN();
    const uint32_t b_next = b_slot == BA * B_SLOT ? 0 : b_slot + B_SLOT, b_fill = b_slot == 0 ? BA * B_SLOT : b_slot - B_SLOT;   // of s + 1, s + BA
    const uint32_t a_fill = (uint32_t)(h + AA) % A_SLOTS * A_SLOT;
    const unsigned char* as = smem + (uint32_t)(h + 1) % A_SLOTS * A_SLOT + a_base;
    const unsigned char* bs = smem + (q < SUB - 1 ? b_slot : b_next) + b_base[(q + 1) % SUB];
    unroll<FA * FB>([&](auto x) {
      constexpr int MF = FA * FB, NR = FA + FB;
      constexpr int f = x / FA, i = x % FA;
      sums[set][i][f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[f], a[i], sums[set][i][f], 0, 0, 0);
      // the reads in the order in which the next sub-stage needs them: b 0, every a, the rest of b
      constexpr int r = (x * NR + MF - 1) / MF;        // read r goes behind product r MF / NR
      if constexpr (r < NR && r * MF / NR == x) {
        if constexpr (r == 0) bn[0] = *(const bf16x8*)bs;
        else if constexpr (r <= FA) an[r - 1] = *(const bf16x8*)(as + a_frag(r - 1));
        else bn[r - FA] = *(const bf16x8*)(bs + (r - FA) * (32 * BK));
      }
      constexpr int at = x - 1, d = (at * PER + MF - 1) / MF;  // load d behind product d MF / PER + 1
      if constexpr (at >= 0 && d < PER && d * MF / PER == at) {
        if constexpr (d < A_DMA) {
          load_a(std::integral_constant<int, d>{}, a_fill);
          if constexpr (d == A_DMA - 1) step_a(h + AA + 1);
        } else {
          constexpr std::integral_constant<int, q * BP + d - A_DMA> piece;
          if constexpr (piece < B_DMA) {
            load_b(piece, b_fill);
            step_b(piece, s + BA + 1);
          }
        }
      }
      WIDE_PIN();
    });
    if (q == SUB - 1) b_slot = b_next;
  };
  auto stage = [&](int s, auto first) {                // first: the set of its first sub-stage
    unroll<SUB / 2>([&](auto q) {
      sub_stage(s, std::integral_constant<int, 2 * q>{}, std::integral_constant<int, (first + 2 * q) % SETS>{}, a0, b0, a1, b1);
      sub_stage(s, std::integral_constant<int, 2 * q + 1>{}, std::integral_constant<int, (first + 2 * q + 1) % SETS>{}, a1, b1, a0, b0);
    });
  };
  constexpr int STEP = SETS > SUB ? SETS / SUB : 1;    // stages until the sets come round
  int s = 0;
  for (; s + STEP <= KT; s += STEP) unroll<STEP>([&](auto t) { stage(s + t, std::integral_constant<int, t * SUB>{}); });
  unroll<STEP - 1>([&](auto t) {
    if (s + t < KT) stage(s + t, std::integral_constant<int, t * SUB>{});
  });
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // nothing may still be writing LDS when the workgroup ends
  unroll<SETS == 1 ? 0 : SETS == 2 ? 1 : 2>([&](auto n) {               // 4 sets: 0 + 2 and 1 + 3, then both
    constexpr int half = SETS >> (n + 1);
    unroll<half>([&](auto j) {
#pragma unroll
      for (int i = 0; i < FA; ++i)
#pragma unroll
        for (int f = 0; f < FB; ++f) sums[j][i][f] += sums[j + half][i][f];
    });
  });

  // ---- epilogue.  Accumulator r of lane l: activation row l % 16 of its fragment, weight row 4 (l / 16) + r of its own.
  auto row_of = [&](int i) { return mblock * TM + (FM == 1 ? wm * 32 : WGM == 2 ? (i >> 1) * 64 + wm * 32 : wm * 64 + (i >> 1) * 32) + (i & 1) * 16 + (lane & 15); };
  if constexpr (ROPE) {
    // Fragments 2 j and 2 j + 1 hold dimensions i .. i + 3 and i + 64 .. i + 67 of the same head: rotated (q, k), and straight to q or the cache.
    const WideRope& rp = p.rope;
#pragma unroll
    for (int i = 0; i < FA; ++i) {
      const int m = row_of(i);
      if (m >= p.M) continue;
      const float* cs = rp.cs + (size_t)m * rp.cs_step;
      const size_t slot = (size_t)rp.slot[m];
#pragma unroll
      for (int f = 0; f < FB; f += 2) {
        const int n = tile * TN + wn * 16 * FB + f * 16;
        if (n >= p.N) continue;
        const int head = n >> 7, d = (n >> 5 & 3) * 16 + 4 * c;
        floatx4 x1 = acc[i][f], x2 = acc[i][f + 1];
        if (head < rp.H + rp.Hkv) {
          const floatx4 co = *(const floatx4*)(cs + d), si = *(const floatx4*)(cs + 64 + d);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float a = x1[e], b = x2[e];
            x1[e] = a * co[e] - b * si[e];
            x2[e] = b * co[e] + a * si[e];
          }
        }
        bf16_t* dst = head < rp.H             ? rp.q + ((size_t)m * rp.H + head) * 128
                      : head < rp.H + rp.Hkv ? rp.kc + (slot * rp.Hkv + head - rp.H) * 128
                                             : rp.vc + (slot * rp.Hkv + head - rp.H - rp.Hkv) * 128;
        store4_plain(dst, d, x1[0], x1[1], x1[2], x1[3]);
        store4_plain(dst, d + 64, x2[0], x2[1], x2[2], x2[3]);
      }
    }
  } else if (p.epi == GEMM_EPI_PARTIAL) {
    float* out = p.out_f32 + (size_t)split * p.M * p.N;
#pragma unroll
    for (int i = 0; i < FA; ++i) {
      const int m = row_of(i);
      if (m >= p.M) continue;
#pragma unroll
      for (int f = 0; f < FB; ++f) {
        const int n = tile * TN + wn * 16 * FB + f * 16 + 4 * c;
        float* dst = out + (size_t)m * p.N + n;
        if (n + 4 <= p.N) *(row_piece*)dst = acc[i][f];
        else
#pragma unroll
          for (int r = 0; r < 3; ++r)
            if (n + r < p.N) dst[r] = acc[i][f][r];
      }
    }
  } else {
    const int I = p.N >> 1;
#pragma unroll
    for (int i = 0; i < FA; ++i) {
      const int m = row_of(i);
      if (m >= p.M) continue;
      auto swiglu = [](float g, float u) { return g / (1.f + expf(-g)) * u; };
      if constexpr (PAIR == 8) {
#pragma unroll
        for (int f = 0; f < FB; ++f) {
          const int n = tile * (TN / 2) + (wn * FB + f) * 8 + 2 * c;
          if (n >= I) continue;
          *(uint32_t*)(p.out_xf + xf_offset(m, n, I)) = pack_bf16x2(swiglu(acc[i][f][0], acc[i][f][2]), swiglu(acc[i][f][1], acc[i][f][3]));
        }
      } else {
#pragma unroll
        for (int f = 0; f < FB / 2; ++f) {             // fragments of gate rows: two of every four
          const int n = tile * (TN / 2) + wn * 8 * FB + f * 16 + 4 * c, gf = (f >> 1) * 4 + (f & 1);
          if (n >= I) continue;
          float h[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) h[e] = swiglu(acc[i][gf][e], acc[i][gf + 2][e]);
          Act<true>::store4(p.out_xf, m, n, I, h[0], h[1], h[2], h[3]);
        }
      }
    }
  }
}

template <int WGM, int WGN, int FM, int FB, int BK, int A_SLOTS, int B_SLOTS, int OCC, bool STAGGER = false, int SETS = 1, bool ROPE = false>
hipError_t launch_cfg(WideParams& p, int S, hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop) {
  constexpr int TM = 32 * FM * WGM, TN = 16 * FB * WGN;
  constexpr int LDS = A_SLOTS * TM * 64 + B_SLOTS * TN * BK * 2;
  auto kernel = gemm_wide_kernel<WGM, WGN, FM, FB, BK, A_SLOTS, B_SLOTS, OCC, STAGGER, SETS, ROPE>;
  static DeviceOnce configured;                        // the attribute belongs to the loaded code object of a device
  hipError_t ce = configured.run([&] { return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, LDS); });
  if (ce != hipSuccess) return ce;
  const int tiles = (p.N + TN - 1) / TN;
  const int ranges = dealt_ranges(p.M, p.K, S);
  const Divisor by_mblocks = divisor((p.M + TM - 1) / TM), by_stages = divisor(p.K / S / BK);
  const WideGrid grid = wide_grid(tiles, by_mblocks.d, S, ranges);
  const uint32_t place = (uint32_t)p.mode | (uint32_t)p.nmat << 1 | (uint32_t)ranges << 3 | by_stages.shift << 5 | by_mblocks.shift << 10;
  const WideRest rest = {p.w[2], p.rows[1], p.epi, p.out_f32, p.out_xf, p.rope};
  launch_with_events(kernel, dim3(grid.x, grid.y), dim3(64 * WGM * WGN), LDS, st, ev_start, ev_stop, p.x, p.w[0], p.w[1], p.K, p.K / S, p.N, p.M, p.rows[0], place,
                     by_mblocks.mul, by_stages.mul, rest);
  return hipGetLastError();
}

}  // namespace

namespace {

hipError_t fill_params(WideParams& p, const bf16_t* x, const GemmWeights& W, int M, int N, int K, int epi, void* out) {
  if (M <= 0 || N <= 0 || K <= 0 || K % 64) return hipErrorInvalidValue;
  if (epi == GEMM_EPI_SWIGLU ? (W.mode != 1 || N % 8) : W.mode != 0) return hipErrorInvalidValue;
  for (int i = 0; W.mode == 0 && i + 1 < W.nmat; ++i)
    if (W.rows[i] % 8) return hipErrorInvalidValue;    // the rows of one direct load belong to one matrix
  p.x = x;
  for (int i = 0; i < 3; ++i) { p.w[i] = (const bf16_t*)W.w[i]; p.rows[i] = W.rows[i]; }
  p.nmat = W.nmat; p.mode = W.mode;
  p.M = M; p.N = N; p.K = K; p.epi = epi;
  p.out_f32 = (float*)out; p.out_xf = (bf16_t*)out;
  return hipSuccess;
}

}  // namespace

// Picks the tile shape and the split-K factor, then launches.
hipError_t launch_gemm_wide(const bf16_t* x, const GemmWeights& W, int M, int N, int K, int epi, void* out,
                            size_t out_capacity_floats, int* S_out, hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop) {
  WideParams p;
  if (N % 4) return hipErrorInvalidValue;
  if (hipError_t e = fill_params(p, x, W, M, N, K, epi, out)) return e;
  const WideTiles t = many_tiles(M, N, K, epi == GEMM_EPI_SWIGLU, out_capacity_floats);
  if (S_out) *S_out = t.S;
  // Staggered walks (see above) also up to 256 rows.  us, in step / staggered: gate/up 28672 x 4096 77 rows 55.4 / 51.6, 256 rows 75.6 / 72.8,
  // LM head 128256 x 4096 77 rows 252 / 227, 256 rows 329 / 302, 8192 x 8192 in four ranges 77 rows 35.0 / 30.6, 256 rows 48.9 / 49.3; stages of
  // 64 k, LM head 252 / 210, but 8192 x 28672 in seven ranges 115 / 132; and 0 to 8 % slower at 512 and 2048 rows.
  const bool stagger = wide_stagger(M, K, t);
  // Two chains of sums where a range of K is longer than the one that the same rows had before these tiles: 128 x 128 with 128-k stages (q/k/v
  // 6144 x 4096 at 116 rows four ranges instead of eight: error 1.37e-7, 1.89e-7 with one chain; and 2 to 3 % faster, in 198 registers
  // instead of 176 and 88 accumulators), and 256 x 128 above 256 rows (512 rows two ranges instead of four: 1.88e-7, 2.72e-7 with one; 1 % slower).
  if (t.cols == 128 && t.k == 128) {
    if (t.rows == 96)
      return stagger ? launch_cfg<3, 2, 1, 4, 128, 8, 3, 1, true, 2>(p, t.S, st, ev_start, ev_stop)
                     : launch_cfg<3, 2, 1, 4, 128, 8, 3, 1, false, 2>(p, t.S, st, ev_start, ev_stop);
    if (t.rows == 256 && M > 256) return launch_cfg<4, 2, 2, 4, 128, 4, 3, 1, false, 2>(p, t.S, st, ev_start, ev_stop);
    if (t.rows == 256)
      return stagger ? launch_cfg<4, 2, 2, 4, 128, 4, 3, 1, true>(p, t.S, st, ev_start, ev_stop)
                     : launch_cfg<4, 2, 2, 4, 128, 4, 3, 1>(p, t.S, st, ev_start, ev_stop);
    return stagger ? launch_cfg<2, 2, 2, 4, 128, 4, 3, 2, true, 2>(p, t.S, st, ev_start, ev_stop)
                   : launch_cfg<2, 2, 2, 4, 128, 4, 3, 2, false, 2>(p, t.S, st, ev_start, ev_stop);
  }
  if (t.cols == 128) {
    if (t.rows == 256) return launch_cfg<4, 2, 2, 4, 64, 4, 3, 1>(p, t.S, st, ev_start, ev_stop);
    return launch_cfg<2, 2, 2, 4, 64, 4, 3, 2>(p, t.S, st, ev_start, ev_stop);        // never staggered: stream_tiles
  }
  if (t.cols == 224) return launch_cfg<4, 2, 2, 7, 64, 4, 3, 1>(p, t.S, st, ev_start, ev_stop);
  if (t.cols == 192) return launch_cfg<4, 2, 2, 6, 64, 4, 3, 1>(p, t.S, st, ev_start, ev_stop);
  if (t.rows == 96)
    return stagger ? launch_cfg<3, 2, 1, 8, 64, 8, 3, 1, true, 2>(p, t.S, st, ev_start, ev_stop)
                   : launch_cfg<3, 2, 1, 8, 64, 8, 3, 1, false, 2>(p, t.S, st, ev_start, ev_stop);
  if (t.rows == 128)
    return stagger ? launch_cfg<2, 4, 2, 4, 64, 6, 3, 1, true, 2>(p, t.S, st, ev_start, ev_stop)
                   : launch_cfg<2, 4, 2, 4, 64, 6, 3, 1, false, 2>(p, t.S, st, ev_start, ev_stop);
  if (t.rows == 256)
    return stagger ? launch_cfg<2, 4, 4, 4, 64, 4, 3, 1, true>(p, t.S, st, ev_start, ev_stop)
                   : launch_cfg<2, 4, 4, 4, 64, 4, 3, 1>(p, t.S, st, ev_start, ev_stop);
  return stagger ? launch_cfg<2, 4, 3, 4, 64, 4, 3, 1, true>(p, t.S, st, ev_start, ev_stop)
                 : launch_cfg<2, 4, 3, 4, 64, 4, 3, 1>(p, t.S, st, ev_start, ev_stop);
}

// q/k/v of more than 256 rows, rotated and in their places, where the product is not split and its tile has fragments in pairs.  As 50 MB of fp32 results
// and a kernel of its own that read them (rope_kv_write_kernel, whose arithmetic this is) the rotation of 2048 rows of 6144 took 16 us of a layer's 850,
// here the product takes 2 longer: 2048 tokens 26.08 -> 25.65 ms.  224 weight rows have seven fragments to a wavefront, and 128 x 128 tiles are few
// enough rows for the kernel: they stay with it.
bool wide_rope_fits(int M, int N, int K, size_t out_capacity_floats) {
  if (M <= 256 || N % 128) return false;
  const WideTiles t = launch_tiles(M, N, K, false, out_capacity_floats);
  return t.S == 1 && t.cols != 224 && (t.cols != 128 || (t.rows == 256 && t.k == 128));
}
hipError_t launch_gemm_wide_rope(const bf16_t* x, const GemmWeights& W, int M, int N, int K, const WideRope& rope, size_t out_capacity_floats,
                                 hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop) {
  WideParams p;
  if (!wide_rope_fits(M, N, K, out_capacity_floats)) return hipErrorInvalidValue;
  if (hipError_t e = fill_params(p, x, W, M, N, K, GEMM_EPI_PARTIAL, nullptr)) return e;
  p.rope = rope;
  const WideTiles t = launch_tiles(M, N, K, false, out_capacity_floats);
  if (t.cols == 192) return launch_cfg<4, 2, 2, 6, 64, 4, 3, 1, false, 1, true>(p, 1, st, ev_start, ev_stop);
  if (t.cols == 128) return launch_cfg<4, 2, 2, 4, 128, 4, 3, 1, false, 2, true>(p, 1, st, ev_start, ev_stop);
  return t.rows == 256 ? launch_cfg<2, 4, 4, 4, 64, 4, 3, 1, false, 1, true>(p, 1, st, ev_start, ev_stop)
                       : launch_cfg<2, 4, 3, 4, 64, 4, 3, 1, false, 1, true>(p, 1, st, ev_start, ev_stop);
}

// At most 64 rows, in tiles of 64 x cols.
hipError_t launch_gemm_wide64(const bf16_t* x, const GemmWeights& W, int M, int N, int K, int cols, int S, int epi, void* out,
                              hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop) {
  WideParams p;
  if (hipError_t e = fill_params(p, x, W, M, N, K, epi, out)) return e;
  if (M > 64 || S < 1 || (cols != 128 && cols != 256) || K % (S * (cols == 128 ? 128 : 64)) || (epi == GEMM_EPI_SWIGLU && S != 1))
    return hipErrorInvalidValue;
  const bool stagger = few_rows_stagger(K, S);
  if (cols == 128)
    return stagger ? launch_cfg<2, 2, 1, 4, 128, 5, 3, 2, true, 4>(p, S, st, ev_start, ev_stop)
                   : launch_cfg<2, 2, 1, 4, 128, 5, 3, 2, false, 4>(p, S, st, ev_start, ev_stop);
  return stagger ? launch_cfg<2, 4, 1, 4, 64, 8, 4, 1, true, 4>(p, S, st, ev_start, ev_stop)
                 : launch_cfg<2, 4, 1, 4, 64, 8, 4, 1, false, 4>(p, S, st, ev_start, ev_stop);
}
