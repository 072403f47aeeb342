// Causal attention of a run of consecutive positions (forward only): a prefill chunk against its sequence's cache, and the
// draft layer's self-attention during a training-time-test step.
//
// Simulated step s over a training sequence of T positions: query i sees the ORIGINAL positions 0..i (ordinary
// causal context) and, of every simulated step t = 1..s, only position i itself.  The causal part is a flash-style
// pass over the original keys with the matrix cores; the s extra keys of a query are handled as the per-position
// vector dot products they are (one key per query and step: a matrix product would compute T x T scores to keep T).
//
// bf16 kernel (head_dim 128).  A workgroup owns 128 query rows of one KV head: HG (1, 2 or 4) of the query heads that
// share it x 128 / HG consecutive queries, so that every K/V tile it stages serves all of them.  8 wavefronts = 4 groups
// of 32 rows x 2 halves of every 128-key tile; a wavefront takes the first and third or the second and fourth of the tile's
// 32-key blocks, so that both are done early where the last tile ends after 64 keys.  (Where the chip would not be
// full: 64 rows, 4 wavefronts.)
//   * Tiles reach LDS by direct global-to-LDS loads, both K and V two tiles ahead, swizzled per key; K has two slots and V three,
//     as its values are read one block later than its scores; scores are
//     produced transposed (S^T = K Q^T) so that a lane owns one query; the V^T operand comes from the transposing LDS
//     read; exp(S) enters the value product as a bf16 head plus a bf16 tail.
//   * One block is a matrix-unit time of 24 products (8 score + 16 value, 768 cycles) against ~700 issue cycles of everything else (4 a vector
//     instruction, 8 an exponential or a product).  Run one after the other they add up (all wavefronts pass the same barrier, so they stay in
//     phase); here the softmax of block i runs between the score products of block i + 1 and the value products of block i - 1, none of which
//     depend on it, its last four weights a block later, so that both halves of a block have about as much to issue as to multiply.  One v_dot2 for every
//     two weights among them and no more, as they stop the matrix unit, and the direct loads one by one: 85 k -> 70 k cycles for 16 tiles, of which 50 k are products.
//   * Only tiles that reach past a workgroup's first query need a mask.
//   * The own keys of the simulated steps come last; their rows arrive while the last block is worked on.
//   * Workgroups of later queries walk over more keys: they are handed out first, and the KV head is the fastest index,
//     so that with 8 KV heads each XCD keeps one head's keys in its L2.
// What bounds it: the chip's power where every CU has two workgroups and more (at T = 2048, 32 heads over 8, the clock in the loop is 1.9 GHz,
// and was 2.15 with the 18 % more cycles), and the walk of the longest workgroup with its start, own keys and merge where there are fewer.  A workgroup has all of a CU's LDS, so that these
// never run under another one's tiles: of 58 us at T = 2048 with s = 2 some 39 are tiles (17 to a CU, by the cycles above).  The softmax
// must stay in the gaps it is written into: with the sum of the weights formed behind the block, copies between registers, a last
// tile taken whole and the output rescaled at every own key it was 29.0 instead of 22.6 us (T = 517, 64 heads, s = 5), 72 instead
// of 67 (T = 2048, 32 heads over 8, s = 5) and 36.0 instead of 32.6 (T = 2048, 8 heads, s = 0).  Measured against a kernel of one head x 64 queries per workgroup (4 wavefronts, scores,
// softmax and values one after the other, own keys read from global memory by every lane for itself): T = 2048, s = 2:
// 108 -> 65 us; T = 517, 64 heads, s = 5: 61 -> 22.6 us.  Then with the weights' tails by plain instructions, the softmax and the direct loads dealt out and no divisions in front
// of the first load, before / now: T = 2048 s = 2 60.5 -> 57.2, T = 4096 s = 1 207 -> 192, T = 1000 s = 3 27.8 -> 24.9, T = 517 s = 5 21.9 -> 19.7, T = 300 s = 1 10.8 -> 9.8.
// fp32 kernel: one workgroup per (query, head), exact arithmetic, for small checks.
#include <algorithm>

#include "causal_rules.hpp"
#include "common.hpp"
#include "kernels.hpp"

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef short short8v __attribute__((ext_vector_type(8)));
constexpr int D = 128;
constexpr int KT = CAUSAL_KEYS;               // keys per tile: two halves of two 32-key blocks
constexpr int ROWB = D * 2;
constexpr int TILE_BYTES = KT * ROWB;         // of K, and again of V
constexpr int V_BASE = 2 * TILE_BYTES;        // two K slots, then three V slots: all of a CU's 160 KB
constexpr int LDS_BYTES = 5 * TILE_BYTES;
constexpr int Q_BASE = 4 * TILE_BYTES;        // the queries, staged in the third V slot before it is used
constexpr int STAGE_BASE = 8 * 34 * 64 * 4;   // at the end: the exchange of the key halves, then 8 KB per wavefront

constexpr float NEG = -1e30f;
constexpr float MAX_SLACK = 8.f;

struct CausalParams {
  const bf16_t* q;        // [T, H, D]
  const bf16_t* k;        // training: [s+1, T, Hkv, D]; prefill: the cache [slots, Hkv, D]
  const bf16_t* v;
  const SeqInfo* seq;     // prefill: kv_base and n_prefix of the sequence
  int T, H, Hkv, s;
  int hg, qb_log2, n_qblocks, G;    // query heads per workgroup, log2 of its queries, query blocks, query heads per KV head
  Divisor by_groups, by_kv_heads;   // KV heads x head groups; KV heads
  float scale_log2;
  bool q_aligned;         // to 16 bytes
  void* out;              // training: fp32 [T, H, D]; prefill: fragment-major bf16 [T, H * D]
};

__device__ __forceinline__ void pair_values(float x, float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}

// One wavefront-wide direct load: lane l's 16 bytes at base + lane_off land at LDS byte address lds_base + 16 l.  The
// compiler does not see these as memory operations; the kernel counts them itself (s_waitcnt vmcnt).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma16(const void* base, uint32_t lane_off, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_base), "v"(lane_off), "s"(base)
               : "memory", "m0");
}
#pragma clang diagnostic pop
#define CAUSAL_PIN() __builtin_amdgcn_sched_barrier(0)
#define CAUSAL_WAIT_LOADS(n) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(n) : "memory")

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }
// LDS reads at a byte address
__device__ __forceinline__ u32x4 read_lds(uint32_t a) { return *(const u32x4 __attribute__((address_space(3)))*)a; }
__device__ __forceinline__ short4v read_tr(uint32_t a) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((short4v __attribute__((address_space(3)))*)a);
}
__device__ __forceinline__ floatx16 mfma(const u32x4& a, const u32x4& b, const floatx16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

#define INLINE_LAMBDA __attribute__((always_inline))

template <bool V> struct Flag { static constexpr bool value = V; };

// PREFILL: query i sits at position n_prefix + i of a sequence in the cache, whose earlier positions it sees as well.
// RG: 32-row groups per workgroup.
template <bool PREFILL, int RG>
__global__ __launch_bounds__(128 * RG) void causal_attn_bf16_kernel(CausalParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int NW = 2 * RG, ROWS_WG = 32 * RG;
  constexpr int IPW = 32 / NW;                               // direct loads per wavefront per tile, for K and again for V
  constexpr int IPW_ROWS = ROWS_WG / 4 / NW;                 // and for one row of each of the workgroup's queries
  const int rg = wave % RG, sb = wave / RG;                  // row group, key half
  const int kg = lane >> 5;
  const int gh = (int)blockIdx.x % p.by_groups;
  const int qb = p.n_qblocks - 1 - (int)blockIdx.x / p.by_groups;
  const int first_head = gh % p.by_kv_heads * p.G + gh / p.by_kv_heads * p.hg, g = gh % p.by_kv_heads;
  const int QB = 1 << p.qb_log2;                             // queries per workgroup
  const int head = first_head + (rg * 32 >> p.qb_log2);
  const int q_first = qb * QB, q_wave = q_first + (rg * 32 & (QB - 1));
  const int T = p.T;
  const int pos0 = PREFILL ? p.seq[0].n_prefix : 0;          // position of query 0
  const int pos_wave = pos0 + q_wave, pos = pos_wave + (lane & 31);
  const int L = pos0 + min(T, q_first + QB);                 // original keys this workgroup walks over
  const int n_tiles = (L + KT - 1) / KT;

  const size_t row_stride = (size_t)p.Hkv * D;
  const size_t first_key = (PREFILL ? (size_t)p.seq[0].kv_base * row_stride : 0) + (size_t)g * D;
  const bf16_t* kbase = p.k + first_key;
  const bf16_t* vbase = p.v + first_key;
  // Instruction j (0..31) of a tile brings keys 4j .. 4j+3; lane l fetches, for key 4j + (l >> 4), the piece that belongs
  // at position l & 15 of the swizzled row: K rows hold piece c at position c ^ (key & 15), V rows at c ^ ((key & 3) << 2).
  // Keys past the end repeat the last one (masked later).
  const int lkey = lane >> 4;
  const uint32_t vpiece = ((lane & 15) ^ ((lkey & 3) << 2)) * 16;
  uint32_t koff[IPW], voff[IPW];
#pragma unroll
  for (int i = 0; i < IPW; ++i) {
    const int j = wave * IPW + i;
    const uint32_t key_bytes = (uint32_t)(4 * j + lkey) * (uint32_t)(row_stride * 2);
    koff[i] = key_bytes + (uint32_t)(((lane & 15) ^ (4 * (j & 3) + lkey)) * 16);
    voff[i] = key_bytes + vpiece;
  }
  auto clamp_offsets = [&](uint32_t (&off)[IPW], int t) INLINE_LAMBDA {      // for the tile t that the keys end in
    const int last = L - 1 - t * KT;
#pragma unroll
    for (int i = 0; i < IPW; ++i) {
      const int key = 4 * (wave * IPW + i) + lkey;
      off[i] -= (uint32_t)(key - min(key, last)) * (uint32_t)(row_stride * 2);
    }
  };
  // Load r of tile t: its K, then its V
  auto load = [&](int r, int t, uint32_t k_at, uint32_t v_at) INLINE_LAMBDA {
    const size_t first = (size_t)t * KT * row_stride;
    if (r < IPW) dma16(kbase + first, koff[r], lds0 + k_at + wave * IPW * 1024 + r * 1024);
    else dma16(vbase + first, voff[r - IPW], lds0 + v_at + wave * IPW * 1024 + (r - IPW) * 1024);
  };
  auto issue = [&](int t, uint32_t k_at, uint32_t v_at) INLINE_LAMBDA {
    if ((t + 1) * KT > L) {
      clamp_offsets(koff, t);
      clamp_offsets(voff, t);
    }
#pragma unroll
    for (int r = 0; r < 2 * IPW; ++r) load(r, t, k_at, v_at);
  };
  // The simulated steps' own rows: up to hg steps x QB rows = ROWS_WG rows of K and of V at a time go through free tile
  // slots as whole 256-byte rows, piece c of staged row i at position c ^ (i & 15), one copy for all heads and wavefronts.
  // (Read by every lane for itself, 16 and 8 bytes per row and request, they were a third of the kernel: a request that
  // touches 32 lines takes 32 times as long as one that touches one.)
  auto issue_own = [&](int t0, uint32_t k_slot, uint32_t v_slot) INLINE_LAMBDA {
#pragma unroll
    for (int i = 0; i < IPW_ROWS; ++i) {
      const int j = wave * IPW_ROWS + i, r = (4 * j & (QB - 1)) + lkey;       // staged rows 4j .. 4j+3: one step
      const int t = min(t0 + (4 * j >> p.qb_log2), p.s);
      const size_t base = ((size_t)t * T + q_first) * row_stride;
      const uint32_t off = (uint32_t)(min(q_first + r, T - 1) - q_first) * (uint32_t)(row_stride * 2) +
                           (uint32_t)(((lane & 15) ^ (4 * (j & 3) + lkey)) * 16);
      dma16(kbase + base, off, lds0 + k_slot + j * 1024);
      dma16(vbase + base, off, lds0 + v_slot + j * 1024);
    }
  };
  // the workgroup's query rows, staged the same way (row group by row group) behind the tile slots; through registers where the
  // caller's queries do not start at a multiple of 16 bytes
#pragma unroll
  for (int i = 0; i < IPW_ROWS; ++i) {
    const int j = wave * IPW_ROWS + i, r = 4 * j + lkey, rgj = j >> 3;
    const int h = first_head + (rgj * 32 >> p.qb_log2), qr = min(q_first + (rgj * 32 & (QB - 1)) + (r & 31), T - 1);
    const uint32_t off = (uint32_t)(qr - q_first) * (uint32_t)(p.H * ROWB) + (uint32_t)(((lane & 15) ^ (r & 15)) * 16);
    const bf16_t* src = p.q + ((size_t)q_first * p.H + h) * D;
    if (__builtin_expect(p.q_aligned, 1)) {
      dma16(src, off, lds0 + Q_BASE + j * 1024);
    } else {
      u32x4 piece;
      __builtin_memcpy(&piece, (const char*)src + off, 16);
      *(u32x4*)(smem + Q_BASE + j * 1024 + lane * 16) = piece;
    }
  }
  issue(0, 0, V_BASE);
  if (n_tiles > 1) issue(1, TILE_BYTES, V_BASE + TILE_BYTES);

  uint32_t ones = 0x3F803F80u;                 // a bf16 pair, kept in a register
  asm volatile("" : "+v"(ones));

  floatx16 o[4];
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[db][r] = 0.f;
  float m_run = NEG, l_run = 0.f;              // l_run: this lane's share; its partner lane ^ 32 holds the rest

  // my part of the queries and of tile 0 has landed (loads complete in order); the barrier extends that to everyone's
  if (n_tiles > 1) CAUSAL_WAIT_LOADS(2 * IPW);
  else CAUSAL_WAIT_LOADS(0);
  __syncthreads();
  u32x4 qf[8];
#pragma unroll
  for (int ks = 0; ks < 8; ++ks)
    qf[ks] = *(const u32x4*)(smem + Q_BASE + (rg * 32 + (lane & 31)) * ROWB + (((2 * ks + kg) ^ (lane & 15)) * 16));

  // LDS read addresses inside a tile slot.  K operand (32 keys x 16 k) of a block: lane (key = l & 31, pieces 2 ks + kg,
  // whose swizzled offsets are the one of ks = 0 XOR 32 ks bytes).  V^T operand via transposing reads: call c of k-step m
  // returns, for head-dim index db * 32 + (l & 31), keys 16 m + 8 c + 4 kg + 0..3 of the block; the lane hands in the
  // address of 4 head-dim values of ONE of those keys: key + ((l & 15) >> 2), head-dim chunk 16 ((l >> 4) & 1) + 4 (l & 3)
  // (offset of db: XOR 64 db bytes).
  const uint32_t k_rd = lds0 + (uint32_t)((sb * 32 + (lane & 31)) * ROWB + ((kg ^ (lane & 15)) * 16));
  const int vkey0 = sb * 32 + 4 * kg + ((lane & 15) >> 2);
  const uint32_t v_rd = lds0 + (uint32_t)(V_BASE + vkey0 * ROWB + (((2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ ((vkey0 & 3) << 2)) * 16) +
                                          (lane & 1) * 8);
  constexpr uint32_t BLOCK = 64 * ROWB;                      // to a wavefront's second block of the tile

  // Running max over a block of scores; returns the max in force from this block on.  It only moves when some row of the
  // wavefront would raise its own by more than MAX_SLACK (log2 units): until then exp2 may exceed 1 by up to 2^MAX_SLACK,
  // which the fp32 sums and the head/tail split carry without loss, and the output needs no rescaling.
  auto new_max = [&](float mx, bool& grows) INLINE_LAMBDA -> float {
    mx *= p.scale_log2;
    float xa, xb;
    pair_values(mx, xa, xb);
    const float m_cand = fmaxf(m_run, fmaxf(xa, xb));
    grows = __any(m_cand - m_run > MAX_SLACK);
    return grows ? m_cand : m_run;
  };
  // An invisible score is -inf and the max is finite, so its weight is exactly zero.
  auto weight = [&](float x, float m_new) INLINE_LAMBDA -> float {
    return __builtin_amdgcn_exp2f(__builtin_fmaf(x, p.scale_log2, -m_new));
  };
  // Two weights as bf16 heads and tails (p = hi + lo, 16 significant bits): rounding them to a single bf16 would put a 2^-9
  // relative error on the output.  The sum takes what the value products take, so that a rounded weight stays a weight: its
  // error only reaches the output through the distance of its value from the mean.  Plain instructions but for one: the matrix unit
  // stands still while a v_dot2 runs (64 cycles for a product of 32 with five of them behind it, 33 with five of any other kind).
  auto split_pair = [&](float p0, float p1, uint32_t& h, uint32_t& l, float& sum) INLINE_LAMBDA {
    h = pack_bf16x2(p0, p1);
    const float h0 = bf16_lo(h), h1 = bf16_hi(h);
    l = pack_bf16x2(p0 - h0, p1 - h1);
    sum += h0;
    sum += h1;
    sum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, l), __builtin_bit_cast(bf16x2_t, ones), sum, false);
    asm volatile("" : "+v"(h), "+v"(l), "+v"(sum));          // here, among the products, and not where they are used
  };
  auto k_operand = [&](uint32_t at, int ks) INLINE_LAMBDA -> u32x4 { return read_lds(at ^ (32u * ks)); };
  // operand n of a block of values: k-step n >> 2, head-dim block n & 3
  auto v_operand = [&](uint32_t at, int n) INLINE_LAMBDA -> u32x4 {
    const uint32_t a = (at ^ (64u * (n & 3))) + 16 * (n >> 2) * ROWB;
    const short4v lo4 = read_tr(a), hi4 = read_tr(a + 8 * ROWB);
    return __builtin_bit_cast(u32x4, __builtin_shufflevector(lo4, hi4, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  // weights of one block: entry i & 3 of operand i >> 2 of heads and tails
  struct Weights { u32x4 h[2], l[2]; };
  u32x4 va[4];                                 // value operands n of the block in work at n & 3

  // Softmax of the block of scores in s (first key kb) among the products of its neighbours: values of the previous block
  // (weights w; V at v_at, its first two operands already in va) and scores of the next one (K at k_at, into sn).  A block is a
  // matrix-unit time of 24 products (768 cycles) and nearly as many issue cycles of everything else, so the softmax is spread over all of them: weights
  // 0..11 of this block here, and 12..15 of the previous one, whose scores are still in sn, during the search for the max.  Leaves what
  // there is of this block's weights in wn and its first two value operands (V at v_next) in va.  LOAD: the direct loads of tile t_load too, one behind every
  // other product: behind the barrier, all together, they kept the wavefronts from issuing.  The order is written out and pinned:
  // the compiler on its own puts the products first and the exponentials after them.
  constexpr int LATE = 12;
  auto put_pair = [&](float p0, float p1, int n, Weights& w, float& sum) INLINE_LAMBDA {      // weights 2 n and 2 n + 1
    uint32_t h, l;
    split_pair(p0, p1, h, l, sum);
    w.h[n >> 2][n & 3] = h;
    w.l[n >> 2][n & 3] = l;
  };
  auto block = [&](auto has_prev, auto has_next, auto has_load, floatx16& s, floatx16& sn, Weights& w, Weights& wn, int kb, uint32_t k_at, uint32_t v_at,
                   uint32_t v_next, int t_load, uint32_t k_fill, uint32_t v_fill) INLINE_LAMBDA {
    constexpr bool PREV = decltype(has_prev)::value, NEXT = decltype(has_next)::value, LOAD = decltype(has_load)::value;
    auto value = [&](int n, bool tail) INLINE_LAMBDA {
      if constexpr (PREV) o[n & 3] = mfma(va[n & 3], tail ? w.l[n >> 2] : w.h[n >> 2], o[n & 3]);
    };
    auto fetch = [&](int n) INLINE_LAMBDA {
      if constexpr (PREV) va[n & 3] = v_operand(v_at, n);
    };
    auto loads = [&](int at) INLINE_LAMBDA {   // at 0..15
      if constexpr (LOAD)
#pragma unroll
        for (int r = 0; r < 2 * IPW; ++r)
          if (r * 16 / (2 * IPW) == at) load(r, t_load, k_fill, v_fill);
    };
    u32x4 kf[3];
    fetch(2);
    fetch(3);
    if constexpr (NEXT) {
      kf[0] = k_operand(k_at, 0);
      kf[1] = k_operand(k_at, 1);
    }
    if (kb + 31 > pos_wave) {                  // keys after the lane's query: key kb + i is visible iff kb + i <= pos
      const int n_vis = pos - kb + 1;
      const uint32_t vis = (n_vis >= 32 ? 0xFFFFFFFFu : n_vis <= 0 ? 0u : ((1u << n_vis) - 1u)) >> (4 * kg);
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = ((vis >> (8 * (r >> 2) + (r & 3))) & 1u) ? s[r] : -INFINITY;
    }
    CAUSAL_PIN();
    // first half: eight value products over the search for the max and the previous block's last weights
    float late[4] = {0.f, 0.f, 0.f, 0.f}, e[LATE];
    auto late_weight = [&](int i) INLINE_LAMBDA {
      if constexpr (PREV) late[i] = weight(sn[LATE + i], m_run);
    };
    value(0, false);
    loads(0);
    float mx = fmaxf(fmaxf(s[0], s[1]), s[2]);
    mx = fmaxf(fmaxf(mx, s[3]), s[4]); mx = fmaxf(fmaxf(mx, s[5]), s[6]);
    CAUSAL_PIN();
    value(1, false);
    loads(1);
    late_weight(0);
    mx = fmaxf(fmaxf(mx, s[7]), s[8]); mx = fmaxf(fmaxf(mx, s[9]), s[10]);
    CAUSAL_PIN();
    value(0, true);
    loads(2);
    late_weight(1);
    mx = fmaxf(fmaxf(mx, s[11]), s[12]); mx = fmaxf(fmaxf(fmaxf(mx, s[13]), s[14]), s[15]);
    CAUSAL_PIN();
    value(1, true);
    loads(3);
    fetch(4);
    bool grows;
    const float m_new = new_max(mx, grows);
    CAUSAL_PIN();
    value(2, false);
    loads(4);
    fetch(5);
    if constexpr (PREV) put_pair(late[0], late[1], LATE / 2, w, l_run);
    CAUSAL_PIN();
    value(3, false);
    loads(5);
    late_weight(2);
    late_weight(3);
    CAUSAL_PIN();
    value(2, true);
    loads(6);
    if constexpr (PREV) put_pair(late[2], late[3], LATE / 2 + 1, w, l_run);
    CAUSAL_PIN();
    value(3, true);
    loads(7);
    e[0] = weight(s[0], m_new);
    e[1] = weight(s[1], m_new);
    CAUSAL_PIN();
    // second half: eight score products and eight value products; weight 2 + i behind score product at_of[i] / 2 or, odd, value product at_of[i] / 2, and
    // pair pair_at[j] is split behind value product j
    constexpr int at_of[LATE - 2] = {0, 1, 3, 4, 6, 7, 9, 10, 12, 13}, pair_at[8] = {0, 1, -1, 2, 3, -1, 4, 5};
    float ls = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      auto weights = [&](int at) INLINE_LAMBDA {
#pragma unroll
        for (int i = 0; i < LATE - 2; ++i)
          if (at_of[i] == at) e[2 + i] = weight(s[2 + i], m_new);
      };
      if constexpr (NEXT) {
        if (j == 0) {
#pragma unroll
          for (int r = 0; r < 16; ++r) sn[r] = 0.f;
        }
        sn = mfma(kf[j % 3], qf[j], sn);
        if (j < 6) kf[(j + 2) % 3] = k_operand(k_at, j + 2);
      }
      weights(2 * j);
      loads(8 + j);
      CAUSAL_PIN();
      value(4 + (j & 1) + 2 * (j >> 2), (j >> 1) & 1);
      if (j == 1) fetch(6);
      if (j == 2) fetch(7);
      if (j == 6) va[0] = v_operand(v_next, 0);
      if (j == 7) va[1] = v_operand(v_next, 1);
      weights(2 * j + 1);
      if (pair_at[j] >= 0) put_pair(e[2 * pair_at[j]], e[2 * pair_at[j] + 1], pair_at[j], wn, ls);
      CAUSAL_PIN();
    }
    if (grows) {
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
    }
    l_run += ls;
  };
  // the last block's (scores s) last weights and its values: its first two operands are in va
  auto finish = [&](const floatx16& s, Weights& w, uint32_t v_at) INLINE_LAMBDA {
    put_pair(weight(s[LATE], m_run), weight(s[LATE + 1], m_run), LATE / 2, w, l_run);
    put_pair(weight(s[LATE + 2], m_run), weight(s[LATE + 3], m_run), LATE / 2 + 1, w, l_run);
#pragma unroll
    for (int n = 0; n < 8; ++n) {
      if (n > 1) va[n & 3] = v_operand(v_at, n);
      o[n & 3] = mfma(va[n & 3], w.h[n >> 2], o[n & 3]);
      o[n & 3] = mfma(va[n & 3], w.l[n >> 2], o[n & 3]);
    }
  };

  floatx16 s0, s1;
  Weights w0, w1;
#pragma unroll
  for (int r = 0; r < 16; ++r) s0[r] = 0.f;
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) s0 = mfma(k_operand(k_rd, ks), qf[ks], s0);
  // Tile t in two blocks; one barrier between them.  It publishes K and V of tile t + 1, and frees the slots of K t and
  // V t - 1 for K and V of tile t + 2.  So the second block can read K of t + 1, and V operands are in LDS early enough to
  // be read a block ahead.
  int kb = sb * 32;
  uint32_t k_slot = 0, v_slot = 0;             // of tile t
  block(Flag<false>(), Flag<true>(), Flag<false>(), s0, s1, w0, w0, kb, k_rd + BLOCK, v_rd, v_rd, 0, 0, 0);
  auto tile = [&](auto has_load, int t) INLINE_LAMBDA {
    CAUSAL_WAIT_LOADS(0);
    __syncthreads();
    const uint32_t v_1 = v_slot == 2 * TILE_BYTES ? 0 : v_slot + TILE_BYTES;         // V slots of tiles t + 1, t + 2
    const uint32_t v_2 = v_1 == 2 * TILE_BYTES ? 0 : v_1 + TILE_BYTES;
    if (decltype(has_load)::value && (t + 3) * KT > L) {
      clamp_offsets(koff, t + 2);
      clamp_offsets(voff, t + 2);
    }
    const uint32_t k_1 = k_slot ^ TILE_BYTES;
    block(Flag<true>(), Flag<true>(), has_load, s1, s0, w0, w1, kb + 64, k_rd + k_1, v_rd + v_slot, v_rd + v_slot + BLOCK, t + 2, k_slot, V_BASE + v_2);
    kb += KT;
    block(Flag<true>(), Flag<true>(), Flag<false>(), s0, s1, w1, w0, kb, k_rd + k_1 + BLOCK, v_rd + v_slot + BLOCK, v_rd + v_1, 0, 0, 0);
    k_slot = k_1;
    v_slot = v_1;
  };
  int t = 0;
#pragma unroll 1
  for (; t + 2 < n_tiles; ++t) tile(Flag<true>(), t);
  if (t + 1 < n_tiles) tile(Flag<false>(), t);
  // The last tile's second block, where any query of the workgroup sees a key of it.  K's other slot and V's next were last read
  // before the last barrier: the own rows go there.
  uint32_t own_k = k_slot ^ TILE_BYTES, own_v = V_BASE + (v_slot == 2 * TILE_BYTES ? 0 : v_slot + TILE_BYTES), own_v_other = V_BASE + v_slot;
  if (!PREFILL && p.s > 0) issue_own(1, own_k, own_v);
  if (kb + 64 < L) {
    block(Flag<true>(), Flag<false>(), Flag<false>(), s1, s0, w0, w1, kb + 64, 0, v_rd + v_slot, v_rd + v_slot + BLOCK, 0, 0, 0);
    finish(s1, w1, v_rd + v_slot + BLOCK);
  } else {
    finish(s0, w0, v_rd + v_slot);
  }

  // The query's own key of every simulated step: one dot product and one scaled row of values each, the two key halves
  // taking alternate steps.  Last, as they are exact in fp32 against any max; taken first, their max would be in force for
  // the first keys, whose largest weight is then no longer 1 but carried with 16 bits (twice the error in the first rows).  This lane holds the query's entries 16 ks + 8 kg + 0..7 (its partner lane ^ 32 the other
  // half) and the output entries 32 db + 8 gq + 4 kg + 0..3.
  // Batches of hg steps go through the two free slots and the last tile's own in turn, each requested when the one before it is worked on (behind the
  // first batch's barrier nobody reads the last tile any more).
  auto own_step = [&](int i, float& sc, uint2 (&vv)[16]) INLINE_LAMBDA {          // score and values of staged row i
    const unsigned char* kr = smem + own_k + i * ROWB;
    const unsigned char* vr = smem + own_v + i * ROWB + kg * 8;
    u32x4 kk[8];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) kk[ks] = *(const u32x4*)(kr + (((2 * ks + kg) ^ (i & 15)) * 16));
#pragma unroll
    for (int c = 0; c < 16; ++c) vv[c] = *(const uint2*)(vr + ((c ^ (i & 15)) * 16));
    float dot[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        dot[e] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, (uint32_t)qf[ks][e]), __builtin_bit_cast(bf16x2_t, (uint32_t)kk[ks][e]), dot[e], false);
    float xa, xb;
    pair_values((dot[0] + dot[1]) + (dot[2] + dot[3]), xa, xb);
    sc = (xa + xb) * p.scale_log2;
  };
#pragma unroll 1
  for (int t0 = 1; !PREFILL && t0 <= p.s; t0 += p.hg) {
    CAUSAL_WAIT_LOADS(0);
    __syncthreads();
    const uint32_t next_k = own_k ^ TILE_BYTES, next_v = own_v_other;
    if (t0 + p.hg <= p.s) issue_own(t0 + p.hg, next_k, next_v);
#pragma unroll 1
    for (int t = t0 + ((t0 + sb + 1) & 1); t < t0 + p.hg && t <= p.s; t += 2) {
      float sc;
      uint2 vv[16];
      own_step((t - t0) * QB + q_wave - q_first + (lane & 31), sc, vv);
      if (__any(sc - m_run > MAX_SLACK)) {     // as in new_max
        const float m_new = fmaxf(m_run, sc), alpha = __builtin_amdgcn_exp2f(m_run - m_new);
        m_run = m_new;
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
      }
      const float pw = __builtin_amdgcn_exp2f(sc - m_run);
      l_run += kg == 0 ? pw : 0.f;
#pragma unroll
      for (int c = 0; c < 16; ++c) {
        const int db = c >> 2, r = 4 * (c & 3);
        o[db][r] = fmaf(pw, bf16_lo(vv[c].x), o[db][r]);
        o[db][r + 1] = fmaf(pw, bf16_hi(vv[c].x), o[db][r + 1]);
        o[db][r + 2] = fmaf(pw, bf16_lo(vv[c].y), o[db][r + 2]);
        o[db][r + 3] = fmaf(pw, bf16_hi(vv[c].y), o[db][r + 3]);
      }
    }
    own_v_other = own_v;
    own_k = next_k;
    own_v = next_v;
  }
  CAUSAL_WAIT_LOADS(0);

  // Merge the two key halves: each wavefront finishes the half of the head dimension (db = 2 sb, 2 sb + 1) and hands the
  // other half, with its max and sum, to its partner through LDS.
  __syncthreads();
  float* xo = (float*)smem + (size_t)(rg * 2) * (34 * 64);
  {
    float* mine = xo + sb * (34 * 64);
#pragma unroll
    for (int d2 = 0; d2 < 2; ++d2)
#pragma unroll
      for (int r = 0; r < 16; ++r) mine[(d2 * 16 + r) * 64 + lane] = sb == 0 ? o[2 + d2][r] : o[d2][r];
    mine[32 * 64 + lane] = m_run;
    mine[33 * 64 + lane] = l_run;
  }
  __syncthreads();
  const float* theirs = xo + (sb ^ 1) * (34 * 64);
  const float m2 = theirs[32 * 64 + lane], l2 = theirs[33 * 64 + lane];
  const float m_all = fmaxf(m_run, m2);
  const float f1 = __builtin_amdgcn_exp2f(m_run - m_all), f2 = __builtin_amdgcn_exp2f(m2 - m_all);
  float la, lb;
  pair_values(l_run * f1 + l2 * f2, la, lb);
  const float inv = 1.0f / (la + lb);
  floatx4 val[2][4];                           // values 32 d2 + 8 gq + 4 kg + 0..3 of this wavefront's half
  float probe = 0.f;
#pragma unroll
  for (int d2 = 0; d2 < 2; ++d2)
#pragma unroll
    for (int gq = 0; gq < 4; ++gq)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = 4 * gq + e;
        const float x = ((sb == 0 ? o[d2][r] : o[2 + d2][r]) * f1 + theirs[(d2 * 16 + r) * 64 + lane] * f2) * inv;
        val[d2][gq][e] = x;
        probe = fmaf(x, 0.f, probe);           // stays 0 while every value is finite
      }
  if (__builtin_expect(__any(probe != 0.f), 0)) {
    // The value product multiplies keys that a query does not see with weights that are exactly zero, which keeps out everything but
    // an infinity or NaN.  So rows that came out non-finite are formed again one key at a time over the keys they see: either the
    // value at fault is one of those, or it does not count.
    float m = NEG, l = 0.f;
#pragma unroll
    for (int d2 = 0; d2 < 2; ++d2)
#pragma unroll
      for (int gq = 0; gq < 4; ++gq) val[d2][gq] = (floatx4){0.f, 0.f, 0.f, 0.f};
    const int n_orig = min(pos_wave + 32, L);
    const size_t own_row = min(q_wave + (lane & 31), T - 1);
#pragma unroll 1
    for (int j = 0; j < n_orig + (PREFILL ? 0 : p.s); ++j) {
      if ((j & 31) == 31) {                    // a NaN stays one: nothing left to find out in a wavefront that has nothing else
        bool open = false;
#pragma unroll
        for (int d2 = 0; d2 < 2; ++d2)
#pragma unroll
          for (int gq = 0; gq < 4; ++gq)
#pragma unroll
            for (int e = 0; e < 4; ++e) open |= val[d2][gq][e] == val[d2][gq][e];
        if (!__any(open)) break;
      }
      const size_t at = (j < n_orig ? (size_t)j : (size_t)(j - n_orig + 1) * T + own_row) * row_stride;
      float dot = 0.f;
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        const u32x4 kk = *(const u32x4*)(kbase + at + ks * 16 + kg * 8);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          dot = fmaf(bf16_lo(qf[ks][e]), bf16_lo(kk[e]), dot);
          dot = fmaf(bf16_hi(qf[ks][e]), bf16_hi(kk[e]), dot);
        }
      }
      float xa, xb;
      pair_values(dot, xa, xb);
      if (j < n_orig && j > pos) continue;
      const float sc = (xa + xb) * p.scale_log2;
      const float m_new = fmaxf(m, sc);
      const float alpha = __builtin_amdgcn_exp2f(m - m_new), pw = __builtin_amdgcn_exp2f(sc - m_new);
      l = l * alpha + pw;
      m = m_new;
#pragma unroll
      for (int d2 = 0; d2 < 2; ++d2)
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
          const uint2 vv = *(const uint2*)(vbase + at + sb * 64 + d2 * 32 + 8 * gq + 4 * kg);
          const floatx4 v = {bf16_lo(vv.x), bf16_hi(vv.x), bf16_lo(vv.y), bf16_hi(vv.y)};
#pragma unroll
          for (int e = 0; e < 4; ++e) val[d2][gq][e] = val[d2][gq][e] * alpha + pw * v[e];
        }
    }
#pragma unroll
    for (int d2 = 0; d2 < 2; ++d2)
#pragma unroll
      for (int gq = 0; gq < 4; ++gq)
#pragma unroll
        for (int e = 0; e < 4; ++e) val[d2][gq][e] /= l;
  }
  if constexpr (PREFILL) {
    if (q_wave + (lane & 31) >= T) return;
#pragma unroll
    for (int d2 = 0; d2 < 2; ++d2)
#pragma unroll
      for (int gq = 0; gq < 4; ++gq)
        Act<true>::store4((bf16_t*)p.out, q_wave + (lane & 31), head * D + sb * 64 + d2 * 32 + 8 * gq + 4 * kg, p.H * D, val[d2][gq][0],
                          val[d2][gq][1], val[d2][gq][2], val[d2][gq][3]);
  } else {
    // The finished 32 rows x 64 values of this wavefront go through its own 8 KB of LDS, so that the stores are whole
    // 256-byte runs: 16-byte piece c of row i at position c ^ (i & 15).
    unsigned char* stage = smem + STAGE_BASE + wave * 8192;
#pragma unroll
    for (int d2 = 0; d2 < 2; ++d2)
#pragma unroll
      for (int gq = 0; gq < 4; ++gq)
        *(floatx4*)(stage + (lane & 31) * 256 + (((d2 * 8 + 2 * gq + kg) ^ (lane & 15)) * 16)) = val[d2][gq];
    __builtin_amdgcn_wave_barrier();           // one wavefront's LDS operations complete in order
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const int i = 4 * c + lkey;
      const floatx4 v = *(const floatx4*)(stage + i * 256 + (((lane & 15) ^ (i & 15)) * 16));
      if (q_wave + i < T) *(floatx4*)((float*)p.out + ((size_t)(q_wave + i) * p.H + head) * D + sb * 64 + (lane & 15) * 4) = v;
    }
  }
}

// fp32: one workgroup per (query, head); scores of the i + 1 + s visible keys in LDS, the keys of the value sum dealt out to
// 256 / d groups of threads
__global__ __launch_bounds__(256) void ttt_attn_f32_kernel(const float* __restrict__ q, const float* __restrict__ k,
                                                          const float* __restrict__ v, int T, int H, int Hkv, int d, int s,
                                                          float scale, float* __restrict__ out) {
  extern __shared__ float sc[];
  __shared__ float red[17], qs[256], part[256];    // with 60 KB of scores still below the 64 KB of an ordinary launch
  const int i = blockIdx.x, h = blockIdx.y, g = h * Hkv / H, tid = threadIdx.x;
  const int n = i + 1 + s;
  const float* qr = q + ((size_t)i * H + h) * d;
  if (tid < d) qs[tid] = qr[tid];
  __syncthreads();
  auto key_row = [&](int j) { return j <= i ? (size_t)j : (size_t)(j - i) * T + i; };      // row of the [s+1, T] arrays
  float mx = -INFINITY;
  for (int j = tid; j < n; j += 256) {
    const float* kr = k + (key_row(j) * Hkv + g) * d;
    sc[j] = (d <= 256 ? dot_f32(qs, kr, d) : dot_f32(qr, kr, d)) * scale;
    mx = fmaxf(mx, sc[j]);
  }
  mx = block_max(mx, red);
  float sum = 0.f;
  for (int j = tid; j < n; j += 256) {
    const float e = expf(sc[j] - mx);
    sc[j] = e;
    sum += e;
  }
  sum = block_sum(sum, red);                // also publishes sc
  if (d > 128) {
    for (int e = tid; e < d; e += 256) {
      float acc = 0.f;
#pragma unroll 8
      for (int j = 0; j < n; ++j) acc = fmaf(sc[j], v[(key_row(j) * Hkv + g) * d + e], acc);
      out[((size_t)i * H + h) * d + e] = acc / sum;
    }
    return;
  }
  const int groups = 256 / d, grp = tid / d, e = tid - grp * d;
  float acc = 0.f;
  if (grp < groups) {
#pragma unroll 8
    for (int j = grp; j < n; j += groups) acc = fmaf(sc[j], v[(key_row(j) * Hkv + g) * d + e], acc);
  }
  part[tid] = acc;
  __syncthreads();
  if (tid < d) {
    acc = 0.f;
    for (int j = 0; j < groups; ++j) acc += part[j * d + tid];
    out[((size_t)i * H + h) * d + tid] = acc / sum;
  }
}

template <bool PREFILL, int RG>
hipError_t launch_causal(CausalParams& p, hipStream_t st) {
  auto kernel = causal_attn_bf16_kernel<PREFILL, RG>;
  static DeviceOnce configured;                  // the attribute belongs to the loaded code object of a device
  hipError_t ce = configured.run([&] { return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES); });
  if (ce != hipSuccess) return ce;
  p.hg = causal_heads_per_wg(p.H, p.Hkv, RG);
  const int groups = p.H / p.hg;
  p.n_qblocks = causal_workgroups(p.T, p.H, p.Hkv, RG) / groups;
  p.qb_log2 = (RG == 4 ? 7 : 6) - (p.hg == 4 ? 2 : p.hg == 2 ? 1 : 0);         // 32 RG / hg
  p.G = p.H / p.Hkv;
  p.by_groups = divisor(groups); p.by_kv_heads = divisor(p.Hkv);
  p.scale_log2 = 1.4426950408889634f / sqrtf((float)D);
  p.q_aligned = ((uintptr_t)p.q & 15) == 0;
  hipLaunchKernelGGL(kernel, dim3((unsigned)groups * p.n_qblocks), dim3(128 * RG), LDS_BYTES, st, p);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_ttt_attention(bool bf16, const void* q, const void* k, const void* v, int T, int H, int Hkv, int d, int s,
                                float* out, hipStream_t st) {
  if (T < 1 || H < 1 || Hkv < 1 || H % Hkv || s < 0) return hipErrorInvalidValue;
  if (!bf16) {
    const size_t lds = (size_t)(T + s) * sizeof(float);
    if (lds > 60 * 1024 || d > 1024) return hipErrorInvalidValue;
    hipLaunchKernelGGL(ttt_attn_f32_kernel, dim3(T, H), dim3(256), lds, st, (const float*)q, (const float*)k, (const float*)v,
                       T, H, Hkv, d, s, 1.0f / sqrtf((float)d), out);
    return hipGetLastError();
  }
  if (d != D) return hipErrorInvalidValue;
  CausalParams p;
  p.q = (const bf16_t*)q; p.k = (const bf16_t*)k; p.v = (const bf16_t*)v;
  p.seq = nullptr;
  p.T = T; p.H = H; p.Hkv = Hkv; p.s = s;
  p.out = out;
  return causal_half_workgroups(T, H, Hkv, s) ? launch_causal<false, 2>(p, st) : launch_causal<false, 4>(p, st);
}

hipError_t launch_prefill_attention(const void* q, const void* kcache, const void* vcache, const SeqInfo* seq, int n, int H, int Hkv,
                                    int d, void* out, hipStream_t st) {
  if (n < 1 || H < 1 || Hkv < 1 || H % Hkv || d != D) return hipErrorInvalidValue;
  CausalParams p;
  p.q = (const bf16_t*)q; p.k = (const bf16_t*)kcache; p.v = (const bf16_t*)vcache;
  p.seq = seq;
  p.T = n; p.H = H; p.Hkv = Hkv; p.s = 0;
  p.out = out;
  return launch_causal<true, 4>(p, st);
}
