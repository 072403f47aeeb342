// Which output tile the many-row product takes, and into how many K ranges it is cut.  Host arithmetic only.
//
// Workgroups of one weight tile go to one XCD (32 CUs): a launch lasts as many rounds as the fullest XCD has workgroups per CU,
// and that XCD has at most ceil(weight tiles / 8) of them for every row block and K range: exactly that many, unless K ranges are dealt to XCDs (dealt_ranges: then
// ceil(weight tiles / (8 / ranges)) for each of its own ranges, 20 tiles in four ranges 10 and not 12).  The estimates below count the former, and their fits are of
// launches without dealt ranges: of products in dealt ranges they tell the order less well.  1586 split products of 16 model shapes beyond 256 rows: what they pick is 2.1 % slower
// than the best of the tiles on average; counting what an XCD has, and a tile of 192 or 224 weight rows without its margin there, 1.2 %, but 43 of the 263 products
// that take another tile then are slower, by 1 to 10 %, and others sum in longer chains.
#pragma once
#include <cstddef>
#include <initializer_list>

struct WideTiles {
  int rows, cols;      // output tile of a workgroup
  int S;               // K ranges (split-K partial sums); 1 for SwiGLU
  int k;               // width of a weight stage: 64, or 128 for tiles of 128 weight rows
};

// log2 of the K ranges of a split product that are dealt to different XCDs (wide_places.hpp).  Activations that an XCD's 4 MB of L2 cannot hold are fetched by each of
// them again, unless it has some of the K ranges only.  Product alone, us, all ranges / its own: down 4096 x 14336 256 rows 44.2 / 42.5, 512 rows 66.8 / 64.4,
// 2048 rows 184 / 178.  255 split products of 16 model shapes with 6 to 40 MB of activations: 2.0 % faster on average, 161 of them by more than 1 %, 15 slower by more (worst
// 3072 x 8192 at 640 rows 41.3 / 44.0).  Below, where the line was drawn after two products of 4.2 MB (o 4096 x 4096 512 rows 25.6 / 26.0, q/k/v 37.9 / 38.1), 224 others
// with 2 to 6 MB would gain 1.5 % on average: the line could lie lower.
inline int dealt_ranges(int M, int K, int S) {
  int ranges = 0;
  while (ranges < 3 && S % (2 << ranges) == 0 && (size_t)M * K * 2 > ((size_t)6 << 20)) ++ranges;
  return ranges;
}

// Whether the K walks of a launch of 65..256 rows start at a stage of each workgroup's own (gemm_wide.hip has the figures).
inline bool wide_stagger(int M, int K, const WideTiles& t) { return M <= 256 && K / t.S % 2048 == 0 && (t.k == 128 || t.S == 1); }

// 65..256 rows, where activation lines don't count (what is launched: stream_tiles): 128 weight rows to a workgroup, so that every weight line enters one CU, and one block of 128
// or 256 activation rows.  Stages of 128 k, whose row pieces of 256 bytes HBM delivers faster than pieces of 128, take all of a CU's LDS;
// with stages of 64 k two 128 x 128 workgroups run side by side.  The kind and the split whose launch is over first by this estimate,
// in microseconds: a start and an end, a time per stage that grows with the workgroups that stream at once, in rounds of 32 workgroups
// of the fullest XCD (64 side by side), and the writing and reading of the partial sums.  The numbers are fits to 150 products of 34 model
// shapes (K 512..28672, N 512..151936), each with every split and the kernel that reads the sums.  65, 77, 100 and 128 rows: what the estimate
// picks is 0.1 % slower than the best on average, 9 % at worst (151936 x 3584), and nowhere more than 2 % slower than stages of 64 k split by
// workgroup counts.  Before, walks of 64 k were charged too much, and large unsplit products took wide stages: us, wide / 64 k, gate/up
// 57344 x 8192 100 rows 201 / 189, 37888 x 3584 65 rows 84 / 79, LM head 128256 x 4096 65 rows 234 / 212, 64000 x 7168 100 rows 214 / 192;
// but gate/up 28672 x 4096 77 rows 53 / 57, LM head 151936 x 3584 77 rows 248 / 267.
// 129, 160, 200 and 256 rows: 0.3 % and 9 %.  Stages of 64 k are left there for splits whose ranges 128 does not divide: 4096 x 11008
// in four of 2752, 200 rows 54 us, in two of 5504 80; 3584 x 18944 in eight of 2368 53, in four 74.
inline WideTiles wide_tiles_256(int M, int N, int K, bool swiglu, size_t out_capacity_floats, float* time = nullptr) {
  const bool few = M <= 128;
  const int rows = few ? 128 : 256, per_xcd = ((N + 127) / 128 + 7) / 8;
  const float slower = 1.f + 0.0008f * (M - 77);                       // up to 128 rows
  const float start = few ? 6.4f : 8.4f, alone = few ? 1.37f * slower : 1.79f, full = few ? 1.41f * slower : 1.99f;
  WideTiles best = {rows, 128, 1, 64};
  float least = 0.f;
  for (int k : {128, 64})
    for (int S = 1; S <= (swiglu ? 1 : 8); ++S) {
      const int range = K / S, n = per_xcd * S;
      if (K % (k * S) || range < 512 || (S > 1 && (size_t)S * M * N > out_capacity_floats)) continue;
      if (k == 64 && !few && range % 128 == 0) continue;               // for ranges that 128 does not divide
      const float stages = (float)range / k;
      float t = swiglu ? 0.f : (float)S * M * N * (few ? 2.3e-6f : 0.8e-6f);
      if (k == 128 || !few) {
        const float f = k == 128 ? 1.f : 0.55f;                        // of a stage of 128 k
        t += n / 32 * (start + full * f * stages);
        if (n % 32) t += start + stages * f * (full * (n % 32) / 32 > alone ? full * (n % 32) / 32 : alone);
      } else {
        const float last = n % 64 / 64.f;
        t += n / 64 * (3.9f + 1.47f * stages);
        if (last > 0.f) t += 3.9f + stages * (last <= 0.5f ? 0.93f : 1.47f * last > 1.44f ? 1.47f * last : 1.44f);
      }
      if (least == 0.f || t < least) { least = t; best = {rows, 128, S, k}; }
    }
  if (time) *time = least;
  return best;
}

// A tile beyond 256 rows with its split: the smallest that makes `want` workgroups, of ranges of at least `min_stages` stages of 64 k.
inline WideTiles with_split(int M, int N, int K, bool swiglu, size_t out_capacity_floats, int rows, int cols, int want, int min_stages) {
  const int KT = K / 64, wgs = (N + cols - 1) / cols * ((M + rows - 1) / rows);
  int S = 1;
  if (!swiglu)
    for (int s = 1; s <= 8 && wgs * S < want; ++s) {
      if (KT % s) continue;
      if (s > 1 && ((size_t)s * M * N > out_capacity_floats || KT / s < min_stages)) break;
      S = s;
    }
  return {rows, cols, S, 64};
}

// How long a launch beyond 256 rows lasts, in microseconds, with the kernel that reads its partial sums.  A workgroup takes a start and an end, and a
// time per 64 k; the fullest XCD runs its workgroups in rounds of 32, of 64 for 128 x 128 tiles (two on a CU side by side, one
// alone where there are no more than 32 left); writing and reading the partial sums comes on top.  The eleven numbers of the tiles of 256 and of 128 weight rows are a
// fit to 150 products of 34 model shapes at 13 row counts from 257 to 2048, each with all four of them and the kernel that reads the sums: what the
// estimate picks of the four is 0.2 % slower than the best on average (13 % at worst: 2304 x 9216 at 1500 rows), and 12 % faster than picking by
// workgroup counts.  The four numbers of 224 and 192 weight rows: half of 430 launches each of 24 shapes, 300 to 4096 rows, all splits, took longer
// (within 1 %), single ones differ by 8.5 and 7 % on average.  The choice of all six (launch_tiles), 178 products of those shapes: 1.0 % slower than the best
// whose chains of sums are no longer, 14 % at worst (4608 x 3584 at 2048 rows), and 3 % than the best of any chain.
// Fitted to 17 products, the first eleven had charged 128 x 128 tiles too much: us, then / now, down 4352 x 17024 300 rows 114 / 100, gate/up
// 18432 x 2304 257 rows 48 / 43, o 5120 x 5120 300 rows 43 / 40.  8B width, product and reading, us, 256 x 256 / 192 x 256 /
// 256 x 128 / 128 x 128: q/k/v 300 rows 38 / 35 / 36 / 44, 512 rows 44 / 64 / 40 / 50, 600 rows 73 / 52 / 71 / 50; down 300 rows
// 63 / 58 / 60 / 69, 512 rows 73 / 80 / 67 / 83; o 1024 rows 49 / 49 / 42 / 50; gate/up 300 rows 101 / 87 / 116 / 121, 1024 rows
// 197 / 235 / 231 / 274, 2048 rows 382 / 392 / 406 / 509; hidden 2048, gate/up 300 rows 45 / 41 / 31 / 30.
inline float wide_time(int M, int N, int K, bool swiglu, const WideTiles& w) {
  auto ceil_div = [](int a, int b) { return (a + b - 1) / b; };
  const int n = ceil_div(ceil_div(N, w.cols), 8) * ceil_div(M, w.rows) * w.S;
  const float stages = (float)K / 64 / w.S, sums = swiglu ? 0.f : (float)w.S * M * N * 1.2e-6f;
  if (w.cols == 224) return ceil_div(n, 32) * (7.6f + 1.28f * stages) + sums;
  if (w.cols == 192) return ceil_div(n, 32) * (8.f + 1.1f * stages) + sums;
  if (w.cols == 256) return ceil_div(n, 32) * (w.rows == 256 ? 7.4f + 1.36f * stages : 8.2f + 1.1f * stages) + sums;
  if (w.rows == 256) return ceil_div(n, 32) * (8.f + 0.81f * stages) + sums;
  const float two = 7.3f + 1.085f * stages, one = 7.4f + 0.595f * stages;
  const int rest = n % 64;
  return n / 64 * two + (rest == 0 ? 0.f : rest <= 32 ? one : two) + sums;
}

// The tile whose launch is over first by that estimate.
inline WideTiles wide_tiles_k64(int M, int N, int K, bool swiglu, size_t out_capacity_floats) {
  auto pick = [&](int rows, int cols, int want, int min_stages) { return with_split(M, N, K, swiglu, out_capacity_floats, rows, cols, want, min_stages); };
  auto cost = [&](const WideTiles& t) { return wide_time(M, N, K, swiglu, t); };
  WideTiles best = pick(256, 256, 160, 16);
  for (const WideTiles& t : {pick(192, 256, 160, 16), pick(256, 128, 192, 16), pick(128, 128, 384, 8)})
    if (cost(t) < cost(best)) best = t;
  return best;
}

// Stages of 128 k beyond 256 rows: where one workgroup has a CU to itself, 256 x 128 always, 128 x 128 up to 256 workgroups (300 rows LM
// head, 3006 workgroups: 457 us with 64, 530 with 128).  A workgroup's walk has to be long enough, as fewer and larger stages start later.
inline WideTiles wide_tiles(int M, int N, int K, bool swiglu, size_t out_capacity_floats) {
  WideTiles t = wide_tiles_k64(M, N, K, swiglu, out_capacity_floats);
  const int wgs = (N + t.cols - 1) / t.cols * ((M + t.rows - 1) / t.rows) * t.S, range = K / t.S;
  if (t.cols == 128 && range % 128 == 0 && range >= (t.rows == 256 && t.S == 1 ? 256 : 1024) && (t.rows == 256 || wgs <= 256)) t.k = 128;
  return t;
}

// The tile that is launched beyond 256 rows: that, or 256 x 224 or 256 x 192 (4 x 2 wavefronts of 64 x 112 or 64 x 96).  28672 weight rows (8B
// gate/up) are 112 tiles of 256, 3.5 rounds of the chip at 2048 rows, and 128 of 224, four whole ones; 6144 (q/k/v) are 24 of 256, three
// quarters of a round, and 32 of 192.  Taken by a margin of 2 % of the estimate, and only with chains of sums no longer than the other tile's
// (stages of 128 k: two chains).  us, with the kernel that reads partial sums, the other tile / this one: gate/up 2048 rows 371 / 357, 1280 rows 286 / 244, 512 rows
// 99.8 / 98.3 (the same work on more CUs draws the same power), 57344 x 8192 1024 rows 761 / 716, 27648 x 5120 1280 rows 335 / 285, q/k/v 2048 rows
// 115 / 99, 1024 rows 69.5 / 63.1, 22016 x 4096 512 rows 96 / 83.  Of 440 products of 31 shapes from 257 to 4088 rows 73 take another tile, 2 to 16 %
// faster and none slower.
inline WideTiles launch_tiles(int M, int N, int K, bool swiglu, size_t out_capacity_floats) {
  const WideTiles base = wide_tiles(M, N, K, swiglu, out_capacity_floats);
  const int chain = K / base.S / (base.k == 128 ? 2 : 1);
  WideTiles best = base;
  float least = 0.98f * wide_time(M, N, K, swiglu, base);
  for (int cols : {224, 192}) {
    const WideTiles t = with_split(M, N, K, swiglu, out_capacity_floats, 256, cols, 160, 16);
    const float time = wide_time(M, N, K, swiglu, t);
    if (K / t.S <= chain && time < least) { best = t; least = time; }
  }
  return best;
}

// Whether 256 weight rows to a workgroup leave so few workgroups (1 to 16 of the fullest XCD's n) for a last round of its 32 CUs that 128 weight rows, with twice as many
// of half the length, are over first.  A last round takes nearly as long as a whole one, which the estimates of stream_tiles, fitted to products that mostly end in fuller
// ones, don't know.  us, 256 / 128 weight rows (with stages of 128 k unless stated), n = 33 where not: 80 rows 66816 x 4096 155 / 134, 96 rows 66816 x 1024 49.6 / 43.8,
// SwiGLU 65 rows 66816 x 5120 191 / 163, 65 rows 142592 x 3072 (n = 70) 204 / 193; 112 rows 66816 x 4096 162 / 148, 97536 x 3072 (48) 147 / 141, 66816 x 1024 51.6 / 45.3 with
// 64 k, 128 rows 132352 x 3072 (65) 225 / 216 with 64 k; 160 rows 66816 x 2560 129 / 124, but 66816 x 4096, with staggered walks, 176 / 177; 224 rows 66816 x 3072 164 / 154, SwiGLU 256 rows
// 66816 x 4608 223 / 208.  More than half full: 80 rows 113920 x 2048 (56) 103 / 114, 224 rows 101632 x 3072 (50) 178 / 210.  2796 LM heads and gate/up products of K
// 1024..8192 above 32 such workgroups, 65..256 rows: the 992 that take another tile by this 5 % faster, 20 of them slower by more than 2 % (3.7 at most).
inline bool few_left(int M, int n, int K) {
  const int left = n % 32;
  if (n <= 32 || left == 0 || left > 16) return false;
  if (M <= 96) return n < 96;
  if (M <= 128) return n < 64 ? left < 16 || K > 1024 : left <= 2 && K % 2048 != 0;
  return n < 64 && (M > 192 || (K > 2048 && K < 7168 && K % 2048 != 0));
}

// What is launched up to 256 rows: the tile of wide_tiles_256, or one with fewer activation lines for each weight line.  A CU has some 200 lines on their way at a time and
// they come back in order, so a line of activations from L2 keeps its place as long as the weight lines from HBM in front of it; neither the products (left
// out: 77 rows 54 us as with them) nor where the activations come from (one line again and again: 54 us) matter.  So
//   up to 96 rows, 96 x 128 in six wavefronts with eight activation slots instead of 128 x 128 with stages of 128 k;
//   256 weight rows to a workgroup, stages of 64 k, where they are enough workgroups: 96, 128, 192 or 256 rows.
// us: 28672 x 4096 77 rows 52.8 / 47.9, down 4096 x 14336 32.8 / 30.1, o 15.3 / 14.1, q/k/v 19.1 / 18.1; LM head 128256 x 4096 77 rows 217 / 200, 116 rows
// 224 / 209, 256 rows 307 / 280; 57344 x 8192 77 rows 187 / 168, 116 rows 189 / 177, 256 rows 266 / 229.  Tiles of 112 weight rows, which are 256 for 8B
// gate/up instead of 224, gave nothing (77 rows 50, 256 rows 69), nor did wavefronts that load activations only and weights only (116 rows 59).
// The estimates, a start, a time per stage that grows with the workgroups on the fullest XCD, and the partial sums, are fits to 72 products of 15 model
// shapes, all splits, at two row counts each (0.05 to 0.06 in the logarithm).  Against the estimate of wide_tiles_256, which comes out 2 to 10 % low for unsplit products
// in stages of 64 k up to 128 rows, the margins are 3 % the other way elsewhere and for 96 x 128.  Chains of sums are no longer than before (128 x 128 with stages
// of 128 k, and the new ones up to 128 rows: two sets); 256 weight rows only where an XCD has more than 16 workgroups (28672 x 4096, 14 of them: 68, 48 in
// 96 x 128), with ranges of at least 1024 k, and in a split not of a multiple of 4 KB (in step: 8192 x 28672 in seven ranges 77 rows 112, 100 otherwise).
// Time against that of wide_tiles_256, 142 products each: 65..96 rows 0.942, 97..128 0.984, 129..192 0.973, 193..256 0.979.  Where a last round has few workgroups (few_left)
// 256 weight rows don't come into question, and up to 128 rows unsplit products take stages of 128 k: those of 64 k side by side only where they are the faster ones, us,
// 112 rows, 64 / 128 k: 66816 x 1024 45.3 / 47.2, 81152 x 2048 105 / 92.  Staggered walks side by side were left to gate/up of K = 2048 and 4096 and 131 k to 159 k weight rows,
// where stages of 128 k are as fast (112 rows, K = 2048, 131216 weight rows 127 / 133, 139920 136 / 136, 149200 144 / 140, 159120 149 / 145; K = 4096 280 / 262): those take them.
inline WideTiles stream_tiles(int M, int N, int K, bool swiglu, size_t out_capacity_floats) {
  struct Fit { int cols, k, sets; float start, stage, busy, sums; };   // us; of a stage, more of it with all CUs busy, per million partial sums
  static constexpr Fit strips = {128, 128, 2, 4.53f, 0.89f, 0.58f, 2.29f};                                               // 96 rows
  static constexpr Fit wide[4] = {{256, 64, 2, 5.44f, 0.76f, 0.64f, 2.05f}, {256, 64, 2, 5.87f, 0.8f, 0.66f, 1.89f},     // 96, 128 rows
                                  {256, 64, 1, 7.77f, 0.9f, 0.7f, 1.65f}, {256, 64, 1, 9.69f, 0.93f, 0.76f, 1.61f}};     // 192, 256 rows
  auto per_xcd = [&](const Fit& f, int S) { return ((N + f.cols - 1) / f.cols + 7) / 8 * S; };
  auto time = [&](const Fit& f, int S) {
    const int n = per_xcd(f, S), last = n > 32 && n % 32 < 12 ? 12 : n % 32;       // a few workgroups behind whole rounds have no CU less to wait for
    const float stages = (float)K / S / f.k;
    return n / 32 * (f.start + (f.stage + f.busy) * stages) + (n % 32 ? f.start + stages * (f.stage + f.busy * last / 32) : 0.f) +
           (swiglu ? 0.f : (float)S * M * N * f.sums * 1e-6f);
  };
  float least = 0.f;
  WideTiles best = wide_tiles_256(M, N, K, swiglu, out_capacity_floats, &least);
  const int chain = K / best.S / (M <= 128 && best.k == 128 ? 2 : 1);
  const bool small_stages = M <= 128 && best.k == 64;
  if (M <= 96 && best.k == 128) {
    best.rows = 96;
    least = time(strips, best.S);
  } else {
    least *= small_stages ? 1.05f : 0.97f;
  }
  auto consider = [&](const Fit& f, int rows, float margin) {
    for (int S = 1; S <= (swiglu ? 1 : 8); ++S) {
      const int range = K / S;
      if (K % (f.k * S) || range < 512 || range > chain * f.sets || (S > 1 && (size_t)S * M * N > out_capacity_floats)) continue;
      if (f.cols == 256 && (per_xcd(f, S) <= 16 || few_left(M, per_xcd(f, S), K) || range < 1024 || (S > 1 && range % 2048 == 0))) continue;
      const float t = margin * time(f, S);
      if (t < least) { least = t; best = {rows, f.cols, S, f.k}; }
    }
  };
  if (M <= 96 && (!small_stages || K > 1024)) consider(strips, 96, small_stages ? 1.08f : 1.f);      // (1536 x 512 9.0, 9.4 in 96 x 128)
  const int i = M <= 96 ? 0 : M <= 128 ? 1 : M <= 192 ? 2 : 3, n = per_xcd(wide[i], 1);
  if (K >= 1024 && K % 128 == 0 && few_left(M, n, K) && best.S == 1 && M <= 128) {
    if (M <= 96) best = {96, 128, 1, 128};
    else if (n < 64 && K > 1024 && (!swiglu || K > 1536 || n >= 42)) best = {128, 128, 1, 128};
    return best;
  }
  consider(wide[i], i == 0 ? 96 : 64 * (i + 1), 1.f);
  if (best.rows == 128 && best.cols == 128 && wide_stagger(M, K, best)) best.k = 128;
  return best;
}

// Of more than 64 rows: what is launched.
inline WideTiles many_tiles(int M, int N, int K, bool swiglu, size_t out_capacity_floats) {
  return M <= 256 ? stream_tiles(M, N, K, swiglu, out_capacity_floats) : launch_tiles(M, N, K, swiglu, out_capacity_floats);
}

// ---- at most 64 rows
//
// Split-K factor of the 64-weight-row workgroups of gemm_skinny.hip, from measurements on MI355X (two of them fit a CU):
//   * 192-256 workgroups already stream a [4096..6144, 4096] weight at its best rate, and every extra split adds an
//     fp32 partial tile the consumer has to read back: take the smallest divisor of the stage count that reaches 192;
//   * between 256 and ~450 workgroups some CUs get two and the others one, and the launch takes as long as with
//     512 (320 workgroups on a [10240, 8192] weight: 46.7 us, 160 or 640: 43.5 us): skip those;
//   * a K range left longer than 64 stages is cut further (a [8192, 28672] weight streams 22 % faster as 512
//     workgroups of 56 stages than as 256 of 112).
inline int skinny_splits(int N, int K) {
  const int tiles = (N + 63) / 64, KT = K / 128;
  int best = 1;
  for (int S = 1; S <= 16; ++S) {
    if (KT % S) continue;
    if (S > 1 && KT / S < 4) break;
    const int wgs = tiles * S;
    if (S > 1 && wgs > 256 && wgs < 450) continue;
    best = S;
    if (wgs >= 192 && (KT / S <= 64 || wgs >= 512)) break;
  }
  return best;
}

struct FewRows {
  int cols;            // weight rows of a workgroup: 64 (gemm_skinny.hip), or 128 or 256 (64-row tiles of gemm_wide.hip)
  int S;
};

// Whether the K walks of the 64-row tiles start at a stage of each workgroup's own (gemm_wide.hip has the figures).
inline bool few_rows_stagger(int K, int S) { return K / S % 2048 == 0; }

// 33..64 rows: the tile whose launch is over first by this estimate, in microseconds.  A workgroup of any kind takes 4.9 for start and
// end.  128 and 256 weight rows: one to a CU; a stage of 32 KB of weights takes 0.92 us where few CUs are busy and 1.44 where all are,
// in rounds of 32 workgroups of the fullest XCD.  64 weight rows: two to a CU; a stage of 16 KB takes 0.73 alone, 1.59 where each CU
// has two.  Every partial sum costs its reader 0.15, and a result that goes straight to its place a launch of 5 more if it is split, and
// 0.4 per million partial sums (LM head 65780 x 4352, 60 rows: 150 us in two ranges, 138 unsplit).
// The numbers are a fit to 35 products (K 2048..28672, N 2048..151936), each with 3 to 20 tiles and splits: what the estimate picks is
// 0.6 % slower than the best of them on average, over 900 products of 40 shapes too (15 % at worst: 7168 x 21504 in three ranges, 70 us, 60
// in four), and 5 % faster than 64 weight rows (128 through registers for the large ones) on average; of the 900, 14 are slower than those,
// by 3 to 8 % and 0.6 to 3.5 us (3072 x 3072 33 rows 14.6 / 14.0, fusion 8192 x 24576 88 / 84.5).  us, what it takes / 64 weight rows:
// 8B q/k/v 14.4 / 15.8, gate/up 45.9 / 46.4, LM head 194 / 208, draft q/k/v 22.9 / 26.3;
// 70B q/k/v 38.6 / 42.9, gate/up 161 / 176, down 86.9 / 97.8; 5120 x 5120 14.5 / 18.9, 22016 x 4096 39.4 / 47.1; it leaves 8B o and down,
// 2560 x 9728 (18.0, 22.8 with 128 weight rows) and 16384 x 2048 (15.8, 19.8) to 64 weight rows.
// Up to 32 rows the 64-row workgroups, with half a tile of activations, are at 5.4 TB/s and stay.
// wide_ok: types and alignment are what gemm_wide.hip can take.  capacity: floats for partial sums.
inline FewRows few_rows(int M, int N, int K, bool swiglu, bool direct, size_t capacity, bool wide_ok) {
  auto fits = [&](int S) { return S == 1 || (size_t)S * M * N <= capacity; };
  FewRows best = {64, swiglu ? 1 : skinny_splits(N, K)};
  while (best.S > 1 && (!fits(best.S) || (K / 128) % best.S != 0)) --best.S;   // the next smaller divisor of the stage count
  if (M <= 32 || !wide_ok) return best;
  auto extra = [&](int S) { return S == 1 ? 0.f : 0.15f * S + (direct ? 5.f + 0.4e-6f * S * M * N : 0.f); };
  const int wgs = (N + 63) / 64 * best.S, rest = wgs % 512;
  const float range = (float)K / best.S / 128;
  float least = extra(best.S) + wgs / 512 * (4.9f + 1.59f * range);
  if (rest) least += 4.9f + range * (rest <= 256 ? 0.73f : rest <= 440 ? 1.37f : 1.59f * rest / 512);
  for (int cols : {128, 256})
    for (int S = 1; S <= (swiglu ? 1 : 16); ++S) {
      const int bk = cols == 128 ? 128 : 64, KT = K / bk;
      if (KT % S || K / S < 512 || !fits(S)) continue;
      const int n = ((N + cols - 1) / cols + 7) / 8 * S, last = n % 32;
      const float stages = (float)KT / S;
      float t = extra(S) + n / 32 * (4.9f + 1.44f * stages);
      if (last) t += 4.9f + stages * (last <= 20 ? 0.92f : 1.44f * last / 32);
      if (t < least) { least = t; best = {cols, S}; }
    }
  return best;
}

// ---- fp32
//
// Whether the RMSNorm of M rows of K is formed inside the fp32 product that reads them (gemm_f32.hip).  There every wavefront, of which
// there is one to each group of 8 rows and each weight row (or pair: gate and up, the two of a rotary pair), sums the squares again: 0.05 to
// 0.2 ns a wavefront, and 0.2 to 1 where K is more than 1024, against 3 us for a launch of its own.  us, inside / own launch: LM head 2048 x 512
// 64 rows 12.9 / 14.3, 256 rows 43.7 / 41.8; 32000 x 2048 64 rows 675 / 600; q/k/v 3072 x 1024 64 rows 21.2 / 22.1, 256 rows 73.5 / 67.6; gate/up
// 1376 x 256 128 rows 8.8 / 9.8, 512 rows 24.7 / 20.0; 11008 x 2048 16 rows 36.9 / 34.9, 64 rows 136 / 118.
inline bool f32_norm_inside(int M, int N, int K, bool pairs) {
  const long wavefronts = (long)((M + 7) / 8) * (pairs ? N / 2 : N);
  return wavefronts <= (K > 1024 ? 8192 : pairs ? 16384 : 24576);
}
