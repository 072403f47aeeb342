// Which output tile the many-row product takes, and into how many K ranges it is cut.  Host arithmetic only.
//
// Workgroups of one weight tile go to one XCD (32 CUs): a launch lasts as many rounds as the fullest XCD has workgroups per CU,
// and that XCD has ceil(weight tiles / 8) of them for every row block and K range.
#pragma once
#include <cstddef>

struct WideTiles {
  int rows, cols;      // output tile of a workgroup
  int S;               // K ranges (split-K partial sums); 1 for SwiGLU
  int k;               // width of a weight stage: 64, or 128 for tiles of 128 weight rows
};

inline WideTiles wide_tiles_k64(int M, int N, int K, bool swiglu, size_t out_capacity_floats) {
  const int KT = K / 64;
  auto ceil_div = [](int a, int b) { return (a + b - 1) / b; };
  auto pick = [&](int rows, int cols, int want, int min_stages) -> WideTiles {
    const int wgs = ceil_div(N, cols) * ceil_div(M, rows);
    int S = 1;
    if (!swiglu)
      for (int s = 1; s <= 8 && wgs * S < want; ++s) {
        if (KT % s) continue;
        if (s > 1 && ((size_t)s * M * N > out_capacity_floats || KT / s < min_stages)) break;
        S = s;
      }
    return {rows, cols, S, 64};
  };
  // 129..256 rows: ONE 256-row block x 128 weight rows per workgroup (8 wavefronts x 64 x 64), so that every weight line enters
  // exactly one CU and a stage takes in 48 KB instead of the 2 x 32 KB of two 128 x 128 workgroups (measured at 256 rows, 8B
  // shapes: q/k/v 33.4 -> 26.6 us, down 54.3 -> 47.6, gate/up 86.0 -> 78.9)
  if (M > 128 && M <= 256) return pick(256, 128, 192, 8);
  // 256 x 256 tiles when there are enough rows and, with at least 16 stages left per workgroup after split-K, enough workgroups;
  // else 128 x 128 tiles, two workgroups per CU
  const WideTiles big = pick(256, 256, 160, 16);
  const bool few = M < 384 || (ceil_div(N, 256) * ceil_div(M, 256) * big.S < 160 && !swiglu);
  const WideTiles t = few ? pick(128, 128, 384, 8) : big;
  if (few && !(swiglu && M > 256)) return t;
  // 192 x 256 tiles where the fullest XCD gets done sooner with them.  Unit: a 256 x 256 workgroup's walk over all of K; 192 rows
  // take 0.8 of it, two 128 x 128 workgroups on one CU 0.6, one alone 0.4.  Over eleven model widths from 256 to 8192, 257..2048
  // rows, no product becomes slower by this rule (more than 2.5 %), and of those that would gain two are missed.  8B width, 256
  // (or 128) -> 192 rows, us: gate/up 300 rows 120 -> 86, 520 rows 194 -> 160, 1100 rows 302 -> 257; q/k/v 600 rows 67 -> 47; down
  // 1100 rows 167 -> 133.  Not taken: gate/up 2048 rows 423 / 446; hidden 5120, o at 400 rows 40 / 61 (36 instead of 24
  // workgroups on an XCD: a second round); hidden 2048, gate/up at 300 rows 30 / 41 (one 128 x 128 workgroup per CU).
  const WideTiles mid = pick(192, 256, 160, 16);
  auto per_xcd = [&](const WideTiles& w) { return ceil_div(ceil_div(N, w.cols), 8) * ceil_div(M, w.rows) * w.S; };
  auto cost = [&](const WideTiles& w) -> float {
    const int n = per_xcd(w);
    if (w.cols == 256) return ceil_div(n, 32) * (w.rows == 256 ? 1.f : 0.8f) / w.S;
    const int rest = n % 64;
    return (n / 64 * 0.6f + (rest == 0 ? 0.f : rest <= 32 ? 0.4f : 0.6f)) / w.S;
  };
  return cost(mid) < cost(t) ? mid : t;
}

// Tiles of 128 weight rows leave room in LDS for weight stages of 128 k, whose row pieces of 256 bytes HBM delivers faster than
// pieces of 128, where one workgroup has a CU to itself.  256 x 128 always has; 128 x 128 runs two to a CU otherwise, and that
// is the better way between 257 and 512 workgroups (one round of two against two of one), and beyond where row blocks share a weight tile.  A workgroup's walk has to be long
// enough, as fewer and larger stages start later.  8B and 70B widths, us, 64 / 128: 77 rows gate/up (224 workgroups) 59.1 / 54.7, LM
// head (1002) 256 / 242, down (256, 14 stages) 28.9 / 28.1, but o (256, 4 stages) 12.6 / 13.8, q/k/v (384) 18.6 / 22.4 and 70B gate/up
// (448) 185 / 201; 300 rows LM head (3006) 457 / 530; 256 rows gate/up 71.8 / 69.5, q/k/v 24.2 / 23.6, but o (4 stages) 17.8 / 18.4.
inline WideTiles wide_tiles(int M, int N, int K, bool swiglu, size_t out_capacity_floats) {
  WideTiles t = wide_tiles_k64(M, N, K, swiglu, out_capacity_floats);
  const int wgs = (N + t.cols - 1) / t.cols * ((M + t.rows - 1) / t.rows) * t.S, range = K / t.S;
  if (t.cols == 128 && range % 128 == 0 && range >= (t.rows == 256 && t.S == 1 ? 256 : 1024) &&
      (t.rows == 256 || wgs <= 256 || (wgs > 512 && M <= 128)))
    t.k = 128;
  return t;
}
