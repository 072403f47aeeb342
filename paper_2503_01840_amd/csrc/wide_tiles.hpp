// Which output tile the many-row product takes, and into how many K ranges it is cut.  Host arithmetic only.
//
// Workgroups of one weight tile go to one XCD (32 CUs): a launch lasts as many rounds as the fullest XCD has workgroups per CU,
// and that XCD has ceil(weight tiles / 8) of them for every row block and K range.
#pragma once
#include <cstddef>
#include <initializer_list>

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
  if (M <= 128) return pick(128, 128, 384, 8);
  // More rows: the tile whose launch is over first by this estimate, in microseconds.  A workgroup takes a start and an end, and a
  // time per 64 k; the fullest XCD runs its workgroups in rounds of 32, of 64 for 128 x 128 tiles (two on a CU side by side, one
  // alone where there are no more than 32 left); the consumer then reads the partial sums (5 TB/s).  The ten numbers are a fit to 17 products
  // of the 8B, 70B and two narrower widths at 16 row counts from 257 to 2048, each with all four tiles: what the estimate picks is 0.3 %
  // slower than the best of the four on average (15 % at worst: gate/up of hidden 2048, 576 and 1300 rows), and 6 % faster than
  // picking by workgroup counts.  8B width, product and reading, us, 256 x 256 / 192 x 256 / 256 x 128 / 128 x 128: q/k/v 300 rows
  // 38 / 35 / 36 / 44, 512 rows 44 / 64 / 40 / 50; down 300 rows 63 / 58 / 60 / 69, 512 rows 73 / 80 / 67 / 83; o 1024 rows 49 / 49 / 42 / 50;
  // gate/up 300 rows 101 / 88 / 117 / 119, 1024 rows 197 / 235 / 231 / 274, 2048 rows 384 / 395 / 426 / 507; hidden 2048, gate/up 450 rows
  // 47 / 41 / 32 / 41.
  auto cost = [&](const WideTiles& w) -> float {
    const int n = ceil_div(ceil_div(N, w.cols), 8) * ceil_div(M, w.rows) * w.S;
    const float stages = (float)KT / w.S, read = swiglu ? 0.f : (float)w.S * M * N * (4.f / 5e6f);
    if (w.cols == 256) return ceil_div(n, 32) * (w.rows == 256 ? 8.72f + 1.43f * stages : 8.0f + 1.14f * stages) + read;
    if (w.rows == 256) return ceil_div(n, 32) * (6.74f + 0.85f * stages) + read;
    const float two = 8.4f + 1.13f * stages, one = 4.66f + 0.79f * stages;
    const int rest = n % 64;
    return n / 64 * two + (rest == 0 ? 0.f : rest <= 32 ? one : two) + read;
  };
  WideTiles best = pick(256, 256, 160, 16);
  for (const WideTiles& t : {pick(192, 256, 160, 16), pick(256, 128, 192, 16), pick(128, 128, 384, 8)})
    if (cost(t) < cost(best)) best = t;
  return best;
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
