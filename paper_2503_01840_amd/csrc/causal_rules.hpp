// How many rows a workgroup of the causal attention kernel (causal_attention.hip) has, and which prompts take it.  Host arithmetic only.
#pragma once
#include <algorithm>

constexpr int CAUSAL_KEYS = 128;             // of a tile

// 32 RG rows per workgroup: as many heads of one KV head as divide its group (4, 2 or 1, and no more than RG) x the matching
// number of queries
inline int causal_heads_per_wg(int H, int Hkv, int RG) {
  const int G = H / Hkv;
  return G % 4 == 0 && RG >= 4 ? 4 : G % 2 == 0 ? 2 : 1;
}
inline int causal_workgroups(int T, int H, int Hkv, int RG) {
  const int hg = causal_heads_per_wg(H, Hkv, RG), qb = 32 * RG / hg;
  return H / hg * ((T + qb - 1) / qb);
}

// Workgroups of 64 rows instead of 128 where those leave CUs idle: a lone wavefront on a SIMD then takes 1.4 us per tile instead of the 2.0 to 2.4 that
// two take side by side, and there are twice as many workgroups.  Up to 256 of them each has a CU to itself (64-row
// form against 128-row form, us: 4 heads 4096 positions 49 / 66, 8 heads 2048 positions 28.1 / 36.9, 32 heads over 8 300
// positions 9.2 / 10.9).  Up to 512, the shorter half of them (workgroup i of w walks over 1 - i / w of the tiles) starts on the CUs that are
// done with the longer half's shorter ones, and pays the start, the own keys and the merge again: 32 over 8 517 positions 12.0 / 14.8, 900 positions 20.5 / 21.4,
// but 64 over 8 300 positions with 3 simulated steps 16.7 / 13.1, and 1000 positions of 32 over 8 with 3 steps 27.0 / 25.4.  The constants are fitted to both forms at
// 198 sizes (33..2048 positions, 8 to 64 heads over 4 to 32, 0 to 6 steps); what they pick is 0.06 % slower than the better form on average, 2.3 % at worst (those of
// the kernel before its softmax was spread over all products, 1.81 and 2.39 us a tile: 0.3 % and 9 %, 400 positions of 40 heads over 8 with 2 steps 16.3 / 14.9).  Beyond 512 the
// shared tiles win: 1100 positions of 32 over 8 29.8 / 25.4.
inline bool causal_half_workgroups(int T, int H, int Hkv, int s) {
  const int w = causal_workgroups(T, H, Hkv, 2);
  if (w <= 256) return true;
  if (w > 512) return false;
  const float tiles = 0.5f * ((T + CAUSAL_KEYS / 2 - 1) / (CAUSAL_KEYS / 2));    // a last tile of no more than 64 keys takes half of a tile's time
  auto fixed = [&](int RG, float start, float batch) { const int hg = causal_heads_per_wg(H, Hkv, RG); return start + batch * ((s + hg - 1) / hg); };
  const float start2 = fixed(2, 5.2f, 2.f), two = 2.f * (1.5f * tiles * (1.f - 256.f / w) + start2);
  return std::max(1.5f * tiles + start2, two) < 2.4f * tiles + fixed(4, 5.5f, 1.8f);
}

// Whether this kernel, which does not split the keys, is the better one for n rows of a prompt that see up to max_len keys.  Against the tree kernel, which cuts the keys
// into splits and merges them (us, 32 heads over 8 unless stated, tree / this kernel):
//   more than 128 workgroups: the tree kernel has two for each of them, more than CUs, and the last few take as long as all, at any
//     length: 640 rows (160) behind 1500 positions 58 / 37, 513 rows (136) behind 16 k 340 / 257, 1024 rows behind 2048 83 / 63; but 449 rows (120) behind 16 k
//     196 / 254;
//   walks so short that the merge costs more than the idle CUs: up to 4 tiles, 100 rows behind 128 positions 13.3 / 8.7, 384 rows behind 64 21.6 / 12.0;
//   between the two the line runs near 6.5 workgroups per tile of walk: 300 rows (80) and 11 tiles 35.7 / 25.2, 256 rows (64) and 10 tiles 24.0 / 24.3.  Where a
//     group has one head, or an odd number, so that a workgroup's rows are of one head, the tree kernel's are the fuller ones and it is near 10: 16 heads over 16 300
//     rows (48) and 8 tiles 16.6 / 20.2, 32 over 32 160 rows (64) and 9 tiles 18.5 / 21.8.
// What it picks of both at 2504 prompts (17..1025 rows behind 0 to 16 k positions, 8 to 64 heads over 2 to 32) is 1.5 % slower than the better one on average.  (The line of the former
// kernels, 192 workgroups or 10 to a tile, 5.2 %; 284 of them take the other kernel now, 24 % faster, and 2 of those are slower, by 2 %.)  The error against 64 bits is
// that of rounding the output to bf16 in both (1.660e-3 each).
inline bool prefill_attention_fits(int n, int H, int Hkv, int max_len) {
  const int wgs = causal_workgroups(n, H, Hkv, 4), tiles = (max_len + CAUSAL_KEYS - 1) / CAUSAL_KEYS;
  return wgs > 128 || tiles <= 4 || 2 * wgs >= (causal_heads_per_wg(H, Hkv, 4) == 1 ? 20 : 13) * tiles;
}
