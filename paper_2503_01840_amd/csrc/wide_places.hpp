// Which weight tile, activation-row block and K range each workgroup of a many-row product (gemm_wide.hip) has.  Host and device.
#pragma once
#include "divisor.hpp"

struct WidePlace {
  int tile, mblock, split;
};
struct WideGrid {
  int x, y;
};

// The launch: 8 XCDs x (groups of weight tiles x activation-row blocks), K ranges that one XCD goes through.  ranges: log2 of 1, 2, 4 or 8, whose power divides S;
// XCD x has the K ranges x % 2^ranges + 2^ranges i only.
inline WideGrid wide_grid(int tiles, int mblocks, int S, int ranges) {
  const int groups = (tiles + (8 >> ranges) - 1) >> (3 - ranges);
  return {8 * groups * mblocks, S >> ranges};
}

// Workgroups go to the XCDs round-robin by their linear id: x % 8 is the XCD, as the launch is a multiple of 8 wide.  Consecutive workgroups of one
// XCD take the activation-row blocks of ONE weight tile, so that the tile is fetched into that L2 once.  A tile past the last one has nothing to do.
HOST_AND_DEVICE WidePlace wide_place(int x, int y, int ranges, const Divisor& by_mblocks) {
  const int xcd = x & 7, j = x >> 3, group = j / by_mblocks;
  return {(group << (3 - ranges)) + (xcd >> ranges), j - group * by_mblocks.d, (y << ranges) + (xcd & ((1 << ranges) - 1))};
}
