"""Where the workgroups of a many-row product work (host and device code, compiled with the host compiler; no GPU): over a whole launch every weight tile,
activation-row block and K range comes exactly once, and what is left is past the last tile."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_tile_block_and_range_comes_once(tmp_path):
    (tmp_path / "m.cpp").write_text('''#include <cstdio>
#include <vector>
#include "wide_places.hpp"
int main() {
  long launches = 0;
  for (int tiles : {1, 2, 3, 7, 8, 9, 15, 20, 24, 31, 32, 33, 56, 112, 257, 501})
    for (int mblocks : {1, 2, 3, 5, 6, 7, 8, 11, 16, 22, 63, 91, 127, 1000, 4099})                     // up to 393 k rows
      for (int S = 1; S <= 8; ++S)
        for (int ranges = 0; ranges <= 3 && S % (1 << ranges) == 0; ++ranges) {
          if ((long)tiles * mblocks * S > 1500000) continue;
          const WideGrid grid = wide_grid(tiles, mblocks, S, ranges);
          if (grid.x % 8) { printf("x is no multiple of 8\\n"); return 1; }                               // the XCD of a workgroup is x % 8
          const Divisor by = divisor(mblocks);
          std::vector<unsigned char> seen((size_t)tiles * mblocks * S);
          for (int y = 0; y < grid.y; ++y)
            for (int x = 0; x < grid.x; ++x) {
              const WidePlace p = wide_place(x, y, ranges, by);
              if (p.tile >= tiles) continue;
              if (p.tile < 0 || p.mblock < 0 || p.mblock >= mblocks || p.split < 0 || p.split >= S || p.split % (1 << ranges) != (x & 7) % (1 << ranges) ||
                  seen[((size_t)p.tile * mblocks + p.mblock) * S + p.split]++) {
                printf("%d tiles, %d blocks, %d ranges by %d: workgroup %d, %d\\n", tiles, mblocks, S, 1 << ranges, x, y);
                return 1;
              }
            }
          for (unsigned char s : seen)
            if (!s) { printf("%d tiles, %d blocks, %d ranges by %d: one is missing\\n", tiles, mblocks, S, 1 << ranges); return 1; }
          ++launches;
        }
  return launches < 3000;
}
''')
    inc = os.path.join(ROOT, "paper_2503_01840_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", inc, str(tmp_path / "m.cpp"), "-o", str(tmp_path / "m")], check=True)
    r = subprocess.run([str(tmp_path / "m")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
