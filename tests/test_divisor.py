"""Division by multiplication, as the kernels divide by sizes of a launch (host part compiled with the host compiler; no GPU): exact for every dividend below
2^31 at the multiples of the divisor and beside them, where a rounded factor goes wrong first."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_division_by_multiplication_is_exact(tmp_path):
    (tmp_path / "m.cpp").write_text('''#include <cstdio>
#include <initializer_list>
#include "divisor.hpp"
static long bad = 0;
static void at(uint64_t n, int d, const Divisor& by) {
  if (n >> 31) return;
  const int q = (int)n / by, r = (int)n % by;                       // the expressions that the kernels use
  if (q != (int)(n / d) || r != (int)(n % d)) { if (!bad++) printf("%llu / %d: %d, %d\\n", (unsigned long long)n, d, q, r); }
}
int main() {
  for (int64_t d = 1; d < (1ll << 31); d += d < 70000 ? 1 : d / 1000) {
    const Divisor by = divisor((int)d);
    if (by.d != d) return 2;
    const uint64_t last = ((1ull << 31) - 1) / d;
    for (uint64_t k : {0ull, 1ull, 2ull, 3ull, 1000ull, (unsigned long long)(last / 2), (unsigned long long)(last - (last > 0)), (unsigned long long)last})
      for (int o = -1; o <= 1; ++o)
        if (k * d + o != ~0ull) at(k * d + o, (int)d, by);
    at((1ull << 31) - 1, (int)d, by);
  }
  return bad != 0;
}
''')
    inc = os.path.join(ROOT, "paper_2503_01840_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", inc, str(tmp_path / "m.cpp"), "-o", str(tmp_path / "m")], check=True)
    r = subprocess.run([str(tmp_path / "m")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
