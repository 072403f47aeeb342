"""The rules by which causal attention takes its workgroups and prompts their kernel (host code, compiled with the host compiler; no GPU), against what was measured on
both sides of their lines."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# training-time test, (positions, query heads, KV heads, simulated steps): microseconds with 64 rows to a workgroup, with 128
MEASURED_ROWS = [
    ((300, 32, 8, 0), 9.2, 10.9), ((2048, 8, 8, 0), 28.1, 36.9), ((4096, 4, 4, 0), 49.2, 66.2), ((517, 32, 8, 0), 12.0, 14.8), ((900, 32, 8, 0), 20.5, 21.4),
    ((600, 32, 8, 3), 18.2, 17.0), ((400, 40, 8, 2), 16.3, 14.9), ((900, 28, 4, 2), 24.4, 23.2), ((900, 32, 32, 1), 23.0, 24.2), ((2048, 16, 4, 6), 41.7, 43.2),
    ((1000, 32, 8, 0), 22.6, 23.3), ((1000, 32, 8, 3), 27.0, 25.4), ((300, 64, 8, 3), 16.7, 13.1), ((1100, 32, 8, 0), 29.8, 25.4),
]


def _ask(tmp_path, call, queries):
    n = len(queries[0])
    rows = ", ".join("{" + ", ".join(map(str, q)) + "}" for q in queries)
    (tmp_path / "m.cpp").write_text('#include <cstdio>\n#include "causal_rules.hpp"\nint main() { const int q[][%d] = {%s};\n'
                                    '  for (auto& c : q) printf("%%d\\n", (int)%s(c[0], c[1], c[2], c[3])); }\n' % (n, rows, call))
    inc = os.path.join(ROOT, "paper_2503_01840_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", inc, str(tmp_path / "m.cpp"), "-o", str(tmp_path / "m")], check=True)
    return list(map(int, subprocess.run([str(tmp_path / "m")], capture_output=True, text=True, check=True).stdout.split()))


def test_64_rows_to_a_workgroup_where_they_are_the_faster_ones(tmp_path):
    for (q, half, whole), got in zip(MEASURED_ROWS, _ask(tmp_path, "causal_half_workgroups", [q for q, _, _ in MEASURED_ROWS])):
        assert got == (half < whole), q


# prompts, (rows, query heads, KV heads, keys): microseconds in the tree kernel, in the unsplit one
MEASURED_PROMPTS = [
    ((640, 32, 8, 2140), 58.3, 37.5), ((513, 32, 8, 16513), 340.0, 256.7), ((641, 28, 4, 12641), 256.3, 203.9), ((1024, 32, 8, 3072), 82.9, 62.9), ((449, 32, 8, 16449), 196.1, 254.3),
    ((257, 64, 8, 8257), 183.2, 131.4), ((230, 64, 8, 8230), 106.5, 130.5), ((100, 32, 8, 228), 13.3, 8.7), ((384, 32, 8, 448), 21.6, 12.0), ((33, 32, 8, 33), 9.3, 5.8),
    ((300, 32, 8, 1300), 35.7, 25.2), ((200, 32, 8, 712), 19.6, 16.0), ((230, 32, 8, 2730), 32.7, 46.6), ((768, 8, 2, 1468), 23.1, 27.1), ((300, 16, 16, 1000), 16.6, 20.2),
    ((160, 32, 32, 1060), 18.5, 21.8), ((513, 32, 32, 8513), 166.1, 136.9), ((449, 32, 32, 8449), 119.1, 133.4), ((17, 40, 8, 617), 12.1, 14.7),
]


def test_prompts_in_the_kernel_that_is_the_faster_one(tmp_path):
    for (q, tree, unsplit), got in zip(MEASURED_PROMPTS, _ask(tmp_path, "prefill_attention_fits", [q for q, _, _ in MEASURED_PROMPTS])):
        assert got == (unsplit < tree), q
