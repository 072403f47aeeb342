"""The tiles that products of 65..256 rows are launched in (host code, compiled with the host compiler; no GPU): that they can be, against what was
measured, and which of them the GPU tests of test_gpu_stream_tiles.py run."""
import os
import subprocess

import pytest

from test_wide_tiles import BIG, MODELS, ROOT, _products


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    """(M, N, K, SwiGLU, capacity) -> (rows, cols, S, k of a stage, staggered) of the launch of at most 256 rows, and the same of the tile without activation lines in mind"""
    d = tmp_path_factory.mktemp("tiles")
    (d / "m.cpp").write_text('#include <cstdio>\n#include "wide_tiles.hpp"\n'
                             'int main() { int m, n, k, s; long long c; while (scanf("%d %d %d %d %lld", &m, &n, &k, &s, &c) == 5) {\n'
                             '  for (const WideTiles& t : {many_tiles(m, n, k, s, c), wide_tiles_256(m, n, k, s, c)})\n'
                             '    printf("%d %d %d %d %d ", t.rows, t.cols, t.S, t.k, wide_stagger(m, k, t));\n  puts(""); } }\n')
    inc = os.path.join(ROOT, "paper_2503_01840_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", inc, str(d / "m.cpp"), "-o", str(d / "m")], check=True)

    def ask(queries):
        text = "\n".join(" ".join(map(str, q)) for q in queries) + "\n"
        out = subprocess.run([str(d / "m")], input=text, capture_output=True, text=True, check=True).stdout
        return [(t[:5], t[5:]) for t in (tuple(map(int, line.split())) for line in out.splitlines())]
    return ask


def test_every_choice_can_be_launched_and_sums_in_chains_no_longer(rule):
    qs = [(M, N, K, s, cap) for M in (65, 80, 96, 97, 128, 129, 192, 193, 256) for N in (8, 256, 768, 4096, 5120, 10240, 28672, 64000, 128256)
          for K in (128, 256, 512, 1408, 2304, 4096, 7168, 11008, 14336, 28672) for s in (0, 1) for cap in (0, 2048 * 5120, BIG)]
    qs += [(M, N, K, s, 0) for M in (65, 96, 97, 128, 129, 256) for N in (66816, 97536) for K in (1088, 2112) for s in (0, 1)]      # odd numbers of 64-k stages
    qs += [(M, N, K, 1, 0) for M in (97, 112, 128) for N in (131216, 149200, 159120) for K in (2048, 4096)]
    seen = set()
    for (M, N, K, s, cap), ((rows, cols, S, k, staggered), base) in zip(qs, rule(qs)):
        seen.add((rows, cols, k))
        assert not (staggered and (rows, cols, k) == (128, 128, 64))                       # there is no such kernel
        assert M <= rows and (rows, cols, k) in {(96, 128, 128), (96, 256, 64), (128, 128, 64), (128, 128, 128), (128, 256, 64), (192, 256, 64), (256, 128, 64),
                                                 (256, 128, 128), (256, 256, 64)}
        assert K % (S * k) == 0 and 1 <= S <= 8 and (S == 1 or (not s and S * M * N <= cap))
        chains = lambda t: 2 if M <= 128 and (t[3] == 128 or t[1] == 256) else 1                   # sets of sums of the kernels of gemm_wide.hip
        assert K / S / chains((rows, cols, S, k)) <= K / base[2] / chains(base)
    assert {(96, 128, 128), (96, 256, 64), (128, 256, 64), (192, 256, 64), (256, 256, 64)} <= seen


# (rows, outputs, inputs, SwiGLU): microseconds in the tile of wide_tiles_256, in 256 weight rows to a workgroup
@pytest.mark.parametrize("q,other,wide", [
    ((77, 128256, 4096, 0), 217, 200), ((116, 128256, 4096, 0), 224, 209), ((256, 128256, 4096, 0), 307, 280), ((77, 57344, 8192, 1), 187, 168),
    ((116, 57344, 8192, 1), 189, 177), ((256, 57344, 8192, 1), 266, 229), ((77, 37888, 3584, 1), 80, 67), ((77, 34816, 5120, 1), 116, 96),
    ((77, 28672, 4096, 1), 48, 69), ((77, 27648, 5120, 1), 60, 89), ((77, 8192, 28672, 0), 101, 112), ((256, 10240, 8192, 0), 73, 78), ((192, 2048, 512, 1), 12, 16)])
def test_256_weight_rows_where_they_are_the_faster_ones(rule, q, other, wide):
    assert (rule([q + (BIG if q[1] < 20000 else 0,)])[0][0][1] == 256) == (wide < other)


# unsplit, where 256 weight rows leave 1 to 16 workgroups of the fullest XCD for a last round, and beside that: microseconds in 128 weight rows (of 96 rows and 128 k up to 96
# rows; of 64 k where that is noted), in 256
@pytest.mark.parametrize("q,narrow,wide,k", [
    ((80, 66816, 4096, 0), 134, 155, 128), ((96, 66816, 1024, 0), 43.8, 49.6, 128), ((80, 81152, 2048, 0), 84.3, 89.8, 128), ((65, 66816, 5120, 1), 163, 191, 128),
    ((65, 142592, 3072, 0), 193, 204, 128), ((80, 113920, 2048, 0), 114, 103, 128), ((112, 66816, 4096, 0), 148, 162, 128), ((97, 66816, 5120, 1), 177, 195, 128),
    ((112, 66816, 1024, 0), 45.3, 51.6, 64), ((112, 97536, 3072, 0), 141, 147, 128), ((112, 113920, 3072, 0), 169, 157, 128), ((128, 132352, 3072, 0), 214, 225, 64),
    ((160, 66816, 2560, 0), 124, 129, 128), ((160, 65792, 4352, 0), 188, 199, 128), ((192, 65792, 4352, 0), 192, 200, 128), ((160, 66816, 4096, 0), 177, 176, 128),
    ((224, 66816, 3072, 0), 154, 164, 128), ((224, 81152, 3072, 1), 150, 156, 128), ((256, 66816, 4608, 1), 208, 223, 128), ((224, 101632, 3072, 0), 210, 178, 128)])
def test_128_weight_rows_where_256_leave_few_workgroups_for_a_last_round(rule, q, narrow, wide, k):
    M = q[0]
    rows, cols, S, stage, _ = rule([q + (0,)])[0][0]
    if narrow < wide:
        assert (rows, cols, S, stage) == (96 if M <= 96 else 128 if M <= 128 else 256, 128, 1, k)
    else:
        assert (rows, cols, S, stage) == (96 if M <= 96 else 64 * ((M + 63) // 64), 256, 1, 64)


MODELS["split"] = (5120, 40, 8, 17408, 20484)


# (rows, cols, S, k, staggered) of some of q/k/v, o, gate/up, down and the LM head
@pytest.mark.parametrize("model,M,at,want", [
    ("8b", 65, (0, 1, 2, 3, 4), [(96, 128, 4, 128, 0), (96, 128, 8, 128, 0), (96, 128, 1, 128, 1), (96, 128, 8, 128, 0), (96, 256, 1, 64, 1)]),
    ("8b", 96, (2, 4), [(96, 128, 1, 128, 1), (96, 256, 1, 64, 1)]), ("8b", 97, (4,), [(128, 256, 1, 64, 1)]), ("8b", 127, (4,), [(128, 256, 1, 64, 1)]),
    ("8b", 191, (4,), [(192, 256, 1, 64, 1)]), ("8b", 193, (4,), [(256, 256, 1, 64, 1)]), ("8b", 255, (4,), [(256, 256, 1, 64, 1)]),
    ("wide", 80, (0, 2, 4), [(96, 128, 4, 128, 0), (96, 256, 1, 64, 0), (96, 256, 1, 64, 0)]), ("wide", 127, (2, 4), [(128, 256, 1, 64, 0), (128, 256, 1, 64, 0)]),
    ("wide", 192, (2, 4), [(192, 256, 1, 64, 0), (192, 256, 1, 64, 0)]), ("wide", 255, (2, 4), [(256, 256, 1, 64, 0), (256, 256, 1, 64, 0)]),
    ("split", 90, (1, 3, 4), [(96, 128, 5, 128, 0), (96, 128, 4, 128, 0), (96, 128, 1, 128, 0)]), ("split", 180, (3,), [(192, 256, 8, 64, 0)]),
])
def test_tiles_that_the_gpu_tests_cover(rule, model, M, at, want):
    ps = _products(model, M)
    assert [t for t, _ in rule([(M, *ps[i][:3], ps[i][4]) for i in at])] == want
