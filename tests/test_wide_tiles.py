"""The rules by which products take their tiles, splits, weight stages and walks (host code, compiled with the host compiler; no GPU): against
what was measured, and which of them the GPU tests of test_gpu_row_tiles.py run."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BIG = 1 << 40

# (rows M, outputs N, inputs K, SwiGLU): microseconds of the product and the kernel that reads it with the fastest of the other tiles, with
# 192-row tiles
MEASURED = [
    ((300, 28672, 4096, 1), 101, 87), ((520, 28672, 4096, 1), 161, 153), ((1100, 28672, 4096, 1), 263, 234),      # 8B width
    ((2048, 28672, 4096, 1), 382, 392), ((600, 6144, 4096, 0), 50, 52), ((768, 6144, 4096, 0), 75, 55), ((1100, 4096, 14336, 0), 154, 148),
    ((383, 57344, 8192, 1), 382, 325), ((600, 57344, 8192, 1), 546, 589), ((300, 10240, 5120, 0), 59, 65),          # 70B and 13B widths
    ((300, 2048, 512, 1), 8.6, 15), ((300, 5632, 1024, 1), 15, 24), ((2048, 5632, 1024, 1), 30, 44),                # narrow models
    ((300, 11264, 2048, 1), 30, 41), ((576, 11264, 2048, 1), 36, 42), ((2048, 11264, 2048, 1), 95, 115), ((383, 16384, 3072, 1), 47, 62),
    ((257, 18432, 2304, 1), 43, 48), ((300, 17920, 1536, 1), 31, 35), ((300, 4352, 17024, 0), 100, 114), ((300, 5120, 5120, 0), 40, 43),
    ((300, 37888, 3584, 1), 119, 135), ((400, 5120, 5120, 0), 48, 68), ((1024, 5120, 5120, 0), 78, 107),
    ((2048, 5120, 13824, 0), 286, 453), ((2048, 2560, 2560, 0), 59, 80), ((900, 2560, 6912, 0), 61, 87),
    ((1024, 5120, 3072, 0), 60, 79), ((900, 3072, 8192, 0), 70, 99), ((1100, 3072, 3072, 0), 43, 64),
]

# 97..128 rows that are launched in unsplit 128 x 128 tiles: microseconds with stages of 128 k, of 64 k
MEASURED_STAGES = [((128, 32768, 6144, 1), 83, 90), ((100, 27648, 5120, 1), 64, 71), ((112, 66816, 1024, 0), 47.2, 45.3), ((112, 81152, 2048, 0), 92, 105)]


@pytest.fixture(scope="module")
def whole_rule(tmp_path_factory):
    """(M, N, K, SwiGLU, capacity) -> (rows, cols, S, k of a stage, staggered) of the launch up to 256 rows; beyond, of the tile before 224 and 192 weight rows
    come into question (the launch: `launched`)"""
    d = tmp_path_factory.mktemp("tiles")
    (d / "m.cpp").write_text('#include <cstdio>\n#include "wide_tiles.hpp"\n'
                             'int main() { int m, n, k, s; long long c; while (scanf("%d %d %d %d %lld", &m, &n, &k, &s, &c) == 5) {\n'
                             '  WideTiles t = m <= 256 ? many_tiles(m, n, k, s, c) : wide_tiles(m, n, k, s, c); printf("%d %d %d %d %d\\n", t.rows, t.cols, t.S, t.k, wide_stagger(m, k, t)); } }\n')
    inc = os.path.join(ROOT, "paper_2503_01840_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", inc, str(d / "m.cpp"), "-o", str(d / "m")], check=True)

    def ask(queries):
        text = "\n".join(" ".join(map(str, q)) for q in queries) + "\n"
        out = subprocess.run([str(d / "m")], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return ask


@pytest.fixture(scope="module")
def rule(whole_rule):
    return lambda queries: [t[:3] for t in whole_rule(queries)]


def test_192_row_tiles_where_they_are_the_faster_ones(rule):
    for (q, without, with192), (rows, cols, S) in zip(MEASURED, rule([q + (BIG,) for q, _, _ in MEASURED])):
        assert (rows == 192) == (with192 < without), (q, rows, cols, S)


def test_every_choice_can_be_launched(rule):
    qs = [(M, N, K, s, cap) for M in (65, 128, 129, 256, 257, 383, 384, 520, 1000, 2048) for N in (256, 768, 5120, 28672)
          for K in (128, 256, 2816, 4096, 14336) for s in (0, 1) for cap in (0, 2048 * 5120, BIG)]
    tiles = {(256, 256), (192, 256), (256, 128), (128, 128), (128, 256), (96, 256), (96, 128)}
    for (M, N, K, s, cap), (rows, cols, S) in zip(qs, rule(qs)):
        assert (rows, cols) in tiles and (rows in (192, 256) or M <= 128 or (rows, cols) == (128, 128)) and 1 <= S <= 8 and (K // 64) % S == 0
        assert S == 1 or (not s and S * M * N <= cap)


# K a multiple of 128, and of the ranges only those of a split that 128 does not divide fill the chip: the split comes before wide stages
@pytest.mark.parametrize("N,K,S", [(512, 1408, 2), (1024, 2816, 4), (2048, 5632, 8), (3584, 18944, 8), (4096, 11008, 4)])
def test_splits_whose_ranges_128_does_not_divide(rule, N, K, S):
    assert rule([(M, N, K, 0, BIG) for M in (129, 160, 200, 256)]) == [(256, 128, S)] * 4


def test_weight_stages_where_they_are_the_faster_ones(whole_rule):
    for (q, wide, narrow), (rows, cols, S, k, _) in zip(MEASURED_STAGES, whole_rule([q + (0,) for q, _, _ in MEASURED_STAGES])):
        assert (rows, cols, S) == (128, 128, 1) and (k == 128) == (wide < narrow), (q, k)


def test_weight_stages_divide_every_range_of_k(tmp_path):
    (tmp_path / "m.cpp").write_text('#include <cstdio>\n#include <initializer_list>\n#include "wide_tiles.hpp"\n'
                                    'int main() { for (int M : {65, 77, 128, 129, 200, 256, 257, 300, 383, 520, 2048})\n'
                                    '  for (int N = 256; N <= 131072; N += N / 3) for (int K = 128; K <= 28672; K += 128) for (int s : {0, 1}) {\n'
                                    '    const WideTiles t = many_tiles(M, N, K, s, (size_t)1 << 40);\n'
                                    '    if (K / t.S % t.k || (t.k != 64 && (t.k != 128 || t.cols != 128))) { printf("%d %d %d %d\\n", M, N, K, s); return 1; } }\n'
                                    '  return 0; }\n')
    inc = os.path.join(ROOT, "paper_2503_01840_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", inc, str(tmp_path / "m.cpp"), "-o", str(tmp_path / "m")], check=True)
    r = subprocess.run([str(tmp_path / "m")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_few_rows_choices_can_be_launched(tmp_path):
    (tmp_path / "m.cpp").write_text('#include <cstdio>\n#include <initializer_list>\n#include "wide_tiles.hpp"\n'
                                    'int main() { long seen[3] = {0, 0, 0};\n'
                                    '  for (int M : {1, 32, 33, 60, 64}) for (int N = 4; N <= 160000; N += 4 + N / 3) for (int K = 128; K <= 28672; K += 128)\n'
                                    '    for (int s : {0, 1}) for (int direct : {0, 1}) for (int ok : {0, 1}) for (long cap : {0l, 4l * M * N, 1l << 40}) {\n'
                                    '      const FewRows t = few_rows(M, N, K, s, direct, cap, ok);\n'
                                    '      ++seen[t.cols / 128];\n'
                                    '      const bool good = (t.cols == 64 || (M > 32 && ok && (t.cols == 128 || t.cols == 256))) && t.S >= 1 && t.S <= 16 &&\n'
                                    '        K / (t.cols == 256 ? 64 : 128) % t.S == 0 && (t.S == 1 || (!s && (long)t.S * M * N <= cap));\n'
                                    '      if (!good) { printf("%d %d %d %d %d %ld: %d %d\\n", M, N, K, s, direct, cap, t.cols, t.S); return 1; } }\n'
                                    '  return !(seen[0] && seen[1] && seen[2]); }\n')
    inc = os.path.join(ROOT, "paper_2503_01840_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", inc, str(tmp_path / "m.cpp"), "-o", str(tmp_path / "m")], check=True)
    r = subprocess.run([str(tmp_path / "m")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


# 33..64 rows, LM heads whose partial sums cost more than the fuller rounds of a split give: unsplit; features' fusion: split
def test_few_rows_splits_of_results_that_go_to_their_place(tmp_path):
    (tmp_path / "m.cpp").write_text('#include <cstdio>\n#include "wide_tiles.hpp"\n'
                                    'int main() { const int q[][4] = {{60, 65780, 4352, 0}, {33, 65780, 4352, 0}, {64, 65780, 4608, 0}, {64, 4096, 12288, 1}, {33, 5120, 15360, 1}};\n'
                                    '  for (auto& c : q) { const FewRows t = few_rows(c[0], c[1], c[2], false, true, (size_t)1 << 40, true);\n'
                                    '    if ((t.S > 1) != c[3]) { printf("%d %d %d: %d\\n", c[0], c[1], c[2], t.S); return 1; } }\n'
                                    '  return 0; }\n')
    inc = os.path.join(ROOT, "paper_2503_01840_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", inc, str(tmp_path / "m.cpp"), "-o", str(tmp_path / "m")], check=True)
    r = subprocess.run([str(tmp_path / "m")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


# fp32 (rows, weight rows, K, pairs): microseconds with the norm inside the product, as a launch of its own
MEASURED_NORM = [
    ((16, 2048, 256, 0), 3.7, 6.8), ((64, 2048, 512, 0), 12.9, 14.3), ((256, 2048, 512, 0), 43.7, 41.8), ((64, 32000, 2048, 0), 675, 600),
    ((64, 8000, 512, 0), 42.6, 40.5), ((16, 8000, 512, 0), 12.7, 14.0), ((64, 3072, 1024, 1), 21.2, 22.1), ((256, 3072, 1024, 1), 73.5, 67.6),
    ((128, 1376, 256, 1), 8.8, 9.8), ((512, 1376, 256, 1), 24.7, 20.0), ((64, 11008, 2048, 1), 136, 118), ((8, 6144, 2048, 1), 12.7, 14.4),
]


def test_fp32_norm_inside_the_product_where_it_is_the_faster_way(tmp_path):
    rows = ", ".join("{%d, %d, %d, %d, %d}" % (*q, inside < own) for q, inside, own in MEASURED_NORM)
    (tmp_path / "m.cpp").write_text('#include <cstdio>\n#include "wide_tiles.hpp"\n'
                                    'int main() { const int q[][5] = {' + rows + '};\n'
                                    '  for (auto& c : q) if (f32_norm_inside(c[0], c[1], c[2], c[3]) != c[4]) { printf("%d %d %d\\n", c[0], c[1], c[2]); return 1; }\n'
                                    '  return 0; }\n')
    inc = os.path.join(ROOT, "paper_2503_01840_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", inc, str(tmp_path / "m.cpp"), "-o", str(tmp_path / "m")], check=True)
    r = subprocess.run([str(tmp_path / "m")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


# hidden, q heads, kv heads, intermediate, vocabulary of the models of test_gpu_row_tiles.py
MODELS = {"8b": (4096, 32, 8, 14336, 128256), "wide": (3584, 28, 4, 18944, 33004), "deep": (5120, 40, 8, 13824, 20484), "mha": (4096, 32, 32, 11008, 1024),
          "flat": (256, 4, 2, 14336, 1024)}


def _products(model, M):
    """(outputs, inputs, SwiGLU, straight to its place, floats for partial sums) of q/k/v, o, gate/up, down and the LM head"""
    k, H, G, I, V = MODELS[model]
    widest = max((H + 2 * G) * 128, k)
    cap = max(1024 * widest, 4 * M * widest, 8 * M * k, 2 * 2048 * widest)
    return [((H + 2 * G) * 128, k, 0, 0, cap), (k, H * 128, 0, 0, cap), (2 * I, k, 1, 0, cap), (k, I, 0, 0, cap), (V, k, 0, 1, 0)]


# what the comments there say that they cover: (rows, cols, S, k, staggered) of the products listed
@pytest.mark.parametrize("model,M,at,want", [
    ("8b", 65, (0, 1, 2, 3, 4), [(96, 128, 4, 128, 0), (96, 128, 8, 128, 0), (96, 128, 1, 128, 1), (96, 128, 8, 128, 0), (96, 256, 1, 64, 1)]),
    ("8b", 128, (0, 1, 2, 3, 4), [(128, 128, 4, 128, 0), (128, 128, 8, 64, 0), (128, 128, 1, 128, 1), (128, 128, 8, 128, 0), (128, 256, 1, 64, 1)]),
    ("8b", 129, (0, 2, 3, 4), [(256, 128, 4, 128, 0), (256, 128, 1, 128, 1), (256, 128, 8, 128, 0), (192, 256, 1, 64, 1)]),
    ("8b", 256, (0, 2, 3, 4), [(256, 128, 4, 128, 0), (256, 128, 1, 128, 1), (256, 128, 7, 128, 1), (256, 256, 1, 64, 1)]),
    ("8b", 600, (0, 1, 2, 3), [(128, 128, 2, 64, 0), (192, 256, 4, 64, 0), (192, 256, 1, 64, 0), (192, 256, 4, 64, 0)]),
    ("wide", 65, (1, 2, 3, 4), [(96, 128, 7, 128, 0), (96, 256, 1, 64, 0), (128, 128, 8, 64, 0), (96, 256, 1, 64, 0)]),
    ("wide", 128, (1, 2, 3, 4), [(128, 128, 7, 64, 0), (128, 256, 1, 64, 0), (128, 128, 8, 64, 0), (128, 256, 1, 64, 0)]),
    ("wide", 129, (0, 2, 3, 4), [(256, 128, 4, 128, 0), (192, 256, 1, 64, 0), (256, 128, 8, 64, 0), (192, 256, 1, 64, 0)]),
    ("mha", 129, (3,), [(256, 128, 4, 64, 0)]), ("mha", 256, (3,), [(256, 128, 4, 64, 0)]),
    ("flat", 257, (2,), [(192, 256, 1, 64, 0)]), ("flat", 384, (2,), [(192, 256, 1, 64, 0)]), ("flat", 385, (2,), [(256, 256, 1, 64, 0)]),
    ("flat", 576, (2,), [(192, 256, 1, 64, 0)]), ("flat", 577, (2,), [(192, 256, 1, 64, 0)]),
])
def test_tiles_that_the_gpu_tests_cover(whole_rule, model, M, at, want):
    ps = _products(model, M)
    assert whole_rule([(M, *ps[i][:3], ps[i][4]) for i in at]) == want


# 33..64 rows: (cols, S, staggered)
@pytest.mark.parametrize("model,at,want", [("8b", (0, 2, 4), [(128, 4, 0), (128, 1, 1), (256, 1, 1)]), ("wide", (2, 4), [(256, 1, 0), (256, 1, 0)]),
                                           ("deep", (1, 3, 4), [(128, 5, 0), (128, 6, 0), (128, 1, 0)])])
@pytest.mark.parametrize("M", [33, 48, 63, 64])
def test_few_row_tiles_that_the_gpu_tests_cover(tmp_path, model, at, want, M):
    ps = [_products(model, M)[i] for i in at]
    ask = ", ".join("{%d, %d, %d, %d, %d}" % (n, k, s, d, cap or 1 << 30) for n, k, s, d, cap in ps)
    (tmp_path / "m.cpp").write_text('#include <cstdio>\n#include "wide_tiles.hpp"\nint main() { const long q[][5] = {' + ask + '};\n'
                                    '  for (auto& c : q) { const FewRows t = few_rows(' + str(M) + ', c[0], c[1], c[2], c[3], c[4], true);\n'
                                    '    printf("%d %d %d\\n", t.cols, t.S, few_rows_stagger(c[1], t.S)); } }\n')
    inc = os.path.join(ROOT, "paper_2503_01840_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", inc, str(tmp_path / "m.cpp"), "-o", str(tmp_path / "m")], check=True)
    out = subprocess.run([str(tmp_path / "m")], capture_output=True, text=True, check=True).stdout
    assert [tuple(map(int, line.split())) for line in out.splitlines()] == want


# beyond 256 rows: (rows, outputs, inputs, SwiGLU): microseconds in the best of the other tiles, in tiles of 224 or 192 weight rows
MEASURED_ROUNDS = [
    ((512, 28672, 4096, 1), 99.8, 98.3), ((1024, 28672, 4096, 1), 217, 207), ((1280, 28672, 4096, 1), 286, 244), ((2048, 28672, 4096, 1), 371, 357),
    ((300, 28672, 4096, 1), 85.4, 94.9), ((4096, 28672, 4096, 1), 702, 718), ((2048, 6144, 4096, 0), 115, 99), ((1024, 6144, 4096, 0), 69.5, 63.1),
    ((512, 6144, 4096, 0), 43.9, 47.7), ((2048, 4096, 4096, 0), 72.5, 83.0), ((512, 4096, 14336, 0), 71.5, 80.0), ((1024, 57344, 8192, 1), 761, 716),
    ((512, 22016, 4096, 1), 96, 83), ((1024, 12288, 4096, 0), 112, 101), ((2048, 18432, 2304, 1), 175, 149), ((512, 128256, 4096, 0), 529, 547),
]


@pytest.fixture(scope="module")
def launched(tmp_path_factory):
    """(M, N, K, SwiGLU, capacity) -> (rows, cols, S, k of a stage) beyond 256 rows: of the launch, and of the tile that wide_tiles picks"""
    d = tmp_path_factory.mktemp("launched")
    (d / "m.cpp").write_text('#include <cstdio>\n#include "wide_tiles.hpp"\n'
                             'int main() { int m, n, k, s; long long c; while (scanf("%d %d %d %d %lld", &m, &n, &k, &s, &c) == 5) {\n'
                             '  for (const WideTiles& t : {launch_tiles(m, n, k, s, c), wide_tiles(m, n, k, s, c)}) printf("%d %d %d %d ", t.rows, t.cols, t.S, t.k);\n'
                             '  puts(""); } }\n')
    inc = os.path.join(ROOT, "paper_2503_01840_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", inc, str(d / "m.cpp"), "-o", str(d / "m")], check=True)

    def ask(queries):
        text = "\n".join(" ".join(map(str, q)) for q in queries) + "\n"
        out = subprocess.run([str(d / "m")], input=text, capture_output=True, text=True, check=True).stdout
        return [(t[:4], t[4:]) for t in (tuple(map(int, line.split())) for line in out.splitlines())]
    return ask


def test_tiles_that_make_up_whole_rounds_where_they_are_the_faster_ones(launched):
    for (q, without, by_rounds), (t, _) in zip(MEASURED_ROUNDS, launched([q + (BIG,) for q, _, _ in MEASURED_ROUNDS])):
        assert (t[1] in (192, 224)) == (by_rounds < without), (q, t)


def test_every_launch_is_possible_and_sums_in_chains_no_longer(launched):
    qs = [(M, N, K, s, cap) for M in (257, 383, 512, 1000, 2048, 4096) for N in (256, 768, 4608, 5120, 6144, 12288, 28672)
          for K in (128, 256, 2304, 4096, 14336) for s in (0, 1) for cap in (0, 2048 * 5120, BIG)]
    seen = set()
    for (M, N, K, s, cap), (t, base) in zip(qs, launched(qs)):
        seen.add(t[:2])
        if t == base:
            continue
        assert t[0] == 256 and t[1] in (192, 224) and t[3] == 64
        assert 1 <= t[2] <= 8 and (K // 64) % t[2] == 0 and (t[2] == 1 or (not s and t[2] * M * N <= cap))
        assert K // t[2] <= K // base[2] // (2 if base[3] == 128 else 1)
    assert {(256, 192), (256, 224)} <= seen


def test_whole_rounds_that_the_gpu_tests_cover(launched):
    at = {"8b": [(2, 224, 1)], "deep": [(2, 224, 1)], "mha": [(0, 192, 2), (2, 192, 1)]}
    for name, M in [("8b", 512), ("8b", 427), ("deep", 488), ("mha", 512), ("mha", 497)]:
        for i, cols, splits in at[name]:
            p = _products(name, M)[i]
            assert launched([(M, *p[:3], p[4])])[0][0][:3] == (256, cols, splits), (name, M, i)
    # and what test_tiles_that_the_gpu_tests_cover says of more than 256 rows is what is launched there
    for name, M, rows in [("8b", 600, (0, 1, 2, 3)), ("flat", 257, (2,)), ("flat", 384, (2,)), ("flat", 385, (2,)), ("flat", 576, (2,)), ("flat", 577, (2,))]:
        for i in rows:
            p = _products(name, M)[i]
            launch, base = launched([(M, *p[:3], p[4])])[0]
            assert launch == base, (name, M, i)


# K ranges, and log2 of those dealt to different XCDs, of products that the GPU tests of test_gpu_row_tiles.py and test_gpu_stream_tiles.py run
@pytest.mark.parametrize("model,M,at,want", [("8b", 1100, (0, 1, 3), [(2, 1), (2, 1), (2, 1)]), ("8b", 600, (3,), [(4, 2)]), ("8b", 512, (3,), [(4, 2)]),
                                             ("8b", 256, (3,), [(7, 0)]), ("wide", 256, (3,), [(8, 3)])])
def test_dealt_ranges_that_the_gpu_tests_cover(tmp_path, model, M, at, want):
    ask = ", ".join("{%d, %d, %d, %d}" % (p[0], p[1], p[2], p[4]) for p in (_products(model, M)[i] for i in at))
    (tmp_path / "m.cpp").write_text('#include <cstdio>\n#include "wide_tiles.hpp"\nint main() { const long q[][4] = {' + ask + '};\n'
                                    '  for (auto& c : q) { const WideTiles t = many_tiles(' + str(M) + ', c[0], c[1], c[2], c[3]);\n'
                                    '    printf("%d %d\\n", t.S, dealt_ranges(' + str(M) + ', c[1], t.S)); } }\n')
    inc = os.path.join(ROOT, "paper_2503_01840_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", inc, str(tmp_path / "m.cpp"), "-o", str(tmp_path / "m")], check=True)
    out = subprocess.run([str(tmp_path / "m")], capture_output=True, text=True, check=True).stdout
    assert [tuple(map(int, line.split())) for line in out.splitlines()] == want


# the tiles of test_rows_rotated_by_the_product
def test_unsplit_tiles_that_the_gpu_tests_cover(launched):
    for H, G, k, M, want in [(56, 8, 512, 1280, (256, 192, 1, 64)), (56, 7, 512, 1280, (256, 192, 1, 64)), (32, 8, 4096, 1280, (256, 128, 1, 128)), (64, 16, 256, 1100, (256, 256, 1, 64)),
                             (48, 8, 1024, 1100, (192, 256, 1, 64)), (32, 4, 512, 1100, (256, 128, 1, 128))]:
        n = (H + 2 * G) * 128
        widest = max(n, k)
        cap = max(1024 * widest, 4 * M * widest, 8 * M * k, 2 * 2048 * widest)
        assert launched([(M, n, k, 0, cap)])[0][0] == want, (H, G, k, M)


# the tiles of test_prefill_rotated_by_the_product: target and draft product
def test_unsplit_tiles_of_prompts_that_the_gpu_tests_cover(launched):
    for H, G, k, T, want in [(64, 16, 256, 300, ((256, 128, 1, 128), (256, 128, 1, 128))), (64, 16, 256, 650, ((192, 256, 1, 64), (192, 256, 1, 64))),
                             (64, 16, 256, 1000, ((256, 256, 1, 64), (256, 192, 1, 64))), (56, 7, 512, 1200, ((256, 192, 1, 64), (256, 192, 1, 64)))]:
        n = (H + 2 * G) * 128
        assert [t for t, _ in launched([(T, n, k, 0, 2 * 2048 * n), (T - 1, n, 2 * k, 0, 2 * 2048 * n)])] == list(want), (H, G, k, T)
