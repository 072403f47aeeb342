"""The products of more than 32 rows at the edges of their tiles: the same rows in few and in many, and prompts against the oracle.  Which
tile each of them takes is pinned in test_wide_tiles.py."""
import numpy as np
import pytest
import torch

import eagle3_synth as S
from test_gpu_prefill import test_prefill_at_block_and_chunk_edges as _prefill_against_the_oracle
from test_gpu_shapes import TOL, _E, _rms

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# the small model in 128 x 128 tiles just above the 256-row line, one row over a 64-row piece, over a tile, a full last tile
@pytest.mark.parametrize("T", [257, 384, 386, 576, 577])
def test_prefill_at_192_row_edges(T):
    _prefill_against_the_oracle("bf16", T)


# one layer of the 8B shape: 577..640 rows (o and down in split, gate/up in unsplit 192-row tiles, q/k/v in 128 x 128 tiles side by side) against the same
# sequences ten (128 x 128 tiles, the last few rows the few-row kernel) and 25 (256 x 128 tiles) at a time
@pytest.mark.parametrize("B,N", [(58, 10), (60, 10), (64, 10)])
@pytest.mark.parametrize("group", [10, 25])
def test_rows_do_not_depend_on_the_batch(B, N, group):
    _rows_alone_and_together(S.get_shape("c3"), B, N, group)


# a gate/up of many weight rows in 192-row tiles at 257, 384, 576 and 577 rows (256-row ones at 385): the edges of a tile against at most 64 rows
# at a time
@pytest.mark.parametrize("B,N,group", [(257, 1, 64), (64, 6, 10), (77, 5, 12), (64, 9, 7), (577, 1, 50)])
def test_rows_at_192_row_edges(B, N, group):
    _rows_alone_and_together(S.get_shape("c3").with_(name="flat", hidden=256, n_heads=4, n_kv_heads=2, vocab=1024), B, N, group, logits=True)


# 65..256 rows, logits included, against at most 64 rows at a time: the first and last row count of 128 x 128 (split, and gate/up) and of 256 x 128 tiles and
# one between.  8B width: q/k/v and down in ranges and gate/up staggered with 128-k weight stages, o in ranges of 64-k stages from 97 to 128 rows.
# "wide" (in FEW): q/k/v and down in step.  Up to 96 rows, and where 256 weight rows are taken (the LM heads, gate/up of "wide"): test_gpu_stream_tiles.py.
@pytest.mark.parametrize("name", ["8b", "wide"])
@pytest.mark.parametrize("B,N,group", [(65, 1, 64), (43, 3, 21), (128, 1, 64), (129, 1, 64), (64, 3, 20), (64, 4, 16)])
def test_rows_in_wide_weight_stages(name, B, N, group):
    _rows_alone_and_together(FEW[name], B, N, group, logits=True)


# 64-k weight stages in split products of 129..256 rows: down in four ranges of 2752; a LM head of fewer rows than inputs, split and summed
@pytest.mark.parametrize("B,N,group", [(129, 1, 64), (64, 3, 20), (64, 4, 16)])
def test_rows_in_ranges_that_wide_weight_stages_do_not_divide(B, N, group):
    _rows_alone_and_together(S.get_shape("c3").with_(name="mha", n_kv_heads=32, intermediate=11008, vocab=1024), B, N, group, logits=True)


# 33..64 rows, logits included, against at most 32 rows at a time (the few-row kernel).  8B width: q/k/v in 64 x 128 tiles in step,
# gate/up staggered, LM head 64 x 256 staggered.  "wide": gate/up and a LM head that ends within a tile in 64 x 256 tiles in step.
# "deep": o in five ranges, down in six, a LM head of a few rows more than whole 64 x 128 tiles.
FEW = {"8b": S.get_shape("c3"),
       "wide": S.get_shape("c3").with_(name="wide", hidden=3584, n_heads=28, n_kv_heads=4, intermediate=18944, vocab=33004),
       "deep": S.get_shape("c3").with_(name="deep", hidden=5120, n_heads=40, n_kv_heads=8, intermediate=13824, vocab=20484)}


# LM heads that do not end at a multiple of four, so that the rows of logits start anywhere: unsplit and in ranges, ending within a tile
@pytest.mark.parametrize("hidden,heads,vocab", [(1024, 8, 30001), (3584, 28, 33002), (2048, 16, 8197), (2048, 16, 131)])
@pytest.mark.parametrize("B", [33, 64])
def test_rows_of_an_odd_vocabulary(hidden, heads, vocab, B):
    _rows_alone_and_together(S.get_shape("c3").with_(name=f"odd{hidden}", hidden=hidden, n_heads=heads, n_kv_heads=4, intermediate=1024, vocab=vocab,
                                                     draft_vocab=64), B, 1, 32, logits=True)


@pytest.mark.parametrize("name", list(FEW))
@pytest.mark.parametrize("B,N,group", [(33, 1, 32), (12, 4, 8), (63, 1, 32), (64, 1, 32), (1, 64, 1)])
def test_rows_of_64_row_tiles(name, B, N, group):
    _rows_alone_and_together(FEW[name], B, N, group, logits=True)


# 256 x 224 and 256 x 192 tiles against at most 64 rows at a time.  8B width: gate/up in whole tiles of 224; "deep": a last tile of 96 weight rows; "mha": gate/up
# in tiles of 192, the last one of 128 rows, q/k/v in two ranges in tiles of 192; row blocks that end full and anywhere.
ROUNDS = [("8b", 64, 8, 8), ("8b", 61, 7, 9), ("deep", 61, 8, 8), ("mha", 64, 8, 8), ("mha", 71, 7, 9)]


@pytest.mark.parametrize("name,B,N,group", ROUNDS)
def test_rows_in_tiles_that_make_up_whole_rounds(name, B, N, group):
    mha = S.get_shape("c3").with_(name="mha", n_kv_heads=32, intermediate=11008, vocab=1024)
    _rows_alone_and_together(mha if name == "mha" else FEW[name].with_(vocab=1024), B, N, group, logits=True)


# 8B width, 1100 rows: q/k/v, o and down in two K ranges, each the work of four XCDs (four and eight ranges, of two and of one: 600 and 65..256 rows above)
@pytest.mark.parametrize("B,N,group", [(55, 20, 3)])
def test_rows_in_two_ranges_dealt_to_xcds(B, N, group):
    _rows_alone_and_together(FEW["8b"].with_(vocab=1024), B, N, group, logits=True)


# q/k/v rotated and put into the cache by the product, where it is not split: each tile that does so, row blocks and weight rows that end within
# one ("ragged"), against at most 64 rows at a time.  (q heads, KV heads, hidden, sequences, rows of each)
ROTATED = {"192": (56, 8, 512, 64, 20), "192-ragged": (56, 7, 512, 64, 20), "8b": (32, 8, 4096, 64, 20), "256x256": (64, 16, 256, 55, 20), "192x256": (48, 8, 1024, 55, 20),
           "256x128": (32, 4, 512, 55, 20)}


@pytest.mark.parametrize("name", list(ROTATED))
def test_rows_rotated_by_the_product(name):
    H, G, hidden, B, N = ROTATED[name]
    # up to 1024 columns a residual below the attention's share of the layer's output: without the last query head (planted in the oracle) that output is
    # 0.05 to 0.14 off, where bf16 rounding makes 0.004 and the bound is 0.02; at 4096 columns it is 1.2 off behind a residual of 8, bound 0.16
    _rows_alone_and_together(S.get_shape("c3").with_(name=f"r{name}", hidden=hidden, n_heads=H, n_kv_heads=G, intermediate=1024, vocab=1024), B, N, 64 // N,
                             scale=0.25 if hidden <= 1024 else 8.0)


def _rows_alone_and_together(full, B, N, group, logits=False, scale=8.0):
    """All B sequences of N rows at once against `group` of them at a time; one sequence: against its first 32 rows.  Layer output, the cache with
    what must stay as it was, logits."""
    E = _E()
    shape = full.with_(n_layers=1, taps=(0, 0, 0))
    W = {k: v.to(DEV) for k, v in S.layer_weights(full, 3).items()}
    tg = {k: v.to(DEV) for k, v in S.target_globals(full).items()}
    ctx = E.Eagle3Context(shape, max_batch=B, max_nodes=N, max_depth=2, max_topk=2, max_new=1 if full.vocab % 4 else 4, device=DEV)
    ctx.set_weights({"layers": [W], **tg}, None)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(B)
    i32 = lambda v: torch.as_tensor(np.asarray(v), dtype=torch.int32, device=DEV)
    x_in = scale * torch.randn(B, N, full.hidden, device=DEV, generator=gen)
    parent = i32(np.tile(np.arange(-1, N - 1), (B, 1)))
    tok = torch.zeros(B, N, dtype=torch.int32, device=DEV)
    P = 40
    k0 = torch.randn(B * (P + N), full.n_kv_heads, full.head_dim, device=DEV, generator=gen).bfloat16()
    v0 = torch.randn(B * (P + N), full.n_kv_heads, full.head_dim, device=DEV, generator=gen).bfloat16()

    def run(b0, b1, n_rows=N):
        n, at = b1 - b0, slice(b0 * (P + N), (b1 - 1) * (P + N) + P + n_rows)
        k, v = k0[at].clone(), v0[at].clone()
        kv = E.KVCache([k], [v], i32(np.append(np.arange(n) * (P + N), k.shape[0])), i32([P] * n), P)
        x_out, lg = E.eagle3_tree_verify_layers(ctx, tok[b0:b1, :n_rows].contiguous(), parent[b0:b1, :n_rows].contiguous(), kv,
                                               x_in[b0:b1, :n_rows].contiguous(), 0, 1, want_logits=True)
        torch.cuda.synchronize()
        for t, t0 in ((k, k0[at]), (v, v0[at])):
            assert all(torch.equal(t[b * (P + N):][:P], t0[b * (P + N):][:P]) for b in range(n)), "rows beside the new ones were written"
        return x_out.cpu().numpy(), k.float().cpu().numpy(), v.float().cpu().numpy(), lg.float().cpu().numpy() if logits else None

    x, k, v, lg = run(0, B)
    rows = N if B > 1 else 32
    for b0 in range(0, B, group):
        b1 = min(B, b0 + group)
        xr, kr, vr, lr = run(b0, b1, rows)
        assert np.max(np.abs(x[b0:b1, :rows] - xr)) < TOL * max(1.0, _rms(xr))
        at = slice(b0 * (P + N), b0 * (P + N) + len(kr))
        assert np.max(np.abs(k[at] - kr)) < 4e-2
        # sums in another order may round to the bf16 neighbour: 2^-5 below 8, twice that above
        assert np.max(np.abs(v[at] - vr) / np.maximum(1.0, np.abs(vr) / 8.0)) < 4e-2
        if logits:
            assert np.max(np.abs(lg[b0:b1, :rows] - lr)) < TOL * max(1.0, _rms(lr))
