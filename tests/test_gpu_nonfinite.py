"""What a row may not see must not reach it, whatever its value: an infinity or NaN at one position leaves the results of every
earlier position as they are (in a matrix product a weight of zero does not: 0 x Inf is NaN)."""
import numpy as np
import pytest
import torch

import eagle3_synth as S

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
INF, NAN = float("inf"), float("nan")


def _reference(q, k, v):
    """fp64, every query over exactly the keys it sees."""
    T, H, d = q.shape
    s, G = k.shape[0] - 1, k.shape[2]
    q, k, v = q.double(), k.double(), v.double()
    out = torch.empty(T, H, d, dtype=torch.float64)
    for h in range(H):
        g = h * G // H
        for i in range(T):
            kk = torch.cat([k[0, :i + 1, g], k[1:, i, g]])
            vv = torch.cat([v[0, :i + 1, g], v[1:, i, g]])
            w = ((kk * q[i, h]).sum(1) / d ** 0.5).softmax(0)
            out[i, h] = (w[:, None] * vv).sum(0)
    return out.numpy()


# every number of query heads per workgroup (4, 2, 1); the bad position at the edges of 32-key blocks and of a workgroup's queries
@pytest.mark.parametrize("H,Hkv", [(4, 1), (2, 1), (3, 1), (2, 2)])
@pytest.mark.parametrize("T,at", [(1, 0), (40, 39), (130, 31), (130, 64), (200, 127), (200, 128), (200, 199)])
@pytest.mark.parametrize("where,bad", [("v", INF), ("v", NAN), ("k", NAN), ("own v", -INF)])
def test_ttt_attention_keeps_a_bad_position_to_the_rows_that_see_it(H, Hkv, T, at, where, bad):
    import paper_2503_01840_amd as E
    s = 2
    q, k, v = (S.normal(S.SEED + T, i, dims, dtype=torch.bfloat16)
               for i, dims in ((1, (T, H, 128)), (2, (s + 1, T, Hkv, 128)), (3, (s + 1, T, Hkv, 128))))
    t = {"k": k[0], "v": v[0], "own v": v[1]}[where]
    t[at, Hkv - 1, 3:70] = bad
    got = E.eagle3_ttt_attention(q.to(DEV), k.to(DEV), v.to(DEV)).cpu().numpy()
    ref = _reference(q, k, v)
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    ok = np.isfinite(ref)
    assert np.array_equal(np.sign(got[~ok & ~np.isnan(ref)]), np.sign(ref[~ok & ~np.isnan(ref)]))
    # the bound of the tile-edge tests: weights carried with 16 bits, |values| < 5
    assert np.max(np.abs(got[ok] - ref[ok]), initial=0.0) < 2 * 5 * (2e-6 + 2.0 ** -16)


# everything NaN (a broken model): the same results, in time that does not grow with the number of keys
@pytest.mark.parametrize("where", ["k", "v"])
def test_ttt_attention_of_nothing_but_nan(where):
    import paper_2503_01840_amd as E
    T, H, Hkv = 3000, 8, 2
    q, k, v = (torch.randn(*dims, dtype=torch.bfloat16, device=DEV) for dims in ((T, H, 128), (2, T, Hkv, 128), (2, T, Hkv, 128)))
    {"k": k, "v": v}[where].fill_(NAN)
    assert bool(torch.isnan(E.eagle3_ttt_attention(q, k, v)).all())


def _prefill(E, shape, W, tokens, parts):
    ctx = E.Eagle3Context(shape, max_batch=1, max_nodes=8, max_depth=2, max_topk=2, max_new=4, device=DEV)
    ctx.set_weights(W["target"], W["draft"])
    T = sum(parts)
    i32 = lambda v: torch.tensor(v, dtype=torch.int32, device=DEV)
    z = lambda: torch.zeros(T, shape.n_kv_heads, shape.head_dim, dtype=ctx.storage_dtype, device=DEV)
    ks, vs = [z() for _ in range(shape.n_layers)], [z() for _ in range(shape.n_layers)]
    kv, dkv = E.KVCache(ks, vs, i32([0, T]), i32([0]), 0), E.KVCache([z()], [z()], i32([0, T]), i32([0]), 0)
    at = 0
    for n in parts:
        E.eagle3_prefill(ctx, tokens[at:at + n].contiguous(), kv, dkv)
        at += n
    torch.cuda.synchronize()
    return torch.stack(ks + vs).float().cpu(), torch.stack([dkv.k_layers[0], dkv.v_layers[0]]).float().cpu()


# a token whose embedding row is NaN in the middle of a prompt; every number of query heads per workgroup
@pytest.mark.parametrize("H,Hkv", [(4, 1), (2, 1), (3, 1), (2, 2)])
@pytest.mark.parametrize("at", [31, 63, 127, 150])
def test_prefill_keeps_a_bad_token_to_the_rows_that_see_it(H, Hkv, at):
    _bad_token(_small(n_heads=H, n_kv_heads=Hkv), [200], at)


# the same through the tree kernels: a chunk that the split kernel takes (few rows behind many keys), and the fp32 model
@pytest.mark.parametrize("parts,at", [([700, 100], 730), ([700, 100], 763), ([700, 100], 799), ([1000, 20], 1001)])
def test_prefill_behind_a_long_context_keeps_a_bad_token_to_the_rows_that_see_it(parts, at):
    _bad_token(_small(), parts, at)


# (heads of 64 and 128 and heads of other sizes have a kernel each)
@pytest.mark.parametrize("d", [64, 128, 32, 72])
@pytest.mark.parametrize("parts,at", [([130], 60), ([130], 100), ([40, 90], 100)])
def test_prefill_fp32_keeps_a_bad_token_to_the_rows_that_see_it(parts, at, d):
    _bad_token(S.get_shape("c1").with_(head_dim=d), parts, at)


# an infinity and a NaN among the values of tree slots that other rows do not see, in every kernel of the fp32 attention
@pytest.mark.parametrize("d", [64, 128, 32, 72])
@pytest.mark.parametrize("bad", [INF, NAN])
def test_verification_fp32_keeps_bad_values_to_the_nodes_that_see_them(d, bad):
    import paper_2503_01840_amd as E
    import pipeline as PL
    shape = S.get_shape("c1").with_(head_dim=d, n_layers=1, taps=(0, 0, 0))
    N, P, at = 30, 40, 3
    parent = S.random_tree(S.SEED, 3, N, 6, 3)[0]
    below = np.zeros(N, bool)
    for i in range(N):
        below[i] = i == at or (i > 0 and below[parent[i]])
    W = PL.device_weights(shape, device=DEV)
    ctx = E.Eagle3Context(shape, max_batch=1, max_nodes=N, max_depth=2, max_topk=2, max_new=4, device=DEV)
    ctx.set_weights(W["target"], W["draft"])
    i32 = lambda v: torch.tensor(np.asarray(v), dtype=torch.int32, device=DEV)
    tok = S.uniform_ints(S.SEED, 5, (1, N), 0, shape.vocab).to(torch.int32).to(DEV)

    def stream(x_in):
        k, v = (S.normal(S.SEED, i, (P + N, shape.n_kv_heads, d)).float().to(DEV) for i in (1, 2))
        return E.eagle3_tree_verify_layers(ctx, tok, i32(parent)[None], E.KVCache([k], [v], i32([0, P + N]), i32([P]), P), x_in, 0, 1)[0][0].cpu()

    x_in = S.normal(S.SEED, 9, (1, N, shape.hidden)).float().to(DEV)
    clean = stream(x_in)
    x_in[0, at, 5] = bad                                          # its row of keys and values is NaN throughout
    got = stream(x_in)
    assert bool(torch.isnan(got[below]).any(1).all()) and not below.all()
    assert bool(torch.isfinite(got[~below]).all()) and float((got[~below] - clean[~below]).abs().max()) < 1e-4


# a bad node in a tree: nodes that do not descend from it keep their logits
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("P", [0, 5, 600])
def test_verification_keeps_a_bad_node_to_its_descendants(dtype, P):
    import paper_2503_01840_amd as E
    import pipeline as PL
    shape = S.get_shape("c1") if dtype == "fp32" else _small()
    N = 30
    parent = S.random_tree(S.SEED, 3, N, 6, 3)[0]
    bad = 2
    below = np.zeros(N, bool)
    for i in range(N):
        below[i] = i == bad or (i > 0 and below[parent[i]])
    W = PL.device_weights(shape, device=DEV)
    ctx = E.Eagle3Context(shape, max_batch=1, max_nodes=N, max_depth=2, max_topk=2, max_new=4, device=DEV)
    i32 = lambda v: torch.tensor(np.asarray(v), dtype=torch.int32, device=DEV)
    tok = S.uniform_ints(S.SEED, 5, (1, N), 0, shape.vocab - 1).to(torch.int32).to(DEV)

    def logits():
        ctx.set_weights(W["target"], W["draft"])
        kv = [[S.normal(S.SEED + l, i, (P + N, shape.n_kv_heads, shape.head_dim)).to(ctx.storage_dtype).to(DEV)
               for l in range(shape.n_layers)] for i in (1, 2)]
        return E.eagle3_tree_verify(ctx, tok, i32(parent)[None], E.KVCache(*kv, i32([0, P + N]), i32([P]), P))[0][0].cpu()

    clean = logits()
    W["target"]["embed"] = W["target"]["embed"].clone()
    W["target"]["embed"][shape.vocab - 1] = NAN
    tok[0, bad] = shape.vocab - 1
    got = logits()
    assert bool(torch.isnan(got[below]).all()) and not below.all()
    assert bool(torch.isfinite(got[~below]).all())
    assert float((got[~below] - clean[~below]).abs().max()) < (1e-4 if dtype == "fp32" else 2e-2)


def _small(**over):
    from test_gpu_edges import SMALL
    return SMALL.with_(**over)


def _bad_token(shape, parts, at):
    import paper_2503_01840_amd as E
    import pipeline as PL
    W = PL.device_weights(shape, device=DEV)
    T = sum(parts)
    tokens = S.uniform_ints(S.SEED + T, S.TensorIds.PREFIX_TOK, (T,), 0, shape.vocab - 1).to(torch.int32).to(DEV)
    clean, clean_d = _prefill(E, shape, W, tokens, parts)
    W["target"]["embed"] = W["target"]["embed"].clone()
    W["target"]["embed"][shape.vocab - 1] = NAN
    tokens[at] = shape.vocab - 1
    got, got_d = _prefill(E, shape, W, tokens, parts)
    # rows in the same kernels as before, their sums in another order where a row was formed again: the prefill tests' bounds
    tol = 1e-4 if shape.dtype == "fp32" else 4e-2
    assert bool(torch.isnan(got[:, at]).all())
    # (the draft row of position i holds token i + 1; the last position of a call gets none)
    n_draft = at - len(parts)
    for a, b in ((clean[:, :at], got[:, :at]), (clean_d[:, :n_draft], got_d[:, :n_draft])):
        assert bool(torch.isfinite(b).all()) and float((a - b).abs().max()) < tol
