"""Prefill in chunks of many rows: prompt lengths at the edges of the 64-row attention blocks and of the chunks (256 rows in
fp32, 2048 in bf16), every cache row, the fused feature and the logits of the last position against the oracle's prefill."""
import numpy as np
import pytest
import torch

import eagle3_synth as S
from oracle import eagle3_oracle as O
import pipeline as PL
from test_gpu_edges import SMALL, _E

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype,T", [("fp32", 64), ("fp32", 129), ("fp32", 256), ("fp32", 257),
                                     ("bf16", 65), ("bf16", 192), ("bf16", 385), ("bf16", 2049)])
def test_prefill_at_block_and_chunk_edges(dtype, T):
    _check(S.get_shape("c1") if dtype == "fp32" else SMALL, dtype, T)


# three and more chunks: of 256 rows (fp32), and in workspaces of which 0, 2, 10 or 50 % of the part that prefill needs is there
@pytest.mark.parametrize("dtype,T,part", [("fp32", 513, 1.0), ("fp32", 700, 1.0), ("fp32", 300, 0.0), ("fp32", 300, 0.5), ("bf16", 300, 0.0),
                                          ("bf16", 700, 0.02), ("bf16", 700, 0.1), ("bf16", 2500, 0.5), ("bf16", 200, 0.0)])
def test_prefill_in_several_chunks(dtype, T, part):
    _check(S.get_shape("c1") if dtype == "fp32" else SMALL, dtype, T, part)


# every grouping of query heads in a workgroup of the causal kernel (four of a group, two such workgroups per KV head, two, one), with
# the sequence behind others in a larger pool
@pytest.mark.parametrize("H,Hkv", [(4, 1), (8, 1), (16, 2), (2, 1), (3, 1), (2, 2)])
@pytest.mark.parametrize("T,base", [(129, 0), (300, 37)])
def test_prefill_over_head_layouts_and_pool_offsets(H, Hkv, T, base):
    _check(SMALL.with_(n_heads=H, n_kv_heads=Hkv), "bf16", T, base=base)


# no feature behind the last layer, so that only the last position goes through all of it: one position, the edges of the 64-row
# blocks, a second chunk of one position, several chunks
@pytest.mark.parametrize("dtype,T,part", [("fp32", 2, 1.0), ("fp32", 65, 1.0), ("fp32", 257, 1.0), ("fp32", 300, 0.0), ("bf16", 2, 1.0),
                                          ("bf16", 64, 1.0), ("bf16", 65, 1.0), ("bf16", 577, 1.0), ("bf16", 2049, 1.0), ("bf16", 300, 0.0)])
def test_prefill_without_a_feature_of_the_last_layer(dtype, T, part):
    shape = S.get_shape("c1") if dtype == "fp32" else SMALL.with_(n_layers=3)
    _check(shape.with_(taps=(0, 0, shape.n_layers - 2)), dtype, T, part)


# hidden 512 and 768: the fusion of the features in three and four ranges of K, summed by a launch of its own; 64 rows: the few-row product
@pytest.mark.parametrize("hidden,T", [(512, 64), (512, 65), (512, 130), (512, 300), (768, 77), (768, 200), (768, 513)])
def test_prefill_with_a_split_fusion(hidden, T):
    _check(SMALL.with_(name=f"h{hidden}", hidden=hidden), "bf16", T)


# queries, keys and values rotated and put into the cache by the product (above 256 rows, unsplit): each tile that does so, row blocks and weight
# rows that end within one.  w_q times 8, so that attention depends on its queries: without the last query head of layer 0 (planted in the oracle)
# keys and values of layer 1 are 0.22 off and more.
ROTATED = [(64, 16, 256, 300), (64, 16, 256, 650), (64, 16, 256, 1000), (56, 7, 512, 1200)]


@pytest.mark.parametrize("H,Hkv,hidden,T", ROTATED)
def test_prefill_rotated_by_the_product(H, Hkv, hidden, T):
    _check(SMALL.with_(name=f"r{H}x{hidden}", hidden=hidden, n_heads=H, n_kv_heads=Hkv), "bf16", T, q_scale=8.0)


def _check(shape, dtype, T, part=1.0, base=0, q_scale=1.0):
    E = _E()
    rounding = "none" if dtype == "fp32" else "bf16"
    # fp32: the exact path's 1e-4; bf16: the 2-layer bounds of the two-chunk test (one bf16 ulp of a rotated key at |k| < 8
    # is 2^-5, of everything else below 2e-2)
    tol_k, tol = (1e-4, 1e-4) if dtype == "fp32" else (4e-2, 2e-2)
    model = PL.OracleModel(shape)
    prompt = S.uniform_ints(S.SEED + T, S.TensorIds.PREFIX_TOK, (T,), 0, shape.vocab).numpy()
    pre = O.prefill(shape, lambda l: dict(model.layer(l), wq=model.layer(l)["wq"] * q_scale), model.globals(), prompt, rounding=rounding)
    dw, emb = model.draft(), model.globals()["embed"]
    g_all = O.fuse_features(dw["w_fc"], pre["taps"][0], pre["taps"][1], pre["taps"][2], rounding=rounding)
    Kd = np.zeros((T - 1, shape.n_kv_heads, shape.head_dim)); Vd = np.zeros_like(Kd)
    O.draft_forward(shape, dw, emb, g_all[:T - 1], prompt[1:], np.arange(T - 1), Kd, Vd, 0, 0,
                    np.tril(np.ones((T - 1, T - 1), dtype=bool)), O._rounder(rounding))
    ctx = E.Eagle3Context(shape, max_batch=1, max_nodes=8, max_depth=2, max_topk=2, max_new=4, device=DEV)
    left = PL.shrink_workspace(ctx, part) if part < 1.0 else None
    W = PL.device_weights(shape, device=DEV)
    for w in W["target"]["layers"]:
        w["wq"] *= q_scale
    ctx.set_weights(W["target"], W["draft"])
    i32 = lambda v: torch.tensor(v, dtype=torch.int32, device=DEV)
    z = lambda n: torch.full((n, shape.n_kv_heads, shape.head_dim), 7.0, dtype=ctx.storage_dtype, device=DEV)
    ks, vs = [z(base + T + 3) for _ in range(shape.n_layers)], [z(base + T + 3) for _ in range(shape.n_layers)]
    kv = E.KVCache(ks, vs, i32([base, base + T]), i32([0]), 0)
    dkv = E.KVCache([z(base + T + 3)], [z(base + T + 3)], i32([base, base + T - 1]), i32([0]), 0)
    g_last, logits = E.eagle3_prefill(ctx, i32(prompt), kv, dkv)
    torch.cuda.synchronize()
    for t, n in [(t, T) for t in ks + vs] + [(dkv.k_layers[0], T - 1), (dkv.v_layers[0], T - 1)]:
        assert bool((t[:base] == 7.0).all()) and bool((t[base + n:] == 7.0).all()), "rows beside the prompt's were written"
    f = lambda t: t[base:].float().cpu().numpy() if t.dim() == 3 else t.float().cpu().numpy()
    assert int(kv.prefix_len[0]) == T and int(dkv.prefix_len[0]) == T - 1
    for l in range(shape.n_layers):
        assert np.max(np.abs(f(ks[l])[:T] - pre["k_new"][l])) < tol_k, l
        assert np.max(np.abs(f(vs[l])[:T] - pre["v_new"][l])) < tol, l
    assert np.max(np.abs(f(logits) - pre["logits"][-1])) < tol
    assert np.max(np.abs(f(g_last) - g_all[-1])) < tol
    assert np.max(np.abs(f(dkv.k_layers[0])[:T - 1] - Kd)) < tol_k
    assert np.max(np.abs(f(dkv.v_layers[0])[:T - 1] - Vd)) < tol
    if left is not None:
        assert bool((PL.beyond_workspace(ctx, left) == 171).all()), "bytes past the workspace were written"
