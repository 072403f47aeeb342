"""The causal attention kernel at the edges of its tiles (32-key blocks, 128-key tiles, 128 / heads queries per workgroup)."""
import numpy as np
import pytest
import torch

import eagle3_synth as S
from oracle import eagle3_oracle as O

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# (H, Hkv): 4 heads of a group per workgroup, two such workgroups, 2 heads, 1 head; s: no simulated step, one, a whole batch
# of staged steps (4, 2 or 1 of them), one more than that
@pytest.mark.parametrize("T", [1, 32, 33, 127, 128, 129, 161, 290])
@pytest.mark.parametrize("H,Hkv,s", [(4, 1, 0), (8, 1, 5), (8, 2, 4), (4, 2, 3), (2, 1, 2), (3, 1, 2), (2, 2, 1)])
@pytest.mark.parametrize("spread", [1.0, 4.0])
def test_ttt_attention_at_tile_edges(T, H, Hkv, s, spread):
    import paper_2503_01840_amd as E
    q = (spread * S.normal(S.SEED + T, 1, (T, H, 128), dtype=torch.float32)).to(torch.bfloat16)
    k = S.normal(S.SEED + T, 2, (s + 1, T, Hkv, 128), dtype=torch.bfloat16)
    v = S.normal(S.SEED + T, 3, (s + 1, T, Hkv, 128), dtype=torch.bfloat16)
    got = E.eagle3_ttt_attention(q.to(DEV), k.to(DEV), v.to(DEV)).cpu().numpy()
    ref = O.ttt_attention(O.as_f64(q), O.as_f64(k), O.as_f64(v), "mask")
    # |values| < 5.  A score is a sum of 128 products whose absolute values add up to ~ 82 spread: fp32 leaves it ~ 1e-5 spread
    # off before the 1 / sqrt(128), the weights are carried with 16 bits: 5 * (2e-6 spread + 2^-16) at the very most, doubled
    assert np.max(np.abs(got - ref)) < 2 * 5 * (2e-6 * spread + 2.0 ** -16), (T, H, Hkv, s)


# every number of 32-key blocks in the last tile (a wavefront takes the first and third or the second and fourth), the own rows
# behind a tile whose second pair is left out, one and several tiles
@pytest.mark.parametrize("T", [64, 65, 96, 97, 160, 192, 193, 224, 225, 256])
@pytest.mark.parametrize("H,Hkv,s", [(8, 2, 5), (3, 3, 2), (2, 1, 0)])
def test_ttt_attention_with_partly_filled_last_tiles(T, H, Hkv, s):
    test_ttt_attention_at_tile_edges(T, H, Hkv, s, 3.0)


# sizes around the lines between 64-row and 128-row workgroups (256 and 512 of the smaller ones)
@pytest.mark.parametrize("T,H,Hkv,s", [(2048, 8, 8, 1), (2049, 8, 8, 0), (1025, 16, 16, 3), (513, 32, 8, 2), (1030, 32, 8, 0), (300, 64, 8, 2)])
def test_ttt_attention_around_the_workgroup_sizes(T, H, Hkv, s):
    import paper_2503_01840_amd as E
    q = S.normal(S.SEED + T, 1, (T, H, 128), dtype=torch.bfloat16)
    k = S.normal(S.SEED + T, 2, (s + 1, T, Hkv, 128), dtype=torch.bfloat16)
    v = S.normal(S.SEED + T, 3, (s + 1, T, Hkv, 128), dtype=torch.bfloat16)
    got = E.eagle3_ttt_attention(q.to(DEV), k.to(DEV), v.to(DEV)).cpu().numpy()
    q64, K, V = O.as_f64(q), O.as_f64(k).reshape((s + 1) * T, Hkv, 128), O.as_f64(v).reshape((s + 1) * T, Hkv, 128)
    sets = O.ttt_visible_sets(T, s)
    rows = sorted({0, 31, 32, 63, 64, 127, 128, T // 2, T - 65, T - 64, T - 2, T - 1})
    for i in rows:
        ref = O.attention_explicit_sets(q64[i:i + 1], K, V, [sets[i]])
        assert np.max(np.abs(got[i] - ref[0])) < 2 * 5 * (2e-6 + 2.0 ** -16), i          # the tile-edge bound
    assert np.isfinite(got).all()


# queries at any address; every number of query heads per workgroup
@pytest.mark.parametrize("H,Hkv", [(4, 1), (4, 2), (3, 1)])
@pytest.mark.parametrize("shift", [1, 2, 4, 8])
@pytest.mark.parametrize("T", [33, 200])
def test_ttt_attention_with_queries_at_any_address(H, Hkv, shift, T):
    import paper_2503_01840_amd as E
    q = S.normal(S.SEED + T, 1, (T, H, 128), dtype=torch.bfloat16)
    k = S.normal(S.SEED + T, 2, (2, T, Hkv, 128), dtype=torch.bfloat16)
    v = S.normal(S.SEED + T, 3, (2, T, Hkv, 128), dtype=torch.bfloat16)
    flat = torch.zeros(q.numel() + 8, dtype=torch.bfloat16, device=DEV)
    moved = flat[shift:shift + q.numel()].view(q.shape)
    moved.copy_(q)
    assert torch.equal(E.eagle3_ttt_attention(moved, k.to(DEV), v.to(DEV)), E.eagle3_ttt_attention(q.to(DEV), k.to(DEV), v.to(DEV)))


# a prompt in two calls: P rows first, then n rows behind them, against the same prompt in one call.  n rows with P behind them
# take the causal kernel (few tiles of keys) or the split one (long context, few rows)
@pytest.mark.parametrize("P,n", [(1, 63), (64, 64), (77, 130), (127, 1), (200, 312), (700, 20), (1000, 500)])
def test_prefill_continues_a_cached_prefix(P, n):
    from test_gpu_edges import SMALL
    _prompt_in_two_calls(SMALL, P, n)


# just more than 128 workgroups of the causal kernel behind a context of twelve tiles; fewer, but enough for its length
@pytest.mark.parametrize("P,n", [(1500, 530), (400, 230)])
def test_prefill_of_many_workgroups_behind_a_prefix(P, n):
    from test_gpu_edges import SMALL
    _prompt_in_two_calls(SMALL.with_(name="h32", n_heads=32, n_kv_heads=8), P, n)


def _prompt_in_two_calls(shape, P, n):
    import pipeline as PL
    from test_gpu_edges import _E
    E = _E()
    ctx = E.Eagle3Context(shape, max_batch=1, max_nodes=8, max_depth=2, max_topk=2, max_new=4, device=DEV)
    W = PL.device_weights(shape, device=DEV)
    ctx.set_weights(W["target"], W["draft"])
    T = P + n
    i32 = lambda v: torch.tensor(v, dtype=torch.int32, device=DEV)
    tokens = S.uniform_ints(S.SEED + T, S.TensorIds.PREFIX_TOK, (T,), 0, shape.vocab).to(torch.int32).to(DEV)

    def prefill(parts):
        z = lambda: torch.zeros(T, shape.n_kv_heads, shape.head_dim, dtype=ctx.storage_dtype, device=DEV)
        ks, vs = [z() for _ in range(shape.n_layers)], [z() for _ in range(shape.n_layers)]
        kv = E.KVCache(ks, vs, i32([0, T]), i32([0]), 0)
        dkv = E.KVCache([z()], [z()], i32([0, T]), i32([0]), 0)
        at = 0
        for m in parts:
            g, logits = E.eagle3_prefill(ctx, tokens[at:at + m].contiguous(), kv, dkv)
            at += m
        torch.cuda.synchronize()
        return torch.stack(ks + vs).float(), logits.float(), g.float()

    for a, b in zip(prefill([T]), prefill([P, n])):
        assert bool(torch.isfinite(b).all())
        # same sums in another order, rounded to bf16 between the two layers: the two-layer bounds of the prefill tests
        assert float((a - b).abs().max()) < 4e-2, (P, n)
