"""The fp32 kernels where their loads and reductions change form: row lengths that are not a multiple of four, groups of 8 rows
with a remainder, head sizes around 128 and 256, key counts around the groups a value sum is dealt out to."""
import numpy as np
import pytest
import torch

import eagle3_synth as S
import pipeline as PL
from oracle import eagle3_oracle as O

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("T,d,s", [(1, 2, 0), (3, 64, 1), (130, 30, 2), (70, 62, 0), (33, 128, 3), (40, 130, 1), (37, 256, 0),
                                   (21, 300, 2), (5, 1024, 1), (9, 17, 1)])
def test_ttt_attention_fp32(T, d, s):
    from test_gpu_ttt import _case
    import paper_2503_01840_amd as E
    assert _case(E, T, 4, 2, d, s, torch.float32, 100 + d) < 1e-5        # fp32 sums of up to 1024 terms of order 1


# hidden a multiple of 4 (what the row kernels ask for), query width and intermediate size not; 1, 7, 8, 9 and 17 rows
@pytest.mark.parametrize("hidden,heads,kv_heads,d,inter", [(64, 4, 4, 16, 100), (100, 3, 1, 24, 54), (36, 5, 5, 8, 33), (260, 2, 1, 72, 258)])
@pytest.mark.parametrize("N", [1, 7, 8, 9, 17])
def test_small_models_fp32(hidden, heads, kv_heads, d, inter, N):
    import paper_2503_01840_amd as E
    shape = S.get_shape("c1").with_(name=f"f{hidden}", hidden=hidden, n_heads=heads, n_kv_heads=kv_heads, head_dim=d, intermediate=inter,
                                    vocab=131, draft_vocab=131, n_layers=3, taps=(0, 1, 2))
    model = PL.OracleModel(shape)
    P = 21
    prefix = S.uniform_ints(S.SEED + N, S.TensorIds.PREFIX_TOK, (P,), 0, shape.vocab).numpy()
    pre = O.prefill(shape, model.layer, model.globals(), prefix, rounding="none")
    parent, _ = S.random_tree(5, N, N, 6, 3)
    tok = S.uniform_ints(S.SEED + N, 77, (N,), 0, shape.vocab).numpy().astype(np.int32)
    ref = O.tree_verify(shape, model.layer, model.globals(), tok, np.asarray(parent), lambda l: (pre["k_new"][l], pre["v_new"][l]))
    ctx = E.Eagle3Context(shape, max_batch=1, max_nodes=max(N, 2), max_depth=2, max_topk=2, max_new=4, device=DEV)
    W = PL.device_weights(shape, device=DEV)
    ctx.set_weights(W["target"], W["draft"])
    i32 = lambda v: torch.tensor(np.asarray(v), dtype=torch.int32, device=DEV)
    ks, vs = [], []
    for l in range(shape.n_layers):
        for dst, src in ((ks, pre["k_new"][l]), (vs, pre["v_new"][l])):
            t = torch.zeros(P + N, kv_heads, d, device=DEV)
            t[:P] = torch.from_numpy(np.asarray(src)).float().to(DEV)
            dst.append(t)
    kv = E.KVCache(ks, vs, i32([0, P + N]), i32([P]), P)
    logits, taps = E.eagle3_tree_verify(ctx, i32(tok)[None], i32(parent)[None], kv)
    assert np.max(np.abs(logits[0].cpu().numpy() - ref["logits"])) < 1e-4
    assert np.max(np.abs(taps[:, 0].cpu().numpy() - ref["taps"])) < 1e-4


# heads of 64 and 128: lane groups that share a key; 21 + N keys around a full batch of them (80 and 40), fewer keys than groups
@pytest.mark.parametrize("heads,kv_heads,d", [(4, 2, 64), (3, 1, 128)])
@pytest.mark.parametrize("N", [1, 18, 19, 20, 58, 59, 60, 64])
def test_small_models_fp32_with_wide_heads(heads, kv_heads, d, N):
    test_small_models_fp32(64, heads, kv_heads, d, 100, N)


# the norm inside the products (one sequence) and as a launch of its own (all of them): LM head from 97 rows on, gate/up from 185, q/k/v from
# 337; rows that are no multiple of 8, and a second layer's norm behind the first one's residual sums
@pytest.mark.parametrize("B,N", [(7, 13), (8, 13), (14, 13), (16, 13), (27, 13), (64, 16)])
def test_rows_alone_and_together(B, N):
    import paper_2503_01840_amd as E
    shape = S.get_shape("c1").with_(n_layers=2, taps=(0, 1, 1))
    P = 9
    ctx = E.Eagle3Context(shape, max_batch=B, max_nodes=N, max_depth=2, max_topk=2, max_new=4, device=DEV)
    W = PL.device_weights(shape, device=DEV)
    ctx.set_weights(W["target"], W["draft"])
    i32 = lambda v: torch.tensor(np.asarray(v), dtype=torch.int32, device=DEV)
    tok = S.uniform_ints(S.SEED + N, 77, (B, N), 0, shape.vocab).to(torch.int32).to(DEV)
    parent = i32(np.tile(np.asarray(S.random_tree(5, N, N, 6, 3)[0]), (B, 1)))
    pool = S.normal(S.SEED, 3, (4, B * (P + N), shape.n_kv_heads, shape.head_dim)).float().to(DEV)

    def run(b0, b1):
        t = pool[:, b0 * (P + N):b1 * (P + N)].clone()
        kv = E.KVCache([t[0], t[1]], [t[2], t[3]], i32(np.arange(b1 - b0 + 1) * (P + N)), i32([P] * (b1 - b0)), P)
        logits, taps = E.eagle3_tree_verify(ctx, tok[b0:b1].contiguous(), parent[b0:b1].contiguous(), kv)
        return logits.cpu().numpy(), taps.cpu().numpy(), t.cpu().numpy()

    logits, taps, cache = run(0, B)
    for b in sorted({0, B // 2, B - 1}):
        lg, tp, c = run(b, b + 1)
        assert np.max(np.abs(logits[b] - lg[0])) < 1e-4 and np.max(np.abs(taps[:, b] - tp[:, 0])) < 1e-4
        assert np.max(np.abs(cache[:, b * (P + N):(b + 1) * (P + N)] - c)) < 1e-4
