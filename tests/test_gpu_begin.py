"""The first launch of a pass: residual rows from an embedding table or a residual stream that start anywhere, rows of one and of two passes
of a workgroup, trees of one node up to the largest, prompts around a workgroup's 4 or 16 rows of bookkeeping."""
import numpy as np
import pytest
import torch

import eagle3_synth as S
from oracle import eagle3_oracle as O
import pipeline as PL

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _shape(dtype, hidden):
    base = S.get_shape("c1") if dtype == "fp32" else S.get_shape("c2").with_(n_heads=4, n_kv_heads=2, intermediate=512)
    return base.with_(name=f"b{hidden}", hidden=hidden, vocab=1024, draft_vocab=512, n_layers=1, taps=(0, 0, 0))


def _shifted(t, by):
    """The same values, `by` elements behind an aligned address."""
    flat = torch.empty(t.numel() + by, dtype=t.dtype, device=t.device)
    flat[by:] = t.reshape(-1)
    return flat[by:].reshape(t.shape)


def _trees(B, N):
    return torch.as_tensor(np.stack([S.random_tree(5, b, N, 8, 2)[0] for b in range(B)]).astype(np.int32), device=DEV)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("hidden,B,N", [(256, 1, 1), (256, 3, 17), (256, 2, 64), (4352, 1, 33)])
def test_residual_rows_from_anywhere(dtype, hidden, B, N):
    import paper_2503_01840_amd as E
    shape = _shape(dtype, hidden)
    W = PL.device_weights(shape, device=DEV, draft=False)["target"]
    P = 21
    tok = S.uniform_ints(S.SEED, S.TensorIds.TREE_TOK, (B, N), 0, shape.vocab).to(torch.int32).to(DEV)
    k, v = (torch.cat([t] * B).to(DEV) for t in S.kv_layer(shape, 0, P + N))
    i32 = lambda a: torch.tensor(a, dtype=torch.int32, device=DEV)
    x_in = W["embed"][tok.long()].float().contiguous()
    out = []
    for embed, x in [(W["embed"], None), (_shifted(W["embed"], 1), None), (W["embed"], x_in), (W["embed"], _shifted(x_in, 1))]:
        ctx = E.Eagle3Context(shape, max_batch=B, max_nodes=N, max_depth=2, max_topk=2, max_new=4, device=DEV)
        ctx.set_weights({**W, "embed": embed}, None)
        kv = E.KVCache([k.clone()], [v.clone()], i32([b * (P + N) for b in range(B + 1)]), i32([P] * B), P)
        x_out, logits = E.eagle3_tree_verify_layers(ctx, tok, _trees(B, N), kv, x, 0, 1, want_logits=True)
        nothing, _ = E.eagle3_tree_verify_layers(ctx, tok, _trees(B, N), kv, x, 0, 0)
        torch.cuda.synchronize()
        assert torch.equal(nothing, x_in)
        out.append((x_out, logits, kv.k_layers[0], kv.v_layers[0]))
    assert torch.isfinite(out[0][1]).all()
    for o in out[1:]:
        assert all(torch.equal(a, b) for a, b in zip(o, out[0]))


# the same prompt at once and in two calls: bookkeeping of the rows of a chunk, lengths, last features, and the draft's cache: each call adds the rows
# of its positions but the last, those of the second call behind those of the first
@pytest.mark.parametrize("T,cut", [(2, 1), (5, 4), (17, 16), (18, 1), (65, 33)])
def test_prompts_in_two_calls(T, cut):
    import paper_2503_01840_amd as E
    shape = _shape("fp32", 256)
    W = PL.device_weights(shape, device=DEV)
    ctx = E.Eagle3Context(shape, max_batch=1, max_nodes=64, max_depth=2, max_topk=2, max_new=64, device=DEV)
    ctx.set_weights(W["target"], W["draft"])
    tokens = S.uniform_ints(S.SEED, S.TensorIds.TREE_TOK, (T,), 0, shape.vocab).to(torch.int32).to(DEV)
    i32 = lambda a: torch.tensor(a, dtype=torch.int32, device=DEV)
    cache = lambda: E.KVCache([torch.zeros(T, shape.n_kv_heads, shape.head_dim, device=DEV)], [torch.zeros(T, shape.n_kv_heads, shape.head_dim, device=DEV)],
                              i32([0, T]), i32([0]), 0)
    kv, dkv = cache(), cache()
    g, logits = E.eagle3_prefill(ctx, tokens, kv, dkv)
    kv2, dkv2 = cache(), cache()
    E.eagle3_prefill(ctx, tokens[:cut], kv2, dkv2)
    assert (int(kv2.prefix_len[0]), int(dkv2.prefix_len[0])) == (cut, cut - 1)
    g2, logits2 = E.eagle3_prefill(ctx, tokens[cut:], kv2, dkv2)
    torch.cuda.synchronize()
    assert (int(kv.prefix_len[0]), int(dkv.prefix_len[0])) == (T, T - 1) and (int(kv2.prefix_len[0]), int(dkv2.prefix_len[0])) == (T, T - 2)
    model = PL.OracleModel(shape)
    dw, emb, toks = model.draft(), model.globals()["embed"], tokens.cpu().numpy()
    pre = O.prefill(shape, model.layer, model.globals(), toks)
    g_all = O.fuse_features(dw["w_fc"], *pre["taps"])
    Kd = np.zeros((T, shape.n_kv_heads, shape.head_dim)); Vd = np.zeros_like(Kd)
    for lo, hi, at in [(0, cut - 1, 0), (cut, T - 1, cut - 1)]:        # positions, and their place in the draft's cache
        if hi > lo:
            O.draft_forward(shape, dw, emb, g_all[lo:hi], toks[lo + 1:hi + 1], at + np.arange(hi - lo), Kd, Vd, at, at, np.tril(np.ones((hi - lo, hi - lo), bool)),
                            lambda a: a)
    for got, want in [(dkv2.k_layers[0], Kd), (dkv2.v_layers[0], Vd)]:
        assert np.max(np.abs(got.cpu().numpy() - want)) < 1e-4          # zeros behind the last row among them
    for got, want in [(dkv2.k_layers[0], dkv.k_layers[0]), (dkv2.v_layers[0], dkv.v_layers[0])]:
        assert torch.allclose(got[:cut - 1], want[:cut - 1], rtol=1e-4, atol=1e-4)
    # fp32 sums of other row groups: a few last bits of values of order one
    for a, b in [(g, g2), (logits, logits2), (kv.k_layers[0], kv2.k_layers[0]), (kv.v_layers[0], kv2.v_layers[0])]:
        assert torch.allclose(a, b, rtol=1e-4, atol=1e-4)
