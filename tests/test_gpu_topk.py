"""Draft trees at draft-vocabulary sizes around the 512-entry spans and the 64 spans one wavefront merges from registers, and at
the K where the merge kernel changes."""
import numpy as np
import pytest
import torch

import eagle3_synth as S
import pipeline as PL

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("Vd", [17, 511, 513, 32768, 32769, 70000])
@pytest.mark.parametrize("D,K,N", [(2, 1, 3), (3, 4, 20), (4, 5, 40), (3, 10, 60), (2, 11, 50), (3, 16, 64)])
def test_draft_expand_over_draft_vocabularies(Vd, D, K, N):
    import paper_2503_01840_amd as E
    base = S.get_shape("c1")
    shape = base.with_(name=f"v{Vd}", draft_vocab=Vd, vocab=max(base.vocab, Vd))
    model = PL.OracleModel(shape)
    ctx = E.Eagle3Context(shape, max_batch=1, max_nodes=64, max_depth=4, max_topk=16, max_new=4, device=DEV)
    W = PL.device_weights(shape, device=DEV)
    ctx.set_weights(W["target"], W["draft"])
    inp = PL.synthetic_step_inputs(shape, n_new=2, prefix=42)
    ks, vs, indptr, plen, P = PL.device_kv([inp["draft_kv"]], 2 + (D - 1) * K, DEV)
    got = E.eagle3_draft_expand(ctx, inp["g_new"].to(DEV), inp["tok_new"].to(DEV), E.KVCache(ks, vs, indptr, plen, P), D, K, N, debug=True)
    torch.cuda.synchronize()
    got = {k: v.cpu().numpy() for k, v in got.items()}
    ref = PL.oracle_draft(shape, model, inp, D, K, N,
                          follow={"pool_tok": got["pool_tok"], "frontier": got["frontier"], "chosen": got["chosen"]})
    for key in ("tree_tok", "parent", "depth", "chosen"):
        assert np.array_equal(got[key], ref[key]), key
    assert np.max(np.abs(got["score"] - ref["score"])) < 1e-4          # fp32 logits and their log-sum-exp, up to D of them added


# draft logits of which only a few are numbers: every id that comes out is one of the vocabulary, the numbers come first
@pytest.mark.parametrize("Vd", [700, 32768, 32769, 70000])
@pytest.mark.parametrize("n_good,K", [(0, 1), (0, 16), (3, 1), (3, 5), (5, 5), (17, 16)])
@pytest.mark.parametrize("nan_bits", [0x7FC00000, -1])                 # -1: all bits set, as in memory filled with 0xFF
def test_draft_expand_with_undefined_logits(Vd, n_good, K, nan_bits):
    import paper_2503_01840_amd as E
    shape = S.get_shape("c1").with_(name=f"n{Vd}", draft_vocab=Vd, vocab=Vd)
    D, N = 3, 2 if K == 1 else 20
    ctx = E.Eagle3Context(shape, max_batch=2, max_nodes=64, max_depth=4, max_topk=16, max_new=4, device=DEV)
    W = PL.device_weights(shape, device=DEV)
    good = np.sort(np.random.RandomState(Vd + K).choice(Vd, n_good, replace=False))
    head = torch.full_like(W["draft"]["lm_head"], nan_bits, dtype=torch.int32).view(torch.float32)
    head[good] = W["draft"]["lm_head"][good]
    W["draft"]["lm_head"] = head
    ctx.set_weights(W["target"], W["draft"])
    inp = PL.synthetic_step_inputs(shape, n_new=2, prefix=42)
    ks, vs, indptr, plen, P = PL.device_kv([inp["draft_kv"]], 2 + (D - 1) * K, DEV)
    kv = E.KVCache(ks, vs, indptr, plen, P)
    got = E.eagle3_draft_expand(ctx, inp["g_new"].to(DEV), inp["tok_new"].to(DEV), kv, D, K, N, debug=True)
    torch.cuda.synchronize()
    got = {k: v.cpu().numpy() for k, v in got.items()}
    pool = got["pool_tok"][1:]
    assert ((pool >= 0) & (pool < Vd)).all()
    for c in range(0, len(pool), K):
        first = pool[c:c + min(n_good, K)]
        assert np.isin(first, good).all() and len(set(first)) == len(first)
    assert (got["parent"][1:] >= 0).all() and (got["parent"][1:] < np.arange(1, N)).all()
    assert (np.diff(got["chosen"]) > 0).all() and got["chosen"].min() >= 1
    g = inp["g_new"].to(DEV)[None, :1].repeat(2, 1, 1).contiguous()
    two = lambda v: torch.tensor([v, v], dtype=torch.int32, device=DEV)
    kv2 = E.KVCache([torch.cat([ks[0], ks[0]])], [torch.cat([vs[0], vs[0]])], torch.tensor([0, len(ks[0]), 2 * len(ks[0])], dtype=torch.int32, device=DEV),
                    two(P), P)
    tok, _ = E.eagle3_draft_chain(ctx, g, two(1)[:, None].contiguous(), two(1), kv2, 2)
    tok = tok.cpu().numpy()[:, 1:]
    d2t = W["draft"]["d2t"].cpu().numpy()
    assert np.isin(tok, d2t[good] if n_good else d2t[:1]).all()


# Pools around the register sizes of the rerank (256, 768) and of more entries than its threads (1024); one forward only; K whose rows take
# every wavefront (16) or leave none free for the candidates (15); rows of one and of two passes.
@pytest.mark.parametrize("D,K,N,hidden", [(1, 1, 2, 256), (1, 4, 5, 256), (1, 16, 12, 256), (4, 9, 60, 256), (2, 15, 64, 256), (4, 16, 64, 256),
                                          (5, 16, 64, 256), (8, 10, 60, 256), (8, 12, 64, 256), (8, 16, 33, 256), (3, 3, 9, 4352), (2, 16, 40, 8192)])
def test_draft_expand_over_pool_sizes_and_widths(D, K, N, hidden):
    import paper_2503_01840_amd as E
    shape = S.get_shape("c1").with_(name=f"p{hidden}", hidden=hidden)
    model = PL.OracleModel(shape)
    ctx = E.Eagle3Context(shape, max_batch=1, max_nodes=64, max_depth=8, max_topk=16, max_new=4, device=DEV)
    W = PL.device_weights(shape, device=DEV)
    ctx.set_weights(W["target"], W["draft"])
    inp = PL.synthetic_step_inputs(shape, n_new=3, prefix=42)
    ks, vs, indptr, plen, P = PL.device_kv([inp["draft_kv"]], 3 + (D - 1) * K, DEV)
    got = E.eagle3_draft_expand(ctx, inp["g_new"].to(DEV), inp["tok_new"].to(DEV), E.KVCache(ks, vs, indptr, plen, P), D, K, N, debug=True)
    torch.cuda.synchronize()
    got = {k: v.cpu().numpy() for k, v in got.items()}
    ref = PL.oracle_draft(shape, model, inp, D, K, N,
                          follow={"pool_tok": got["pool_tok"], "frontier": got["frontier"], "chosen": got["chosen"]})
    for key in ("tree_tok", "parent", "depth", "chosen"):
        assert np.array_equal(got[key], ref[key]), key
    # fp32 logits and their log-sum-exp, 1e-4 for up to three levels as above, each further level adding as much as one of those
    assert np.max(np.abs(got["score"] - ref["score"])) < 1e-4 * max(1.0, D / 3)


# the smallest workspace holds fewer rotary tables than there are forwards: the same tree
@pytest.mark.parametrize("n_new,D,K", [(4, 8, 2), (1, 5, 1), (4, 2, 2)])
def test_draft_expand_in_the_smallest_workspace(n_new, D, K):
    import paper_2503_01840_amd as E
    shape = S.get_shape("c1")
    W = PL.device_weights(shape, device=DEV)
    inp = PL.synthetic_step_inputs(shape, n_new=n_new, prefix=42)
    out = []
    for small in (False, True):
        ctx = E.Eagle3Context(shape, max_batch=1, max_nodes=4, max_depth=8, max_topk=2, max_new=4, device=DEV)
        ctx.set_weights(W["target"], W["draft"])
        beyond = PL.beyond_workspace(ctx, PL.shrink_workspace(ctx)) if small else None
        ks, vs, indptr, plen, P = PL.device_kv([inp["draft_kv"]], n_new + (D - 1) * K, DEV)
        tree = E.eagle3_draft_expand(ctx, inp["g_new"].to(DEV), inp["tok_new"].to(DEV), E.KVCache(ks, vs, indptr, plen, P), D, K, 4)
        torch.cuda.synchronize()
        assert beyond is None or bool((beyond == 171).all())
        out.append((tree, ks[0], vs[0]))
    assert all(torch.equal(out[0][0][n], out[1][0][n]) for n in out[0][0])
    assert torch.equal(out[0][1], out[1][1]) and torch.equal(out[0][2], out[1][2])
