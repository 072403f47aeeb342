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
