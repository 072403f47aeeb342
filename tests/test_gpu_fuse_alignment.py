"""Feature fusion from inputs whose address allows no 16-byte loads, and of a width that is not a multiple of four."""
import numpy as np
import pytest
import torch

import eagle3_synth as S
import pipeline as PL
from oracle import eagle3_oracle as O

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("hidden", [256, 258])
@pytest.mark.parametrize("shift", [0, 1, 2])
@pytest.mark.parametrize("M", [1, 5])
def test_fuse_features_at_any_address(hidden, shift, M):
    import paper_2503_01840_amd as E
    shape = S.get_shape("c1").with_(name=f"h{hidden}", hidden=hidden)
    model = PL.OracleModel(shape)
    ctx = E.Eagle3Context(shape, max_batch=1, max_nodes=8, max_depth=2, max_topk=2, max_new=8, device=DEV)
    W = PL.device_weights(shape, device=DEV)
    ctx.set_weights(W["target"], W["draft"])
    taps = S.normal(S.SEED, S.TensorIds.TAPS, (3, M, hidden))
    flat = [torch.zeros(M * hidden + 4, device=DEV) for _ in range(3)]
    for f, t in zip(flat, taps):
        f[shift:shift + M * hidden] = t.reshape(-1).to(DEV)
    g = E.eagle3_fuse_features(ctx, *[f[shift:shift + M * hidden].view(M, hidden) for f in flat])
    ref = O.fuse_features(model.draft()["w_fc"], *[O.as_f64(t) for t in taps])
    assert np.max(np.abs(g.cpu().numpy() - ref)) < 1e-4
