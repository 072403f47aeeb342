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
