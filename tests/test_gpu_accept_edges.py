"""The acceptance walk at vocabulary sizes around its 512-entry pieces and 2048-entry chunks, with tied maxima, with logits whose
address or row length forbids 16-byte loads, and with more rows than the walk has wavefronts."""
import numpy as np
import pytest
import torch

import eagle3_synth as S
from oracle import eagle3_oracle as O

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("V", [1, 5, 511, 512, 2047, 2048, 2052, 4103, 6148, 40001])
@pytest.mark.parametrize("N", [1, 7, 16, 17, 64])
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("temperature", [0.0, 0.7])
def test_accept_matches_the_oracle(V, N, shift, temperature):
    import paper_2503_01840_amd as E
    B = 3
    rs = np.random.RandomState(V + 7 * N + shift)
    lg = rs.randn(B, N, V).astype(np.float32)
    if temperature == 0.0:
        lg = np.round(lg)                                    # many equal maxima: the smallest id wins
    parent = np.stack([S.random_tree(V, b, N, 8, 4)[0] for b in range(B)]).astype(np.int32)
    tok = rs.randint(0, V, (B, N)).astype(np.int32)
    for b in range(B):                                       # some nodes hold the token their parent's row prefers
        for i in range(1, N):
            if rs.rand() < 0.5:
                tok[b, i] = int(lg[b, parent[b, i]].argmax())
                lg[b, parent[b, i], tok[b, i]] += 3.0 if temperature else 0.0
    U = rs.rand(B, 2 * N).astype(np.float32)
    flat = torch.zeros(B * N * V + 1, device=DEV)
    flat[shift:shift + B * N * V] = torch.from_numpy(lg.reshape(-1)).to(DEV)
    d = lambda a: torch.from_numpy(a).to(DEV)
    got = E.eagle3_accept_static(flat[shift:shift + B * N * V].view(B, N, V), d(tok), d(parent), temperature,
                                 d(U) if temperature else None)
    n, path, bonus = [t.cpu().numpy() for t in got]
    for b in range(B):
        if temperature == 0.0:
            want = O.accept_greedy(lg[b].astype(np.float64), tok[b], parent[b])
        else:
            *want, margin = O.accept_stochastic(lg[b].astype(np.float64), tok[b], parent[b], temperature, U[b])
            if margin < 1e-5:                                # a uniform within the rounding of fp32 sums over V entries
                continue
        assert (int(n[b]), int(bonus[b])) == (want[0], want[2])
        assert path[b, :want[0] + 1].tolist() == list(want[1]) and (path[b, want[0] + 1:] == -1).all()


# more chunks than lanes (131072 entries), and node counts around the rows of a wavefront (16, 32, 48)
@pytest.mark.parametrize("V,N", [(131072, 33), (131073, 5), (133124, 17), (140000, 64), (2052, 31), (2052, 32), (2052, 33), (2052, 48), (2052, 49)])
@pytest.mark.parametrize("temperature", [0.0, 0.7])
def test_accept_over_many_chunks_and_rows(V, N, temperature):
    test_accept_matches_the_oracle(V, N, 0, temperature)
