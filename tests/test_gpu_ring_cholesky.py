"""The blocked Cholesky of the ring inner solver: a zero pivot in every panel of
16 columns and at its edges is reported, and a small positive one is not, at
each geometry.  Two equal columns of G that are alone in their row make their
Gram entries and so the second pivot exact, whatever the other columns are."""

import numpy as np
import pytest

import gsvd_inputs as gi

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _pair(n, i, j, eps):
    F, G, _ = gi.custom_pair(2 * n, 2 * n, n, kappa=10.0, seed=n + j)
    G[:2, :] = 0.0
    G[:, i] = 0.0
    G[0, i] = 1.0
    G[:, j] = G[:, i]
    G[1, j] = eps
    return F, G


@pytest.mark.parametrize("w,lanes", [(16, 8), (16, 16), (32, 4), (32, 8), (32, 16)])
def test_ring_cholesky_pivots(w, lanes):
    import paper_1909_00101_amd as hz
    n = 2 * w
    last = {16: [1, 15, 16, 17, 31], 32: [1, 15, 16, 31, 32, 33, 47, 48, 62, 63]}[w]
    for j in last:
        print(f"w={w} lanes={lanes} column {j}", flush=True)
        for eps in (0.0, 1e-4):
            F, G = _pair(n, 0, j, eps)
            run = lambda: hz.gsvd(torch.from_numpy(np.asfortranarray(F)).cuda(),
                                  torch.from_numpy(np.asfortranarray(G)).cuda(), w=w,
                                  inner_lanes=lanes, inner_ordering=3)
            if eps:
                assert run()["status"] == 0
                continue
            with pytest.raises(hz.GsvdError) as e:
                run()
            assert e.value.status == hz.HZ_ECHOL
            assert e.value.info.failed_pair >= 0
