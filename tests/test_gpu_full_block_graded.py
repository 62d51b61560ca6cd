"""Full-block solves (30 inner sweeps allowed) of pairs whose sigma spans twelve
orders of magnitude.  An inner solve ends after a sweep without big
transformations, and a small one (criterion C1) can still turn the small column of
a pair by much: every pair of columns of U and V has to be orthogonal to the bound
of the other tests, 1e-12, in every form that runs inner sweeps, also where a
single outer sweep of a single block is all there is."""

import numpy as np
import pytest

import gsvd_inputs as gi
from contract import assert_contract

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ORDERINGS = {"mm": 1, "rr": 2, "ring": 3}


def _check(F, G, r):
    out = {k: r[k].cpu().numpy() for k in ("U", "V", "Z", "sigma", "sigma_f", "sigma_g")}
    assert_contract(F, G, out["U"], out["V"], out["Z"], out["sigma_f"], out["sigma_g"],
                    out["sigma"], tol_res=1e-12, tol_orth=1e-12)
    for q in (out["U"], out["V"]):
        assert np.max(np.abs(q.conj().T @ q - np.eye(q.shape[1]))) < 1e-12


@pytest.mark.parametrize("ordering", sorted(ORDERINGS))
@pytest.mark.parametrize("n,cplx,kw", [
    (320, False, {}), (515, False, {}), (200, True, {}), (333, True, {}),
    (200, False, dict(pivot_qr=1, w=16)), (300, False, dict(pivot_qr=1, w=32)),
    (150, True, dict(pivot_qr=1)), (192, False, dict(variant=4)), (192, False, dict(variant=1))],
    ids=["real", "real_ragged", "complex", "complex_ragged", "qr16", "qr32", "qr_complex", "c2",
         "enhanced"])
def test_graded_full_block(n, cplx, kw, ordering):
    import paper_1909_00101_amd as hz
    F, G, _ = gi.custom_pair(n + 70, n + 41, n, kappa=10.0, sig_lo=1e-6, sig_hi=1e6, seed=n,
                             is_complex=cplx)
    r = hz.gsvd(torch.from_numpy(F).cuda(), torch.from_numpy(G).cuda(),
                inner_ordering=ORDERINGS[ordering], **kw)
    assert r["status"] == 0 and r["converged"]
    _check(F, G, r)


@pytest.mark.parametrize("ordering", sorted(ORDERINGS))
@pytest.mark.parametrize("cplx,w", [(False, 8), (False, 16), (False, 32), (True, 8), (True, 16)])
def test_graded_single_block_and_sweep(w, cplx, ordering):
    import paper_1909_00101_amd as hz
    n = 2 * w
    for seed in range(4):
        F, G, _ = gi.custom_pair(n + 30, n + 20, n, kappa=10.0, sig_lo=1e-6, sig_hi=1e6,
                                 seed=100 + seed, is_complex=cplx)
        r = hz.gsvd(torch.from_numpy(F).cuda(), torch.from_numpy(G).cuda(), w=w, pivot_qr=1,
                    inner_ordering=ORDERINGS[ordering], max_sweeps=1)
        assert r["sweeps"] == 1
        _check(F, G, r)


@pytest.mark.parametrize("schedule", [0, 1])
@pytest.mark.parametrize("ordering", sorted(ORDERINGS))
def test_graded_batched(ordering, schedule):
    import paper_1909_00101_amd as hz
    pairs = [gi.custom_pair(n + 40, n + 25, n, kappa=10.0, sig_lo=1e-6, sig_hi=1e6, seed=n)[:2]
             for n in (24, 57, 96, 160)]
    st, rs = hz.gsvd_batched([tuple(torch.from_numpy(a).cuda() for a in p) for p in pairs],
                             inner_ordering=ORDERINGS[ordering], schedule=schedule)
    assert st == 0
    for (F, G), r in zip(pairs, rs):
        _check(F, G, r)
