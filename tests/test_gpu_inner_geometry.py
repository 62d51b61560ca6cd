"""The inner solver at every geometry it is built for (block width, lanes per
column pair, ordering of the pointwise steps), with one and with many inner
sweeps, sorted and not: sigma against the prescribed values and the GSVD
contract, on a ragged pair (bordering columns inside the last block) and on
one whose matrices are a single pivot block.

Tolerances are those of the other real parity tests: the prescribed sigma to
1e-11 (kappa(X) = 20 and the rounding of a 64-bit Gram leave about 1e-13) and
the contract to 1e-12."""

import numpy as np
import pytest

import gsvd_inputs as gi
from contract import assert_contract, max_rel

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GEOMETRY = [(8, 8), (16, 4), (16, 8), (16, 16), (32, 4), (32, 8), (32, 16)]
ORDERINGS = {"mm": 1, "rr": 2, "ring": 3}


@pytest.mark.parametrize("sort", [0, 1])
@pytest.mark.parametrize("inner", [1, 30])
@pytest.mark.parametrize("ordering", sorted(ORDERINGS))
@pytest.mark.parametrize("w,lanes", GEOMETRY)
def test_inner_geometry(w, lanes, ordering, inner, sort):
    import paper_1909_00101_amd as hz
    print(f"w={w} lanes={lanes} {ordering} inner={inner} sort={sort}", flush=True)
    for n, m_f, m_g in ((4 * w + 5, 6 * w + 9, 5 * w), (2 * w, 2 * w, 3 * w + 1)):
        F, G, s_true = gi.custom_pair(m_f, max(m_g, n), n, kappa=20.0, seed=7 * n + lanes)
        r = hz.gsvd(torch.from_numpy(F).cuda(), torch.from_numpy(G).cuda(), w=w,
                    inner_lanes=lanes, inner_ordering=ORDERINGS[ordering],
                    inner_max_sweeps=inner, sort=sort)
        out = {k: r[k].cpu().numpy() for k in ("U", "V", "Z", "sigma", "sigma_f", "sigma_g")}
        assert r["status"] == 0 and r["converged"]
        assert max_rel(out["sigma"], s_true) < 1e-11
        assert_contract(F, G, out["U"], out["V"], out["Z"], out["sigma_f"], out["sigma_g"],
                        out["sigma"], tol_res=1e-12, tol_orth=1e-12)
        # every pair of a sweep once: the first sweep of an unsorted, far from
        # orthogonal block applies them all
        if n == 2 * w and inner == 1:
            one = hz.gsvd(torch.from_numpy(F).cuda(), torch.from_numpy(G).cuda(), w=w,
                          inner_lanes=lanes, inner_ordering=ORDERINGS[ordering],
                          inner_max_sweeps=1, max_sweeps=1, sort=sort, ordering=2)
            pairs = w * (2 * w - 1) if ordering != "mm" else 2 * w * w
            assert one["rot_total"] == pairs


@pytest.mark.parametrize("ordering", ["rr", "ring"])
def test_full_block_on_graded_columns(ordering):
    """Sigma over twelve orders of magnitude: a transformation may be small
    (criterion C1) and still turn the small column of a pair by much, and an
    inner solve ends after a sweep of small ones.  U and V have to come out
    orthonormal to the bound of the other tests, and the pencil diagonal."""
    import paper_1909_00101_amd as hz
    for w, n in ((16, 96), (32, 64)):
        F, G, _ = gi.custom_pair(300, 280, n, kappa=10.0, sig_lo=1e-6, sig_hi=1e6, seed=w)
        r = hz.gsvd(torch.from_numpy(F).cuda(), torch.from_numpy(G).cuda(), w=w,
                    inner_ordering=ORDERINGS[ordering])
        out = {k: r[k].cpu().numpy() for k in ("U", "V", "Z", "sigma", "sigma_f", "sigma_g")}
        assert r["status"] == 0 and r["converged"]
        assert_contract(F, G, out["U"], out["V"], out["Z"], out["sigma_f"], out["sigma_g"],
                        out["sigma"], tol_res=1e-12, tol_orth=1e-12)
