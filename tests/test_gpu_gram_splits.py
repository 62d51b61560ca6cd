"""The row splits of the pivot Gram blocks: the inner solver adds few or small
partials itself and leaves many large ones to a kernel of its own (2w = 64
from five on), so every split count is taken past its edge, at every lane
count, on a ragged pair.  A repeated call has to give the same bits.

Tolerances are those of the other real parity tests: the prescribed sigma to
1e-11 (kappa(X) = 20 and the rounding of a 64-bit Gram leave about 1e-13) and
the contract to 1e-12."""

import pytest

import gsvd_inputs as gi
from contract import assert_contract, max_rel

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,lanes", [(8, 8), (16, 4), (16, 8), (16, 16), (32, 4), (32, 8), (32, 16)])
def test_gram_splits(w, lanes):
    import paper_1909_00101_amd as hz
    n = 4 * w + 5
    F, G, s_true = gi.custom_pair(1100, 1030, n, kappa=20.0, seed=w + lanes)
    Fd, Gd = torch.from_numpy(F).cuda(), torch.from_numpy(G).cuda()
    for splits in (1, 2, 3, 4, 5, 7, 8, 9, 15, 16):
        print(f"w={w} lanes={lanes} splits={splits}", flush=True)
        runs = [hz.gsvd(Fd, Gd, w=w, inner_lanes=lanes, gram_splits=splits) for _ in range(2)]
        r = runs[0]
        assert r["status"] == 0 and r["converged"]
        assert all(torch.equal(r[k], runs[1][k]) for k in ("U", "V", "Z", "sigma"))
        out = {k: r[k].cpu().numpy() for k in ("U", "V", "Z", "sigma", "sigma_f", "sigma_g")}
        assert max_rel(out["sigma"], s_true) < 1e-11
        assert_contract(F, G, out["U"], out["V"], out["Z"], out["sigma_f"], out["sigma_g"],
                        out["sigma"], tol_res=1e-12, tol_orth=1e-12)
