"""The update of Z beside the next step's inner solves (2w = 64, large or wide
pairs, and every mixed solve), with Z_tilde alternating between two buffers.

The dataflow schedule, which updates Z with F and G, has to give the same bits
as the per-step schedule at sizes on both sides of the rule and for both outer
orderings (an odd and an even number of steps).  Elsewhere the tolerances are
those of the other parity tests: the prescribed sigma to 1e-11 and the
contract to 1e-12."""

import pytest

import gsvd_inputs as gi
from contract import assert_contract, max_rel

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

OUT = ("U", "V", "Z", "sigma", "sigma_f", "sigma_g")


def _run(F, G, **kw):
    import paper_1909_00101_amd as hz
    return hz.gsvd(torch.from_numpy(F).cuda(), torch.from_numpy(G).cuda(), raise_on_noconv=False,
                   **kw)


def _check(r, F, G, s_true):
    assert r["status"] == 0 and r["converged"]
    o = {k: r[k].cpu().numpy() for k in OUT}
    assert max_rel(o["sigma"], s_true) < 1e-11
    assert_contract(F, G, o["U"], o["V"], o["Z"], o["sigma_f"], o["sigma_g"], o["sigma"],
                    tol_res=1e-12, tol_orth=1e-12)


@pytest.mark.parametrize("ordering", [1, 2])
@pytest.mark.parametrize("m_f,m_g,n", [(900, 850, 832), (1000, 990, 961), (1100, 1024, 1024),
                                       (2400, 2100, 1024), (2400, 2100, 1601)])
def test_z_beside_the_inner_solves_bitwise(m_f, m_g, n, ordering):
    import paper_1909_00101_amd as hz
    print(f"{m_f}x{m_g}x{n} ordering={ordering}", flush=True)
    F, G, _ = gi.custom_pair(m_f, m_g, n, kappa=20.0, seed=n)
    kw = dict(w=32, inner_lanes=16, inner_max_sweeps=1, max_sweeps=3, ordering=ordering)
    a = _run(F, G, schedule=hz.HZ_SCHED_STEPS, **kw)
    b = _run(F, G, schedule=hz.HZ_SCHED_DATAFLOW, **kw)
    assert a["rot_total"] == b["rot_total"]
    for k in OUT:
        assert torch.equal(a[k], b[k]), k


@pytest.mark.parametrize("lanes", [4, 8])
def test_z_beside_the_inner_solves(lanes):
    F, G, s_true = gi.custom_pair(1100, 1030, 1030, kappa=20.0, seed=lanes)
    for iord in (2, 3):
        _check(_run(F, G, w=32, inner_lanes=lanes, inner_ordering=iord, inner_max_sweeps=1), F, G,
               s_true)


@pytest.mark.parametrize("sort", [0, 1])
@pytest.mark.parametrize("iord", [1, 2, 3])
@pytest.mark.parametrize("lanes", [4, 8, 16])
def test_mixed_side_work(lanes, iord, sort):
    for m_f, m_g, n, ordering in ((300, 290, 64, 2), (500, 420, 203, 1), (700, 600, 384, 2)):
        print(f"lanes={lanes} iord={iord} sort={sort} n={n}", flush=True)
        F, G, s_true = gi.custom_pair(m_f, m_g, n, kappa=20.0, seed=n + lanes)
        r = _run(F, G, mixed=True, w=32, inner_lanes=lanes, inner_ordering=iord, sort=sort,
                 ordering=ordering)
        assert r["sweeps_fp32"] >= 1
        _check(r, F, G, s_true)
