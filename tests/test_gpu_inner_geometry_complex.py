"""The complex inner solver at every geometry it is built for: as the real
test of the same name, with the same tolerances."""

import numpy as np
import pytest

import gsvd_inputs as gi
from contract import assert_contract, max_rel

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ORDERINGS = {"mm": 1, "rr": 2, "ring": 3}


@pytest.mark.parametrize("kw", [dict(inner_max_sweeps=1), dict(), dict(sort=0), dict(variant=5)],
                         ids=["block", "full", "unsorted", "variant5"])
@pytest.mark.parametrize("ordering", sorted(ORDERINGS))
@pytest.mark.parametrize("w,lanes", [(8, 8), (16, 8), (16, 16)])
def test_complex_inner_geometry(w, lanes, ordering, kw):
    import paper_1909_00101_amd as hz
    print(f"w={w} lanes={lanes} {ordering} {kw}", flush=True)
    for n, m_f, m_g in ((4 * w + 5, 6 * w + 9, 5 * w), (2 * w, 2 * w, 3 * w + 1)):
        F, G, s_true = gi.custom_pair(m_f, m_g, n, kappa=20.0, seed=7 * n + lanes, is_complex=True)
        r = hz.gsvd(torch.from_numpy(F).cuda(), torch.from_numpy(G).cuda(), w=w,
                    inner_lanes=lanes, inner_ordering=ORDERINGS[ordering], **kw)
        out = {k: r[k].cpu().numpy() for k in ("U", "V", "Z", "sigma", "sigma_f", "sigma_g")}
        assert r["status"] == 0 and r["converged"]
        assert max_rel(out["sigma"], s_true) < 1e-11
        assert_contract(F, G, out["U"], out["V"], out["Z"], out["sigma_f"], out["sigma_g"],
                        out["sigma"], tol_res=1e-12, tol_orth=1e-12)


@pytest.mark.parametrize("grade", [0, 3, 6])
def test_complex_2x2_on_graded_pencils(grade):
    """What the transformation leaves off the diagonal of both forms, in extended
    precision; tolerance as for the real one: 64 eps times (1 + c)/(1 - c) for
    the cosines c of A' and of B' (entries of a few ulps, sums of four terms)."""
    import paper_1909_00101_amd as hz
    eps = np.finfo(np.float64).eps
    rng = np.random.default_rng(90 + grade)
    k = 4003
    aii = 10.0 ** rng.uniform(-2, 2, k)
    ajj = aii * 10.0 ** rng.uniform(-2 * grade, 2 * grade, k)
    if grade == 0:
        ajj = aii * (1.0 + rng.standard_normal(k) * 10.0 ** rng.uniform(-16, -1, k))
        ajj[::7] = aii[::7]

    def cosine():
        c = rng.uniform(0, 0.9, k) * 10.0 ** (-14 * rng.random(k) * (rng.random(k) < 0.5))
        return c * np.exp(2j * np.pi * rng.random(k))
    c, b = cosine(), cosine()
    a = c * np.sqrt(aii * ajj)
    inp = np.stack([aii, ajj, a.real, a.imag, b.real, b.imag], axis=1)
    o = hz.eval_2x2(torch.from_numpy(np.ascontiguousarray(inp)).cuda()).cpu().numpy()
    assert np.all(np.isfinite(o))
    o = o.astype(np.longdouble)
    z11, z21, z12, z22 = o[:, 0], o[:, 1] + 1j * o[:, 2], o[:, 3] + 1j * o[:, 4], o[:, 5]

    def form(p, q, d1, d2, off):
        return (np.conj(p[0]) * q[0] * d1 + np.conj(p[1]) * q[1] * d2
                + np.conj(p[0]) * off * q[1] + np.conj(p[1]) * np.conj(off) * q[0])
    u, v = (z11, z21), (z12, z22)
    al, bl = a.astype(np.clongdouble), b.astype(np.clongdouble)
    d1, d2, one = aii.astype(np.longdouble), ajj.astype(np.longdouble), np.ones(k, np.longdouble)
    grow = ((1 + abs(c)) / (1 - abs(c))) * ((1 + abs(b)) / (1 - abs(b)))
    cos_a = abs(form(u, v, d1, d2, al)) / np.sqrt(abs(form(u, u, d1, d2, al) * form(v, v, d1, d2, al)))
    assert np.max(cos_a / grow) < 64 * eps
    assert np.max(abs(form(u, v, one, one, bl)) / grow) < 64 * eps
    for p in (u, v):
        assert np.max(abs(form(p, p, one, one, bl) - 1) / grow) < 64 * eps
