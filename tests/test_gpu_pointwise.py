"""The real 2x2 transformation of the inner solver on pencils of graded
diagonals: what it leaves off the diagonal of both forms, in extended
precision.

Tolerance: the transformed columns are u = b'' and v = s'' with computed
coefficients of a few ulps each (16 eps covers the reciprocals and roots, each
one to two ulps, and the roundings of the pencil's differences).  The
off-diagonal entry is a sum of four terms, each at most |u|_M |v|_M in the
norm of M = |A'|, which exceeds the norm of A' by at most (1 + c)/(1 - c) for a
cosine c of A'; so it is below 64 eps ((1 + c)/(1 - c)) ((1 + |x|)/(1 - |x|))
relative to the diagonal, with the same factor for B'."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps


@pytest.mark.parametrize("grade", [0, 3, 6])
def test_real_2x2_on_graded_pencils(grade):
    import paper_1909_00101_amd as hz
    rng = np.random.default_rng(40 + grade)
    k = 4003
    aii = 10.0 ** rng.uniform(-2, 2, k)
    ajj = aii * 10.0 ** rng.uniform(-2 * grade, 2 * grade, k)
    if grade == 0:                      # nearly equal, exactly equal
        ajj = aii * (1.0 + rng.standard_normal(k) * 10.0 ** rng.uniform(-16, -1, k))
        ajj[::7] = aii[::7]
    c = rng.uniform(-0.9, 0.9, k) * 10.0 ** (-14 * rng.random(k) * (rng.random(k) < 0.5))
    x = rng.uniform(-0.9, 0.9, k) * 10.0 ** (-14 * rng.random(k) * (rng.random(k) < 0.5))
    aij = c * np.sqrt(aii * ajj)
    inp = np.stack([aii, ajj, aij, x], axis=1)
    z = hz.eval_2x2(torch.from_numpy(inp).cuda()).cpu().numpy().astype(np.longdouble)
    assert np.all(np.isfinite(z.astype(np.float64)))
    z11, z21, z12, z22 = z.T
    a, b, o, xx = (v.astype(np.longdouble) for v in (aii, ajj, aij, x))

    def form(p, q, d1, d2, off):
        return p[0] * q[0] * d1 + p[1] * q[1] * d2 + (p[0] * q[1] + p[1] * q[0]) * off
    u, v = (z11, z21), (z12, z22)
    one = np.ones_like(a)
    grow = ((1 + abs(c)) / (1 - abs(c))) * ((1 + abs(x)) / (1 - abs(x)))
    cos_a = abs(form(u, v, a, b, o)) / np.sqrt(form(u, u, a, b, o) * form(v, v, a, b, o))
    cos_b = abs(form(u, v, one, one, xx))
    assert np.max(cos_a / grow) < 64 * EPS
    assert np.max(cos_b / grow) < 64 * EPS
    for p in (u, v):
        assert np.max(abs(form(p, p, one, one, xx) - 1) / grow) < 64 * EPS
    # the larger diagonal entry stays the larger one
    big_i = aii > ajj * (1 + 1e-12)
    assert np.all((form(u, u, a, b, o) > form(v, v, a, b, o))[big_i])
