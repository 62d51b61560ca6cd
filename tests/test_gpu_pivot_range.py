"""Pivots at the ends of the exponent range: squares of their differences
overflow or underflow.

A pair that is orthogonal already is left alone whatever its diagonal entries,
also beside pairs of its wave that are transformed or change places: a diagonal
F over an identity G, with and without a dense block of moderate values in
other columns, is solved as at ordinary scales.  Tolerance: the values of the
diagonal part are quotients of column norms (8 eps); those of the dense block
come out to 1e-12, the bound of the other tests of pairs as well conditioned.

A pivot that needs a transformation there has none in doubles.  The 2x2
transformation of such a pencil is not finite, or it does what it says, and a
solve that meets one ends with an error and not with values."""

import numpy as np
import pytest

import gsvd_inputs as gi

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps
FORMS = [dict(w=8), dict(w=16), dict(w=16, inner_ordering=3), dict(w=16, inner_ordering=1),
         dict(w=16, sort=0), dict(w=32), dict(w=32, inner_ordering=3)]


def _solve(F, G, kw):
    import paper_1909_00101_amd as hz
    return hz.gsvd(torch.from_numpy(np.asfortranarray(F)).cuda(),
                   torch.from_numpy(np.asfortranarray(G)).cuda(), **kw)


@pytest.mark.parametrize("cplx", [False, True], ids=["real", "complex"])
@pytest.mark.parametrize("dense", [False, True], ids=["diagonal", "beside_dense"])
@pytest.mark.parametrize("scale", [1e-80, 1e80, 1e120, 1e150])
def test_orthogonal_columns_at_any_scale(scale, dense, cplx):
    n, k = 40, 12
    F0, G0, s0 = gi.custom_pair(20, 18, k, kappa=3.0, seed=2, is_complex=cplx)
    F, G = np.zeros((n + 20, n), F0.dtype), np.zeros((n + 18, n), F0.dtype)
    d = np.arange(1.0, n + 1) * scale              # ascending: every pair changes places
    F[:n], G[:n] = np.diag(d), np.eye(n)
    if dense:
        F[:, 5:5 + k], G[:, 5:5 + k] = 0.0, 0.0
        F[n:, 5:5 + k], G[n:, 5:5 + k] = F0, G0
        d = np.delete(d, np.arange(5, 5 + k))
    for kw in FORMS:
        if cplx and kw["w"] == 32:
            continue
        print(scale, cplx, dense, kw, flush=True)
        r = _solve(F, G, kw)
        assert r["status"] == 0 and r["converged"]
        s = r["sigma"].cpu().numpy()
        big = s > 1e40 if scale > 1 else s < 1e-40
        assert np.max(np.abs(s[big] - d[::-1]) / d[::-1]) < 8 * EPS
        if dense:
            assert np.max(np.abs(s[~big] - np.sort(s0)[::-1]) / np.sort(s0)[::-1]) < 1e-12


@pytest.mark.parametrize("cplx", [False, True], ids=["real", "complex"])
@pytest.mark.parametrize("scale", [1e-150, 1e-100, 1e100, 1e150])
def test_no_values_from_pivots_out_of_range(scale, cplx):
    import paper_1909_00101_amd as hz
    F, G, _ = gi.custom_pair(49, 45, 40, kappa=3.0, seed=1, is_complex=cplx)
    for kw in FORMS:
        if cplx and kw["w"] == 32:
            continue
        print(scale, cplx, kw, flush=True)
        with pytest.raises(hz.GsvdError):
            _solve(F * scale, G, kw)


@pytest.mark.parametrize("cplx", [False, True], ids=["real", "complex"])
def test_2x2_finite_only_if_it_diagonalizes(cplx):
    """NaN, infinite, overflowing and underflowing pencils (a_ii, a_jj, a_ij) with
    moderate b_ij; 64 eps (1 + c)/(1 - c) for |c| = |x| = 1/2 as at ordinary scales."""
    import paper_1909_00101_amd as hz
    v = [np.nan, np.inf, 1e-300, 1e-200, 1e-100, 1.0, 1e100, 1e200, 1e300]
    a, b, x = (g.ravel() for g in np.meshgrid(v, v, [-0.5, 0.0, 0.5], indexing="ij"))
    with np.errstate(all="ignore"):
        o = 0.5 * np.sqrt(a) * np.sqrt(b)
    cols = [a, b, 0.6 * o, 0.8 * o, 0.8 * x, 0.6 * x] if cplx else [a, b, o, x]
    with np.errstate(all="ignore"):
        inp = np.stack(cols, axis=1)
    r = hz.eval_2x2(torch.from_numpy(np.ascontiguousarray(inp)).cuda()).cpu().numpy()
    r = r.astype(np.longdouble)
    if cplx:
        z11, z21, z12, z22 = r[:, 0], r[:, 1] + 1j * r[:, 2], r[:, 3] + 1j * r[:, 4], r[:, 5]
        with np.errstate(all="ignore"):
            off = (inp[:, 2] + 1j * inp[:, 3]).astype(np.clongdouble)
    else:
        z11, z21, z12, z22 = r.T
        off = o.astype(np.longdouble)
    fin = np.all(np.isfinite(r.astype(np.float64)), axis=1)
    la, lb = a.astype(np.longdouble), b.astype(np.longdouble)

    def form(p, q):
        return (np.conj(p[0]) * q[0] * la + np.conj(p[1]) * q[1] * lb
                + np.conj(p[0]) * off * q[1] + np.conj(p[1]) * np.conj(off) * q[0])
    u, w = (z11, z21), (z12, z22)
    with np.errstate(all="ignore"):
        cos = abs(form(u, w)) / np.sqrt(abs(form(u, u))) / np.sqrt(abs(form(w, w)))
    ok = cos < 64 * EPS * 9
    assert np.all(ok[fin]), inp[fin & ~ok]
    mid = (a == 1.0) & (b == 1.0)
    assert np.all(fin[mid]) and mid.any()
