"""The product rounded toward -infinity at the ends of its cases: results at powers
of two (whose lower neighbour has another exponent) and of either sign, products
that vanish, denormals, infinities.  The same bits as the oracle's."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [1.0, 2.0 ** -511, 2.0 ** -537, 2.0 ** 511])
def test_mul_rd_edges(scale):
    import oracle
    import paper_1909_00101_amd as hz
    u = np.nextafter(1.0, 2.0) - 1.0
    m = np.array([0.0, 1.0, 1.0 + u, 1.0 - u / 2, 1.0 - u, 2.0 - u, 1.5, 0.1, 1.0 / 3.0, 2.0 ** -27])
    m = np.r_[m, -m] * scale
    a, b = (g.ravel() for g in np.meshgrid(np.r_[m, np.inf, -np.inf], m))
    c, d = (t.cpu().numpy() for t in hz.eval_mul_rd(torch.from_numpy(a.copy()).cuda(),
                                                    torch.from_numpy(b.copy()).cuda()))
    ref = np.array([oracle.mul_rd(x, y) for x, y in zip(a, b)])
    for got, want in ((c, ref[:, 0]), (d, ref[:, 1])):
        nan = np.isnan(want)
        assert np.array_equal(np.isnan(got), nan)
        assert np.array_equal(got[~nan].view(np.int64), want[~nan].view(np.int64))
