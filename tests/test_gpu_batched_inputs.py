"""The batched binding's outputs for every form its inputs may have: column-major
(copied together), row-major, strided and offset views, one column, one tensor
used twice, a tensor that requires a gradient.  Each has to give the same bits
as a call that may overwrite column-major copies, in storage of its own, and
leave its inputs alone."""

import pytest

import gsvd_inputs as gi

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

OUT = ("U", "V", "Z", "sigma", "sigma_f", "sigma_g")


def _colmajor(t):
    return t.detach().t().contiguous().clone().t()


def _forms():
    for i, n in enumerate((1, 16, 33, 64)):
        F, G, _ = gi.custom_pair(n + 20, n + 9, n, kappa=5.0, seed=i)
        F, G = torch.from_numpy(F).cuda(), torch.from_numpy(G).cuda()
        yield _colmajor(F), _colmajor(G)
        yield F.contiguous(), G.contiguous()
        yield _colmajor(F), G.contiguous()
        big = torch.zeros((n + 3, 2 * (n + 20) + 1), dtype=torch.float64, device="cuda")
        big[2:n + 2, 1::2] = F.t()
        yield big[2:n + 2, 1::2].t(), _colmajor(G)
        flat = torch.zeros(3 + F.numel(), dtype=torch.float64, device="cuda")
        flat[3:] = F.t().reshape(-1)
        yield flat[3:].view(n, n + 20).t(), _colmajor(G)
        f = _colmajor(F)
        yield f, f
        yield _colmajor(F).requires_grad_(), _colmajor(G)


def test_batched_input_forms():
    import paper_1909_00101_amd as hz
    pairs = list(_forms())
    before = [(f.detach().clone(), g.detach().clone()) for f, g in pairs]
    st, rs = hz.gsvd_batched(pairs)
    for (f, g), (f0, g0) in zip(pairs, before):
        assert torch.equal(f, f0) and torch.equal(g, g0)
    st2, ref = hz.gsvd_batched([(_colmajor(f), _colmajor(g)) for f, g in pairs], overwrite=True)
    # the pair with F = G (every angle undetermined) may run out of sweeps, in both
    assert st == st2 and [a["status"] for a in rs] == [b["status"] for b in ref]
    assert all(a["status"] == 0 for a, (f, g) in zip(rs, pairs) if f is not g)
    seen = set()
    for i, (a, b) in enumerate(zip(rs, ref)):
        print(f"pair {i}", flush=True)
        for k in OUT:
            assert torch.equal(a[k], b[k]), k
            assert a[k].stride() == b[k].stride()
            assert a[k].storage_offset() == 0
            assert a[k].untyped_storage().nbytes() == a[k].numel() * 8
            seen.add(a[k].untyped_storage().data_ptr())
    assert len(seen) == len(OUT) * len(rs)
