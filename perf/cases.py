"""What the speed of this library is measured on: whole generalized SVDs through
the Python entry points (``gsvd``, ``gsvd_noalloc``, ``gsvd_batched``), over the
sizes, types and options that the tests, the benchmark and the documentation use.

``listed()`` names the cases, ``draw(rng)`` gives one more case of the same
ranges, ``prepare`` makes the inputs on the GPU, ``run`` is one solve as a program
calls it, ``work`` is what a solve cannot do without and ``exact`` is the result in
64 bits by dense factorizations (numpy).

Inputs: F = U diag(s_f) X, G = V diag(s_g) X with U and V of orthonormal columns, X
of condition number kappa and s_f / s_g one value in every cell of a logarithmic
grid on [sig_lo, sig_hi], so that no two generalized singular values agree to
rounding and the columns of U, V and Z are determined (up to a sign, or a unit
factor for complex pairs, which ``run`` and ``exact`` fix as a program does that
stores or compares decompositions).
"""

import math

import numpy as np
import torch

import paper_1909_00101_amd as hz

EPS = 2.220446049250313e-16

# The launch that the tuner picks for the tall 4096 x 1024 pair (block width 32, one
# inner sweep per block step, ring ordering inside the pivot blocks), for its
# QR-shortened form, for the complex pairs, the mixed form and the batches; a program
# that solves many pairs of one size keeps such a choice.
_TUNED = dict(w=32, inner_max_sweeps=1, inner_ordering=3, inner_lanes=8, gram_splits=8,
              update_rows=48, tol_n=True, keep=True)
_SHORT = dict(w=16, inner_max_sweeps=1, inner_ordering=3, inner_lanes=16, gram_splits=4,
              update_rows=16, qr_shorten=1, tol_n=True, keep=True)
_CPLX = dict(w=16, inner_max_sweeps=1, inner_ordering=3, tol_n=True, keep=True)
_MIXED = dict(w=32, inner_max_sweeps=1, inner_ordering=3, inner_lanes=8, gram_splits=8,
              update_rows=64, tol_n=True, keep=True)
_BATCH = dict(w=32, inner_max_sweeps=1, inner_ordering=3, inner_lanes=16, ordering=2)

_OPTIONS = ("w", "ordering", "inner_ordering", "inner_max_sweeps", "inner_lanes", "gram_splits",
            "update_rows", "qr_shorten", "pivot_qr")


def _case(kind, m_f, m_g, n, kappa, lo, hi, **opt):
    return dict(kind=kind, m_f=m_f, m_g=m_g, n=n, kappa=kappa, sig_lo=lo, sig_hi=hi, **opt)


def listed():
    c = [
        # the smallest ordinary call: the 64 x 32 / 48 x 32 pair of the smoke test, all defaults
        dict(_case("real", 64, 48, 32, 10.0, 1e-2, 1e2, tol_n=True), name="real_64x32"),
        # a serving loop that must not allocate, ragged in every dimension, square G
        dict(_case("noalloc", 333, 65, 65, 50.0, 1e-2, 1e2), name="noalloc_333x65"),
        # an ordinary call with all defaults
        dict(_case("real", 700, 520, 256, 100.0, 1e-2, 1e2), name="real_700x256"),
        # a larger one with all defaults, n no multiple of the block width
        dict(_case("real", 2048, 1500, 630, 100.0, 1e-3, 1e3), name="real_2048x630"),
        # the benchmark's pair at its tuned launch
        dict(_case("real", 4096, 4096, 1024, 100.0, 1e-3, 1e3, **_TUNED), name="real_4096x1024"),
        # the same pair, shortened to 1024 x 1024 first
        dict(_case("real", 4096, 4096, 1024, 100.0, 1e-3, 1e3, **_SHORT), name="short_4096x1024"),
        # block columns too ill-conditioned for Grams: QR factors of the pivot blocks
        dict(_case("real", 1000, 800, 256, 10.0, 1e-3, 1e3, w=32, pivot_qr=1),
             name="pivotqr_1000x256"),
        # complex pairs: a small one with all defaults, and the benchmark's
        dict(_case("complex", 300, 200, 90, 20.0, 1e-2, 1e2), name="complex_300x90"),
        dict(_case("complex", 3072, 2048, 1024, 50.0, 1e-2, 1e2, **_CPLX),
             name="complex_3072x1024"),
        # the largest: mixed precision on the 8192 x 2048 pair
        dict(_case("mixed", 8192, 8192, 2048, 100.0, 1e-2, 1e2, **_MIXED), name="mixed_8192x2048"),
        # many small pairs of uneven sizes in one call, and the benchmark's ensemble
        dict(kind="batched", count=48, n_lo=8, n_hi=64, sig_lo=1e-2, sig_hi=1e2,
             name="batched_48x8_64"),
        dict(kind="batched", count=512, n_lo=16, n_hi=256, sig_lo=1e-2, sig_hi=1e2,
             name="batched_512x16_256", **_BATCH),
    ]
    return c


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One case of the listed ranges: the family by chance, n over the logarithm of its
    range, the row counts between n and a few n."""
    fam = rng.choice(["real", "real", "noalloc", "tuned", "short", "pivotqr", "complex", "complex",
                      "mixed", "batched"])
    kappa = float("%.3g" % 10.0 ** rng.uniform(0.3, 2.0))
    hi = rng.choice([1e2, 1e3])
    lo = 1.0 / hi
    if fam == "batched":
        n_hi = _log_int(rng, 32, 256)
        opt = _BATCH if rng.random() < 0.5 else {}
        return dict(kind="batched", count=_log_int(rng, 8, 512), n_lo=rng.randint(4, n_hi // 2),
                    n_hi=n_hi, sig_lo=1e-2, sig_hi=1e2, **opt)
    n = {"real": lambda: _log_int(rng, 2, 640), "noalloc": lambda: _log_int(rng, 2, 400),
         "tuned": lambda: _log_int(rng, 200, 1200), "short": lambda: _log_int(rng, 128, 1024),
         "pivotqr": lambda: _log_int(rng, 32, 300), "complex": lambda: _log_int(rng, 4, 900),
         "mixed": lambda: _log_int(rng, 256, 1800)}[fam]()
    m_f, m_g = int(n * rng.uniform(1.0, 4.0)) + 1, int(n * rng.uniform(1.0, 4.0)) + 1
    if rng.random() < 0.15:
        m_g = n
    if fam == "tuned":
        return _case("real", m_f, m_g, n, kappa, lo, hi, **_TUNED)
    if fam == "short":
        return _case("real", m_f, m_g, n, min(kappa, 30.0), 1e-2, 1e2, **_SHORT)
    if fam == "pivotqr":
        return _case("real", m_f, m_g, n, kappa, lo, hi, w=rng.choice([16, 32]), pivot_qr=1)
    if fam == "complex":
        opt = _CPLX if n > 128 or rng.random() < 0.5 else {}
        return _case("complex", m_f, m_g, n, min(kappa, 50.0), 1e-2, 1e2, **opt)
    if fam == "mixed":
        return _case("mixed", m_f, m_g, n, kappa, 1e-2, 1e2, **_MIXED)
    opt = dict(tol_n=True) if rng.random() < 0.3 else {}
    return _case(fam, m_f, m_g, n, kappa, lo, hi, **opt)


# ---------------------------------------------------------------- inputs

_DEV = "cuda"


def _units(gen, k, cplx):
    """k random signs, or unit complex numbers."""
    if cplx:
        return torch.polar(torch.ones(k, dtype=torch.float64),
                           2.0 * math.pi * torch.rand(k, generator=gen, dtype=torch.float64)
                           ).to(_DEV)
    return (torch.randint(0, 2, (k,), generator=gen) * 2 - 1).to(torch.float64).to(_DEV)


def _cosines(m, freq):
    """The columns `freq` of the orthonormal cosine transform of order m (m x len(freq))."""
    i = torch.arange(m, dtype=torch.float64, device=_DEV)[:, None] + 0.5
    c = torch.cos(math.pi / m * i * freq.to(torch.float64)[None, :])
    c *= torch.where(freq == 0, math.sqrt(1.0 / m), math.sqrt(2.0 / m))[None, :]
    return c


def _columns(gen, m, n, cplx):
    """m x n with orthonormal columns: n frequencies of the transform of order m drawn at
    random, with the signs (phases) of the rows and columns drawn too."""
    freq = torch.randperm(m, generator=gen)[:n].to(_DEV)
    return _units(gen, m, cplx)[:, None] * _cosines(m, freq) * _units(gen, n, cplx)[None, :]


def _mixing(gen, n, cplx):
    """A square orthogonal (unitary) matrix: two transforms between random signs (phases)."""
    a = _columns(gen, n, n, cplx)
    b = _columns(gen, n, n, cplx)
    return a @ b


def _pair(gen, m_f, m_g, n, kappa, lo, hi, cplx):
    """One pair, column-major, as described at the top."""
    u, v = _columns(gen, m_f, n, cplx), _columns(gen, m_g, n, cplx)
    s = torch.logspace(0.0, -math.log10(kappa), n, dtype=torch.float64, device=_DEV)
    x = (_mixing(gen, n, cplx) * s[None, :]) @ _mixing(gen, n, cplx)
    cell = (torch.arange(n, dtype=torch.float64) + 0.5
            + 0.6 * (torch.rand(n, generator=gen, dtype=torch.float64) - 0.5)) / n
    cell = cell[torch.randperm(n, generator=gen)].to(_DEV)
    sigma = 10.0 ** (math.log10(lo) + (math.log10(hi) - math.log10(lo)) * cell)
    t = torch.sqrt(1.0 + sigma * sigma)
    f = (u * (sigma / t)[None, :]) @ x
    g = (v * (1.0 / t)[None, :]) @ x
    return f.t().contiguous().t(), g.t().contiguous().t()


def _inputs(case, seed):
    gen = torch.Generator().manual_seed(19090 + 7919 * int(seed))
    if case["kind"] != "batched":
        return [_pair(gen, case["m_f"], case["m_g"], case["n"], case["kappa"], case["sig_lo"],
                      case["sig_hi"], case["kind"] == "complex")]
    pairs = []
    for n, m_f, m_g in _batch_sizes(case):
        kappa = 10.0 ** float(2.0 * torch.rand(1, generator=gen))
        pairs.append(_pair(gen, m_f, m_g, n, max(kappa, 1.5), case["sig_lo"], case["sig_hi"],
                           False))
    return pairs


def _batch_sizes(case):
    """The sizes of a batch's pairs, by the case alone: n uniform in its range, rows
    between n and 2n."""
    gen = torch.Generator().manual_seed(11 + case["count"])
    out = []
    for r in torch.rand((case["count"], 3), generator=gen, dtype=torch.float64).tolist():
        n = case["n_lo"] + int(r[0] * (case["n_hi"] - case["n_lo"] + 1))
        out.append((n, n + int(r[1] * (n + 1)), n + int(r[2] * (n + 1))))
    return out


def _reference(n, cplx):
    """A fixed vector: the inner product of it with a column of Z is made positive."""
    gen = torch.Generator().manual_seed(n)
    r = torch.randn(n, generator=gen, dtype=torch.float64)
    return r.to(torch.complex128) if cplx else r


def _options(case):
    kw = {k: case[k] for k in _OPTIONS if k in case}
    if case.get("tol_n"):
        kw["tol"] = case["n"] * EPS
    return kw


# ---------------------------------------------------------------- the cases

def prepare(case, seed):
    kind = case["kind"]
    pairs = _inputs(case, seed)
    st = dict(kind=kind, kw=_options(case))
    if kind == "batched":
        st["pairs"] = pairs
        ns = torch.tensor([p[0].shape[1] for p in pairs])
        cols = torch.repeat_interleave(ns, ns)
        st["ref"] = torch.cat([_reference(int(n), False).repeat(int(n)) for n in ns]).to(_DEV)
        st["lengths"] = cols.to(_DEV)
        ids = torch.arange(len(cols), device=_DEV)
        for key, k in (("u_col", 0), ("v_col", 1)):
            rows = torch.tensor([p[k].shape[0] for p in pairs])
            st[key] = torch.repeat_interleave(ids, torch.repeat_interleave(rows, ns).to(_DEV))
        st["z_col"] = torch.repeat_interleave(ids, st["lengths"])
        return st
    f, g = pairs[0]
    n = case["n"]
    cplx = kind == "complex"
    st.update(f=f, g=g, ref=_reference(n, cplx).to(_DEV))
    if case.get("keep"):
        # a program that solves many pairs of one size keeps the workspace
        import ctypes
        lib = hz.lib()
        size = {"real": lib.hz_dgsvd_work_size, "complex": lib.hz_zgsvd_work_size,
                "mixed": lib.hz_dgsvd_mixed_work_size}[kind]
        p = hz.params(**st["kw"])
        st["work"] = torch.empty(size(ctypes.byref(p), case["m_f"], case["m_g"], n) + 256,
                                 dtype=torch.uint8, device=_DEV)
    if kind == "noalloc":
        # the caller's own buffers, column-major
        st["u"], st["v"] = f.t().contiguous().t().clone(), g.t().contiguous().t().clone()
        st["z"] = torch.empty((n, n), dtype=torch.float64, device=_DEV).t()
        st["s"] = [torch.empty(n, dtype=torch.float64, device=_DEV) for _ in range(3)]
    return st


def _signs(ref, u, v, z):
    """Fixes the sign (unit factor) of every column of u, v and z, in place."""
    d = ref @ z
    d = torch.where(d < 0, -1.0, 1.0) if not d.is_complex() else d.conj() / d.abs()
    return u.mul_(d), v.mul_(d), z.mul_(d)


def run(st):
    if st["kind"] == "batched":
        status, rs = hz.gsvd_batched(st["pairs"], **st["kw"])
        flat = {k: torch.cat([r[k].t().reshape(-1) for r in rs]) for k in ("U", "V", "Z")}
        d = torch.segment_reduce(flat["Z"] * st["ref"], "sum", lengths=st["lengths"])
        d = torch.where(d < 0, -1.0, 1.0).to(torch.float64)
        out = dict(U=flat["U"].mul_(d[st["u_col"]]), V=flat["V"].mul_(d[st["v_col"]]),
                   Z=flat["Z"].mul_(d[st["z_col"]]), status=status)
        for k in ("sigma", "sigma_f", "sigma_g"):
            out[k] = torch.cat([r[k] for r in rs])
        return out
    if st["kind"] == "noalloc":
        u, v, z = st["u"], st["v"], st["z"]
        u.copy_(st["f"])
        v.copy_(st["g"])
        sigma, sigma_f, sigma_g = st["s"]
        status, _ = hz.gsvd_noalloc(u, v, z, sigma, sigma_f, sigma_g, **st["kw"])
    else:
        r = hz.gsvd(st["f"], st["g"], workspace=st.get("work"), mixed=st["kind"] == "mixed",
                    **st["kw"])
        u, v, z, status = r["U"], r["V"], r["Z"], r["status"]
        sigma, sigma_f, sigma_g = r["sigma"], r["sigma_f"], r["sigma_g"]
    u, v, z = _signs(st["ref"], u, v, z)
    return dict(U=u, V=v, Z=z, sigma=sigma, sigma_f=sigma_f, sigma_g=sigma_g, status=status)


def work(case):
    """Bytes: F and G read, U, V, Z and the values written.  Operations: the Grams of F and
    G, the products F Z and G Z, and a dense n x n eigenproblem (9 n^3); four real
    multiplications to a complex one."""
    cplx = case["kind"] == "complex"
    sizes = _batch_sizes(case) if case["kind"] == "batched" else [
        (case["n"], case["m_f"], case["m_g"])]
    nbytes = flops = 0.0
    for n, m_f, m_g in sizes:
        m = m_f + m_g
        nbytes += (16 if cplx else 8) * n * (2 * m + n) + 24 * n
        flops += (4 if cplx else 1) * (3.0 * m * n * n + 9.0 * n ** 3)
    return dict(bytes=nbytes, flops=flops)


# ---------------------------------------------------------------- 64 bits

def _exact_pair(f, g):
    """The GSVD by a QR factorization of [F; G] and the cosine-sine decomposition of its
    orthonormal factor: the values below 1 from the F half, the others from the G half,
    each where it is small."""
    m_f, n = f.shape
    q, r = np.linalg.qr(np.vstack([f, g]))
    q1, q2 = q[:m_f], q[m_f:]

    def right(a):
        return np.linalg.svd(np.linalg.qr(a, mode="r"))[1:]
    c, wh = right(q1)
    w = wh.conj().T
    k = int(np.sum(c > math.sqrt(0.5)))            # the first k: values above 1
    if k:
        s, yh = right(q2 @ w[:, :k])
        w = np.concatenate([w[:, :k] @ yh.conj().T[:, ::-1], w[:, k:]], axis=1)
    a, b = q1 @ w, q2 @ w
    c, s = np.linalg.norm(a, axis=0), np.linalg.norm(b, axis=0)
    z = np.linalg.solve(r, w)
    h = np.hypot(c, s)
    u, v, z, sf, sg = a / c, b / s, z / h, c / h, s / h
    at = np.argsort(-(sf / sg), kind="stable")
    u, v, z, sf, sg = u[:, at], v[:, at], z[:, at], sf[at], sg[at]
    d = _reference(n, np.iscomplexobj(f)).numpy() @ z
    d = d.conj() / np.abs(d)
    return u * d, v * d, z * d, sf / sg, sf, sg


def exact(case, seed):
    if case["kind"] == "mixed" and case["n"] > 1500:
        return None                                # the factorizations take too long
    got = [_exact_pair(f.cpu().numpy(), g.cpu().numpy()) for f, g in _inputs(case, seed)]
    keys = ("U", "V", "Z", "sigma", "sigma_f", "sigma_g")
    if case["kind"] != "batched":
        return dict(zip(keys, got[0]), status=None)
    out = {k: np.concatenate([p[i].T.reshape(-1) for p in got]) for i, k in enumerate(keys[:3])}
    out.update({k: np.concatenate([p[i] for p in got]) for i, k in enumerate(keys) if i > 2})
    return dict(out, status=None)
