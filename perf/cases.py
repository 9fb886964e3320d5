"""The work that this library is measured on: the back-transformation of
tridiagonal eigenvectors in its single and batched forms, the second
back-transformation, and whole standard and generalized eigensolves.

listed() holds fixed cases, draw() gives more of the same ranges, prepare()
makes a case's device inputs from a seed, run() is one pass through the public
entry points, work() counts what a pass cannot do without, and exact() is the
same result in plain float64 without the library.
"""
import math
import random

import numpy as np
import torch

import paper_1811_01277_amd as elpa

_DT = {"r64": torch.float64, "r32": torch.float32, "c64": torch.complex128}
_BYTES = {"r64": 8, "r32": 4, "c64": 16}
_FLOPS = {"r64": 1, "r32": 1, "c64": 4}  # real operations per counted real one


def listed():
    return [
        # the smallest stated workload: a lone small problem at the narrow
        # band, where latency counts
        dict(name="trafo r64 512 nbw32", kind="trafo", n=512, nev=512, nbw=32, dtype="r64"),
        # the small end of an SCF stream (n = 1000 .. 6000, all eigenvectors)
        dict(name="trafo r64 1000", kind="trafo", n=1000, nev=1000, nbw=64, dtype="r64"),
        # early SCF steps in single precision, some of the eigenvectors, odd
        # sizes
        dict(name="trafo r32 2501x1251", kind="trafo", n=2501, nev=1251, nbw=64, dtype="r32"),
        # a Hermitian (k-point) problem of ordinary size
        dict(name="trafo c64 1500", kind="trafo", n=1500, nev=1500, nbw=64, dtype="c64"),
        # the middle of the SCF stream
        dict(name="trafo r64 4500", kind="trafo", n=4500, nev=4500, nbw=64, dtype="r64"),
        # a tenth of the eigenvectors of a mid-size problem
        dict(name="trafo r64 8192x819", kind="trafo", n=8192, nev=819, nbw=64, dtype="r64"),
        # the headline: all eigenvectors at n = 20000
        dict(name="trafo r64 20000", kind="trafo", n=20000, nev=20000, nbw=64, dtype="r64"),
        # many uneven small problems in one call
        dict(name="batch r64 256 nbw32", kind="batch", count=256, lo=200, hi=2000, nbw=32,
             dtype="r64", sizes=401),
        # band -> full, the second step of every eigenvector chain
        dict(name="bt2 r64 6000x3000", kind="bt2", n=6000, nev=3000, nbw=64, dtype="r64"),
        # whole solves: a small real one with all eigenvectors, ...
        dict(name="solve r64 1000", kind="solve", n=1000, nev=1000, nbw=64, dtype="r64"),
        # ... a larger one with a fifth of them, ...
        dict(name="solve r64 4000x800", kind="solve", n=4000, nev=800, nbw=64, dtype="r64"),
        # ... and a generalized Hermitian one, overlap matrix included
        dict(name="gsolve c64 700", kind="gsolve", n=700, nev=700, nbw=32, dtype="c64"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["trafo", "trafo", "trafo", "batch", "bt2", "solve", "gsolve"])
    dtype = rng.choice(["r64", "r64", "r32", "c64"])
    nbw = rng.choice([32, 64, 64])
    if kind == "batch":
        lo = _log_int(rng, 150, 1000)
        return dict(kind=kind, count=_log_int(rng, 4, 128), lo=lo,
                    hi=lo + _log_int(rng, 100, 1500), nbw=nbw, dtype=dtype,
                    sizes=rng.randrange(1 << 20))
    if kind in ("solve", "gsolve"):
        dtype = rng.choice(["r64", "r64", "c64"])
        n = _log_int(rng, 150, 3000)
        nev = n if rng.random() < 0.5 else max(1, int(n * rng.uniform(0.1, 1.0)))
        return dict(kind=kind, n=n, nev=nev, nbw=nbw, dtype=dtype)
    n = _log_int(rng, 300, 7000)
    nev = n if rng.random() < 0.5 else max(1, int(n * rng.uniform(0.1, 1.0)))
    return dict(kind=kind, n=n, nev=nev, nbw=nbw, dtype=dtype)


def _sizes(case):
    r = random.Random(case["sizes"])
    return [r.randint(case["lo"], case["hi"]) for _ in range(case["count"])]


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _randn(shape, dtype, g):
    if dtype == "c64":
        z = torch.randn((*shape, 2), generator=g, device="cuda", dtype=torch.float64)
        return torch.view_as_complex(z) * math.sqrt(0.5)
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float64)


def _tau(nrm2, dtype, g):
    if dtype == "c64":  # any phase keeps the reflector unitary
        th = torch.rand(nrm2.shape, generator=g, device="cuda", dtype=torch.float64)
        return (1.0 - torch.polar(torch.ones_like(th), th * (2 * math.pi))) / nrm2
    return 2.0 / nrm2


def _reflectors(n, b, dtype, g):
    """Reflectors of a bulge chase in the library's slot order (sweep, step):
    unit lead, entries of scale 1/sqrt(b), zero past each one's length."""
    s = torch.arange(n - 1, device="cuda")
    J = (n - 1 - s + b - 1) // b
    sweep = torch.repeat_interleave(s, J)
    first = torch.repeat_interleave(torch.cumsum(J, 0) - J, J)
    j = torch.arange(sweep.numel(), device="cuda") - first
    L = torch.clamp(n - (sweep + 1 + j * b), max=b)
    v = _randn((sweep.numel(), b), dtype, g) * (1.0 / math.sqrt(b))
    v[:, 0] = 1.0
    v.masked_fill_(torch.arange(b, device="cuda")[None, :] >= L[:, None], 0.0)
    tau = _tau((v.real**2 + v.imag**2 if dtype == "c64" else v * v).sum(1), dtype, g)
    if dtype != "c64":
        tau.masked_fill_(L == 1, 0.0)
    return v.reshape(-1).to(_DT[dtype]), tau.to(_DT[dtype])


def _block(n, nev, dtype, g):
    """Column-major (n, nev) block with entries the size of eigenvectors'."""
    return (_randn((nev, n), dtype, g) * (1.0 / math.sqrt(n))).to(_DT[dtype]).t()


def _trafo_inputs(n, nev, nbw, dtype, g):
    hh, tau = _reflectors(n, nbw, dtype, g)
    return _block(n, nev, dtype, g), hh, tau, nbw


def _hermitian(n, dtype, g):
    x = _randn((n, n), dtype, g)
    return ((x + x.mH) / 2).contiguous().t()


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    kind, dtype = case["kind"], case["dtype"]
    st = {"kind": kind}
    if kind == "trafo":
        st["p"] = _trafo_inputs(case["n"], case["nev"], case["nbw"], dtype, g)
    elif kind == "batch":
        st["p"] = [_trafo_inputs(n, n, case["nbw"], dtype, g) for n in _sizes(case)]
    elif kind == "bt2":
        n, b = case["n"], case["nbw"]
        N = max(n - b, 1)
        rows = torch.arange(n, device="cuda")[None, :]
        lead = torch.arange(N, device="cuda")[:, None] + b
        v = _randn((N, n), dtype, g) / torch.sqrt((n + b - lead).clamp(min=1).double())
        v.masked_fill_(rows < lead, 0.0)
        v.masked_fill_(rows == lead, 1.0)
        nrm2 = (v.real**2 + v.imag**2 if dtype == "c64" else v * v).sum(1)
        st["tau"] = _tau(nrm2, dtype, g).to(_DT[dtype])
        st["v"] = v.to(_DT[dtype]).t()
        st["q"] = _block(n, case["nev"], dtype, g)
        st["nbw"] = b
    else:
        n = case["n"]
        st.update(a=_hermitian(n, dtype, g), nev=case["nev"], nbw=case["nbw"])
        if kind == "gsolve":  # an overlap matrix: positive definite, near diagonal
            st["b"] = _hermitian(n, dtype, g) * (0.5 / math.sqrt(n))
            st["b"].diagonal().add_(2.0)
    return st


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def _fix_sign(z):
    """Eigenvectors are free up to a factor of modulus one: a program that
    stores or compares them makes the largest entry real and positive."""
    p = torch.gather(z, 0, z.abs().argmax(0, keepdim=True))
    return z * (p.conj() / p.abs())


def run(st):
    kind = st["kind"]
    if kind == "trafo":
        q, hh, tau, nbw = st["p"]
        return elpa.hh_trafo(q, hh, tau, nbw)
    if kind == "batch":
        elpa.hh_trafo_batched(st["p"])
        return torch.cat([p[0].t().reshape(-1) for p in st["p"]])
    if kind == "bt2":
        return elpa.bt2_trafo(st["q"], st["v"], st["tau"], st["nbw"])
    # the solvers overwrite their matrices, which an SCF program sets up anew
    if kind == "solve":
        lam, z = elpa.eigenvectors(st["a"].clone(), st["nev"], st["nbw"])
    else:
        lam, z = elpa.generalized_eigenvectors(st["a"].clone(), st["b"].clone(), st["nev"],
                                               st["nbw"])
    return {"lam": lam, "z": _fix_sign(z)}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    es, w, b = _BYTES[case["dtype"]], _FLOPS[case["dtype"]], case["nbw"]

    def trafo(n, nev):
        slots = n * n / (2 * b) + n / 2
        return es * (2 * n * nev + slots * (b + 1)), 2 * w * n * (n - 1) * nev

    if case["kind"] == "trafo":
        by, fl = trafo(case["n"], case["nev"])
    elif case["kind"] == "batch":
        each = [trafo(n, n) for n in _sizes(case)]
        by, fl = sum(x[0] for x in each), sum(x[1] for x in each)
    elif case["kind"] == "bt2":
        n, nev = case["n"], case["nev"]
        N = max(n - b, 1)
        by, fl = es * (2 * n * nev + n * n / 2), 2 * w * nev * N * (N + 1)
    else:
        n, nev = case["n"], case["nev"]
        # reduction to band and to tridiagonal form, both back-transformations
        # (the tridiagonal solve's count depends on the values: left out)
        by = es * (n * n + n * nev)
        fl = w * (4 * n**3 / 3 + 6 * n * n * b + 4 * n * n * nev)
        if case["kind"] == "gsolve":  # factor, inverse, both transformations
            by += es * n * n
            fl += w * (2 * n**3 / 3 + 2 * n**3 + n * n * nev)
    return {"bytes": float(by), "flops": float(fl)}


# ---------------------------------------------------------------------------
# the same in plain float64
# ---------------------------------------------------------------------------
def _exact_trafo(q, hh, tau, b):
    n, nev = q.shape
    wide = torch.complex128 if q.is_complex() else torch.float64
    x = torch.zeros((n + b, nev), device=q.device, dtype=wide)
    x[:n] = q
    v, t = hh.to(wide).reshape(-1, b), tau.to(wide)
    # slots run sweep by sweep from s = 0: walk them from the back; the
    # reflectors of one sweep share no rows
    end = t.numel()
    for s in range(n - 2, -1, -1):
        J = (n - 1 - s + b - 1) // b
        vs, ts = v[end - J:end], t[end - J:end]
        end -= J
        rows = x[s + 1:s + 1 + J * b].view(J, b, nev)
        y = torch.bmm(vs.conj().resolve_conj().unsqueeze(1), rows)
        rows.baddbmm_((vs * ts[:, None]).unsqueeze(2), y, alpha=-1)
    return x[:n]


def exact(case, seed):
    kind = case["kind"]
    if kind in ("trafo", "bt2"):
        if case["n"] ** 2 * case["nev"] > 1e12:
            return None  # minutes
    st = prepare(case, seed)
    if kind == "trafo":
        return _exact_trafo(*st["p"])
    if kind == "batch":
        if sum(_sizes(case)) > 400000:
            return None  # that many sweeps, one after the other
        return torch.cat([_exact_trafo(*p).t().reshape(-1) for p in st["p"]])
    if kind == "bt2":
        wide = torch.complex128 if st["q"].is_complex() else torch.float64
        q = st["q"].to(wide).contiguous()
        v, t, b = st["v"].to(wide).t().contiguous(), st["tau"].to(wide), st["nbw"]
        for c in range(case["n"] - b - 1, -1, -1):
            x = v[c, c + b:]
            y = x.conj().resolve_conj()[None, :] @ q[c + b:]
            q[c + b:].addmm_((x * t[c])[:, None], y, alpha=-1)
        return q
    a = st["a"].cpu().numpy()
    if kind == "gsolve":
        L = np.linalg.cholesky(st["b"].cpu().numpy())
        h = np.linalg.solve(L, np.linalg.solve(L, a).conj().T)
        a = (h + h.conj().T) / 2
    if case["n"] > 2500:
        return {"lam": torch.from_numpy(np.linalg.eigvalsh(a)), "z": None}
    lam, z = np.linalg.eigh(a)
    z = z[:, :case["nev"]]
    if kind == "gsolve":
        z = np.linalg.solve(L.conj().T, z)
    return {"lam": torch.from_numpy(lam), "z": _fix_sign(torch.from_numpy(z))}
