"""GPU full -> band reduction (include/elpa_f2b.h) against the oracle's
full_to_band, and the whole eigenvector chain with every stage but the
tridiagonal solve on the device."""
import numpy as np
import pytest

import workload as W
from oracle import checks, stage1, tridiag

from bt2_layout import panels_to_abi

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import time
    t0 = time.time()
    print("importing torch", flush=True)
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1811_01277_amd as P
    P.library()
    print(f"torch ready after {time.time() - t0:.1f} s", flush=True)
    return torch, torch.device("cuda:0")


def to_dev(torch, dev, a):
    return torch.from_numpy(np.ascontiguousarray(a.T)).to(dev).t()


CASES = [(97, 32, 501), (130, 64, 502), (300, 32, 503), (600, 64, 504), (50, 7, 505),
         (20, 19, 506), (65, 64, 507)]


@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("case", CASES, ids=[f"n{c[0]}_b{c[1]}" for c in CASES])
def test_f2b_matches_oracle(torch_dev, case, cplx):
    torch, dev = torch_dev
    import paper_1811_01277_amd as P
    n, b, seed = case
    A = W.herm_gaussian(n, seed) if cplx else W.sym_gaussian(n, seed)
    B0, panels = stage1.full_to_band(A, b)
    V0, t0 = panels_to_abi(panels, n, b, np.complex128 if cplx else np.float64)
    print(f"f2b n={n} b={b} cplx={cplx}", flush=True)
    a = to_dev(torch, dev, A)
    v, tau = P.full_to_band(a, b)
    torch.cuda.synchronize()
    B = a.cpu().numpy()
    scale = float(np.max(np.abs(A)))
    # band structure, Hermitian storage, and the spectrum kept
    far = np.abs(np.subtract.outer(np.arange(n), np.arange(n))) > b
    assert np.all(B[far] == 0)
    assert np.max(np.abs(B - B.conj().T)) <= 1e-13 * scale * n
    lam = np.linalg.eigvalsh(A)
    assert np.max(np.abs(np.linalg.eigvalsh(B) - lam)) <= 50 * n * np.finfo(float).eps * \
        np.linalg.norm(A, 2)
    # the oracle's band matrix and reflectors
    assert np.max(np.abs(B - B0)) <= 1e-11 * scale * n ** 0.5
    N = n - b
    Vg, tg = v.cpu().numpy(), tau.cpu().numpy()
    for c in range(N):
        ref = V0[c + b + 1:, c]
        assert np.max(np.abs(Vg[c + b + 1:, c] - ref), initial=0.0) <= 1e-9 * max(1.0, np.max(np.abs(ref), initial=0.0))
    assert np.max(np.abs(tg[:N] - t0[:N])) <= 1e-10


@pytest.mark.parametrize("cplx", [False, True])
def test_eigenvectors_all_stages_but_the_tridiagonal_solve_on_gpu(torch_dev, cplx):
    """full -> band, band -> tridiagonal, tridiagonal -> band and band -> full
    on the GPU (reflectors and band matrix never leave the device), the
    tridiagonal eigenpairs from the oracle: A Z = Z Lambda, Z^H Z = I."""
    torch, dev = torch_dev
    import paper_1811_01277_amd as P
    n, b = 500, 32
    A = W.herm_gaussian(n, 511) if cplx else W.sym_gaussian(n, 511)
    a = to_dev(torch, dev, A)
    v, tau_v = P.full_to_band(a, b)
    d, e, hh, tau_h = P.band_to_tridiag(a, b)
    lam, Zt = tridiag.eigh_tridiag(d.cpu().numpy(), e.cpu().numpy())
    dt = np.complex128 if cplx else np.float64
    q = to_dev(torch, dev, Zt.astype(dt))
    P.hh_trafo(q, hh, tau_h, b)
    P.bt2_trafo(q, v, tau_v, b)
    torch.cuda.synchronize()
    Z = q.cpu().numpy()
    assert checks.residual_ratio(A, Z, lam) < 50
    assert checks.orth_ratio(Z) < 50
    assert np.max(np.abs(lam - np.linalg.eigvalsh(A))) <= 50 * n * np.finfo(float).eps * \
        np.linalg.norm(A, 2)


def f2b_with_gather(torch, a, nbw, ticks):
    """elpa_full_to_band with the time the one-launch panel's workgroups have
    to come together (negative: one workgroup does every panel)."""
    import ctypes as C

    import paper_1811_01277_amd as P
    n = a.shape[0]
    N = n - nbw
    v = torch.zeros((N, n), dtype=a.dtype, device=a.device).t()
    tau = torch.zeros(N, dtype=a.dtype, device=a.device)
    fn = P.library().elpa_full_to_band_gather
    fn.argtypes = [C.c_int64, C.c_int64, C.c_void_p, C.c_int64, C.c_void_p, C.c_int64, C.c_void_p,
                   C.c_int32, C.c_void_p, C.c_int64]
    fn.restype = C.c_int
    rc = fn(n, nbw, a.data_ptr(), n, v.data_ptr(), n, tau.data_ptr(),
            P.C64 if a.is_complex() else P.R64, None, ticks)
    assert rc == 0, rc
    torch.cuda.synchronize()
    return v, tau


@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("alone", [False, True])
@pytest.mark.parametrize("n,b", [(256 + 64, 64), (256 + 65, 64), (33 + 129, 33), (700, 63),
                                 (545, 32), (300, 3), (200, 65)])
def test_f2b_panel_workgroups(torch_dev, n, b, alone, cplx):
    """Panels of one row more and less than whole workgroups, bands that do
    not fill the waves, and the first band too wide for the one-launch panel;
    done together and by one workgroup, against the oracle's panels."""
    torch, dev = torch_dev
    A = W.herm_gaussian(n, 530 + n) if cplx else W.sym_gaussian(n, 530 + n)
    B0, panels = stage1.full_to_band(A, b)
    V0, t0 = panels_to_abi(panels, n, b, np.complex128 if cplx else np.float64)
    print(f"f2b n={n} b={b} cplx={cplx} alone={alone}", flush=True)
    a = to_dev(torch, dev, A)
    v, tau = f2b_with_gather(torch, a, b, -1 if alone else 10 ** 7)
    B = a.cpu().numpy()
    scale = float(np.max(np.abs(A)))
    assert np.max(np.abs(B - B0)) <= 1e-11 * scale * n ** 0.5
    read = ~np.isnan(V0)  # the entries below the unit leads
    assert np.max(np.abs(v.cpu().numpy()[:, :n - b] - V0)[read], initial=0.0) <= 1e-10
    assert np.max(np.abs(tau.cpu().numpy() - t0)) <= 1e-10


@pytest.mark.parametrize("cplx", [False, True])
def test_f2b_given_up_wait_is_marked(torch_dev, cplx):
    """Waits between a panel's workgroups given up at the second look (a limit
    that the host sets): the call ends, and tau and the diagonal are NaN; the
    next call, with the usual limit, is whole."""
    import ctypes as C
    torch, dev = torch_dev
    import paper_1811_01277_amd as P
    n, b = 2500, 64
    fn = P.library().elpa_full_to_band_limits
    fn.argtypes = [C.c_int64, C.c_int64, C.c_void_p, C.c_int64, C.c_void_p, C.c_int64, C.c_void_p,
                   C.c_int32, C.c_void_p, C.c_int64, C.c_int64]
    g = torch.Generator(device=dev)
    g.manual_seed(540)
    x = torch.randn((n, n), generator=g, device=dev, dtype=torch.float64)
    if cplx:
        x = torch.complex(x, torch.randn((n, n), generator=g, device=dev, dtype=torch.float64))
    A = ((x + x.mH) / 2).t()
    for limit in (0, 10 ** 9):
        a = A.clone()
        v = torch.zeros((n - b, n), dtype=a.dtype, device=dev).t()
        tau = torch.zeros(n - b, dtype=a.dtype, device=dev)
        print(f"f2b wait limit {limit} cplx={cplx}", flush=True)
        rc = fn(n, b, a.data_ptr(), n, v.data_ptr(), n, tau.data_ptr(), P.C64 if cplx else P.R64,
                None, 10 ** 7, limit)
        torch.cuda.synchronize()
        assert rc == 0, rc
        bad = torch.isnan(tau.real), torch.isnan(a.diagonal().real)
        if limit == 0:
            assert bool(bad[0].all()) and bool(bad[1].all())
        else:
            assert not bool(bad[0].any()) and not bool(bad[1].any())


@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("n,b,crew", [(1200, 64, 1), (1200, 64, 3), (1200, 64, 0), (700, 31, 2),
                                      (530, 64, 2)])
def test_f2b_crew_equals_panel(torch_dev, n, b, crew, cplx):
    """Panels whose workgroups do not come together, by one, some and all of
    them: the same bits as together (fp64: 256 rows to a workgroup, complex
    128; the crew's sizes do not divide the panels' groups)."""
    import ctypes as C
    torch, dev = torch_dev
    import paper_1811_01277_amd as P
    fn = P.library().elpa_full_to_band_crew
    fn.argtypes = [C.c_int64, C.c_int64, C.c_void_p, C.c_int64, C.c_void_p, C.c_int64, C.c_void_p,
                   C.c_int32, C.c_void_p, C.c_int64, C.c_int64, C.c_int64]
    g = torch.Generator(device=dev)
    g.manual_seed(550 + n)
    x = torch.randn((n, n), generator=g, device=dev, dtype=torch.float64)
    if cplx:
        x = torch.complex(x, torch.randn((n, n), generator=g, device=dev, dtype=torch.float64))
    A = ((x + x.mH) / 2).t()
    out = []
    for ticks, c in ((10 ** 8, 0), (-1, crew)):
        a = A.clone()
        v = torch.zeros((n - b, n), dtype=a.dtype, device=dev).t()
        tau = torch.zeros(n - b, dtype=a.dtype, device=dev)
        print(f"f2b n={n} b={b} cplx={cplx} gather={ticks} crew={c}", flush=True)
        rc = fn(n, b, a.data_ptr(), n, v.data_ptr(), n, tau.data_ptr(), P.C64 if cplx else P.R64,
                None, ticks, 10 ** 9, c)
        torch.cuda.synchronize()
        assert rc == 0, rc
        out.append((a, v, tau))
    for y, z in zip(*out):
        assert torch.equal(y, z)
