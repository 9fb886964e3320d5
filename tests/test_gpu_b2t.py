"""GPU band -> tridiagonal reduction (include/elpa_b2t.h) against the oracle's
band_to_tridiag, and the reflectors it leaves in device memory used as they
are by the tridiagonal -> band back-transformation."""
import numpy as np
import pytest

import workload as W
from oracle import bt, checks, stage1, stage2, tridiag

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


def band_matrix(n, b, cplx, seed):
    """The first stage's band matrix of a Gaussian Hermitian matrix."""
    A = W.herm_gaussian(n, seed) if cplx else W.sym_gaussian(n, seed)
    B, _ = stage1.full_to_band(A, b)
    return B


def gpu_b2t(torch, dev, B, b):
    import paper_1811_01277_amd as P
    a = torch.from_numpy(np.ascontiguousarray(B.T)).to(dev).t()
    return P.band_to_tridiag(a, b)


def rel(x, ref):
    m = float(np.max(np.abs(ref))) if np.size(ref) else 0.0
    return float(np.max(np.abs(np.asarray(x) - ref))) / (m if m else 1.0) if np.size(ref) else 0.0


CASES = [(97, 32, 401), (130, 64, 402), (300, 32, 403), (40, 1, 404), (20, 19, 405),
         (2, 1, 406), (64, 5, 407)]


@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("case", CASES, ids=[f"n{c[0]}_b{c[1]}" for c in CASES])
def test_b2t_matches_oracle(torch_dev, case, cplx):
    torch, dev = torch_dev
    n, b, seed = case
    B = band_matrix(n, b, cplx, seed)
    d0, e0, hh0, tau0 = stage2.band_to_tridiag(B, b)
    print(f"b2t n={n} b={b} cplx={cplx}", flush=True)
    d, e, hh, tau = gpu_b2t(torch, dev, B, b)
    torch.cuda.synchronize()
    d, e, hh, tau = (x.cpu().numpy() for x in (d, e, hh, tau))
    scale = float(np.max(np.abs(B)))
    assert np.max(np.abs(d - d0)) <= 1e-12 * scale * max(1, n) ** 0.5
    assert np.max(np.abs(e - e0), initial=0.0) <= 1e-12 * scale * max(1, n) ** 0.5
    assert rel(hh, hh0) <= 1e-10 and rel(tau, tau0) <= 1e-10
    # same eigenvalues as the band matrix
    lam = np.linalg.eigvalsh(B)
    T = np.diag(d) + np.diag(e, -1) + np.diag(e, 1)
    assert np.max(np.abs(np.linalg.eigvalsh(T) - lam)) <= 1e-12 * scale * n


@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("nb", [64, 96])
def test_b2t_leaves_the_tridiagonal_matrix(torch_dev, cplx, nb):
    """On return A holds the tridiagonal matrix (d, e) in both triangles and
    zeros elsewhere (the real path with nbw <= 64 updates only the lower
    triangle during the chase and rebuilds the upper one at the end)."""
    torch, dev = torch_dev
    import paper_1811_01277_amd as P
    n = 260
    B = band_matrix(n, nb, cplx, 430)
    a = torch.from_numpy(np.ascontiguousarray(B.T)).to(dev).t()
    d, e, hh, tau = P.band_to_tridiag(a, nb)
    torch.cuda.synchronize()
    d, e, Ar = d.cpu().numpy(), e.cpu().numpy(), a.cpu().numpy()
    T = np.diag(d) + np.diag(e, -1) + np.diag(e, 1)
    assert np.max(np.abs(Ar - T)) <= 1e-12 * float(np.max(np.abs(B)))
    d0, e0, _, _ = stage2.band_to_tridiag(B, nb)
    assert np.max(np.abs(d - d0)) <= 1e-12 * float(np.max(np.abs(B))) * n ** 0.5


@pytest.mark.parametrize("cplx", [False, True])
def test_device_reflectors_drive_back_transform(torch_dev, cplx):
    """d, e from the GPU -> tridiagonal eigenvectors (oracle) -> elpa_hh_trafo
    with the GPU's hh / tau, never copied to the host: the band eigenvectors
    satisfy the residual and orthogonality invariants of B."""
    torch, dev = torch_dev
    import paper_1811_01277_amd as P
    n, b = 256, 32
    B = band_matrix(n, b, cplx, 411)
    d, e, hh, tau = gpu_b2t(torch, dev, B, b)
    lam, Zt = tridiag.eigh_tridiag(d.cpu().numpy(), e.cpu().numpy())
    dt = np.complex128 if cplx else np.float64
    q = torch.from_numpy(np.ascontiguousarray(Zt.astype(dt).T)).to(dev).t()
    P.hh_trafo(q, hh, tau, b)
    torch.cuda.synchronize()
    Zb = q.cpu().numpy()
    assert checks.residual_ratio(B, Zb, lam) < 50
    assert checks.orth_ratio(Zb) < 50
    # the oracle's chain from its own reflectors gives the same vectors
    d0, e0, hh0, tau0 = stage2.band_to_tridiag(B, b)
    ref = bt.bt_tridiag_to_band(hh0, tau0, Zt.astype(dt), n, b)
    assert checks.max_rel_err(Zb, ref) <= 1e-10


def test_whole_eigenvector_chain(torch_dev):
    """Full -> band (oracle), band -> tridiagonal (GPU), tridiagonal solve
    (oracle), tridiagonal -> band and band -> full (GPU): A Z = Z Lambda."""
    torch, dev = torch_dev
    import paper_1811_01277_amd as P
    n, b = 300, 32
    A = W.sym_gaussian(n, 421)
    B, panels = stage1.full_to_band(A, b)
    d, e, hh, tau = gpu_b2t(torch, dev, B, b)
    lam, Zt = tridiag.eigh_tridiag(d.cpu().numpy(), e.cpu().numpy())
    q = torch.from_numpy(np.ascontiguousarray(Zt.T)).to(dev).t()
    P.hh_trafo(q, hh, tau, b)
    V, t1 = panels_to_abi(panels, n, b, np.float64)
    v = torch.from_numpy(np.ascontiguousarray(V.T)).to(dev).t()
    P.bt2_trafo(q, v, torch.from_numpy(t1).to(dev), b)
    torch.cuda.synchronize()
    Z = q.cpu().numpy()
    assert checks.residual_ratio(A, Z, lam) < 50
    assert checks.orth_ratio(Z) < 50


def test_b2t_n2000(torch_dev):
    """n = 2000, nbw = 64 (about 32000 chase steps).  The tridiagonal matrix is
    a forward result whose entries drift from the oracle's as rounding
    differences accumulate over the steps (3e-10 relative here), so they get
    a loose bound; its eigenvalues, which a backward-stable reduction keeps,
    are held to eps-level against the band matrix's."""
    torch, dev = torch_dev
    n, b = 2000, 64
    G = np.random.default_rng(431).standard_normal((n, n))
    B = (G + G.T) / 2.0
    B[np.abs(np.subtract.outer(np.arange(n), np.arange(n))) > b] = 0.0
    d0, e0, hh0, tau0 = stage2.band_to_tridiag(B, b)
    d, e, hh, tau = gpu_b2t(torch, dev, B, b)
    torch.cuda.synchronize()
    d, e = d.cpu().numpy(), e.cpu().numpy()
    scale = float(np.max(np.abs(B)))
    lam = np.linalg.eigvalsh(B)
    lt = np.linalg.eigvalsh(np.diag(d) + np.diag(e, -1) + np.diag(e, 1))
    assert np.max(np.abs(lt - lam)) <= 50 * n * np.finfo(float).eps * np.linalg.norm(B, 2)
    assert np.max(np.abs(d - d0)) <= 1e-7 * scale and np.max(np.abs(e - e0)) <= 1e-7 * scale
    assert rel(hh.cpu().numpy(), hh0) <= 1e-6 and rel(tau.cpu().numpy(), tau0) <= 1e-6


@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("n,b", [(66, 33), (200, 48), (193, 64), (192, 64), (65, 64), (257, 31),
                                 (400, 2), (129, 16)])
def test_b2t_one_launch_sizes(torch_dev, n, b, cplx):
    """The one-launch chase at the edges of its blocks: bands that do not fill
    the four or eight waves, last steps of length 1 and of full length, more
    sweeps than workgroups, and one sweep only."""
    torch, dev = torch_dev
    B = band_matrix(n, b, cplx, 440 + n)
    d0, e0, hh0, tau0 = stage2.band_to_tridiag(B, b)
    print(f"b2t n={n} b={b} cplx={cplx}", flush=True)
    d, e, hh, tau = (x.cpu().numpy() for x in gpu_b2t(torch, dev, B, b))
    scale = float(np.max(np.abs(B)))
    assert np.max(np.abs(d - d0)) <= 1e-12 * scale * n ** 0.5
    assert np.max(np.abs(e - e0)) <= 1e-12 * scale * n ** 0.5
    assert rel(hh, hh0) <= 1e-10 and rel(tau, tau0) <= 1e-10


def b2t_with_gather(torch, dev, B, b, ticks):
    """elpa_band_to_tridiag with the time the resident form's workgroups have
    to come together (negative: the workgroups follow the sweeps)."""
    import ctypes as C

    import paper_1811_01277_amd as P
    n = B.shape[0]
    a = torch.from_numpy(np.ascontiguousarray(B.T)).to(dev).t()
    R = P.num_reflectors(n, b)
    d = torch.empty(n, dtype=torch.float64, device=dev)
    e = torch.empty(n - 1, dtype=torch.float64, device=dev)
    hh = torch.empty(R * b, dtype=a.dtype, device=dev)
    tau = torch.empty(R, dtype=a.dtype, device=dev)
    fn = P.library().elpa_band_to_tridiag_gather
    fn.argtypes = [C.c_int64, C.c_int64, C.c_void_p, C.c_int64, C.c_void_p, C.c_void_p,
                   C.c_void_p, C.c_void_p, C.c_int32, C.c_void_p, C.c_int64]
    fn.restype = C.c_int
    rc = fn(n, b, a.data_ptr(), n, d.data_ptr(), e.data_ptr(), hh.data_ptr(), tau.data_ptr(),
            P.C64 if a.is_complex() else P.R64, None, ticks)
    assert rc == 0, rc
    torch.cuda.synchronize()
    return [x.cpu().numpy() for x in (a, d, e, hh, tau)]


@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("n,b", [(2, 1), (3, 2), (30, 1), (66, 33), (65, 64), (66, 64), (129, 64),
                                 (130, 64), (200, 48), (193, 32), (257, 31), (90, 7)])
def test_b2t_resident_and_moving(torch_dev, n, b, cplx):
    """Workgroups that stay at their chase positions and workgroups that follow
    the sweeps: one position and many, last steps of length 1 and full, bands
    that do not fill the waves.  Same reflectors, and the matrix left behind
    holds the tridiagonal result and zeros."""
    torch, dev = torch_dev
    B = band_matrix(n, b, cplx, 480 + n)
    # B = Q T Q^H with Q the reflectors' product, to 50 n eps |B|: the entries
    # themselves can lose digits without bound (n = 65 with this seed: 5e-11)
    tol = 50 * n * np.finfo(float).eps * np.linalg.norm(B, 2)
    got = []
    for ticks in (10 ** 7, -1):
        print(f"b2t n={n} b={b} cplx={cplx} ticks={ticks}", flush=True)
        a, d, e, hh, tau = b2t_with_gather(torch, dev, B, b, ticks)
        got.append((d, e, hh, tau))
        T = np.diag(d) + np.diag(e, -1) + np.diag(e, 1)
        Q = bt.bt_tridiag_to_band(hh, tau, np.asfortranarray(np.eye(n, dtype=B.dtype)), n, b)
        assert np.max(np.abs(B @ Q - Q @ T)) <= tol
        assert np.max(np.abs(Q.conj().T @ Q - np.eye(n))) <= 50 * n * np.finfo(float).eps
        if cplx:   # the input's diagonal is real to rounding only
            assert np.max(np.abs(np.diag(a).imag)) <= tol
            np.fill_diagonal(a, np.diag(a).real)
        assert np.array_equal(a, T)
    # the sums run in the same order where the waves divide the band (complex
    # products may be contracted differently in the two kernels)
    if not cplx and b % (8 if b > 32 else 4) == 0:
        assert all(np.array_equal(x, y) for x, y in zip(*got))
