"""The one-launch pipelined schedules: path WY's workgroups of four waves, and
the fp64 calls of path SPLIT: the local form (a workgroup per stripe), the device form (one-wave workgroups over the
whole device) and the batched form with one, two, four and eight waves per
workgroup, against the diagonal launch schedule (bitwise: the same per-column
arithmetic) and the oracle."""
import numpy as np
import pytest

import workload as W
from oracle import bt, checks

pytestmark = pytest.mark.gpu

TOL = 1e-12


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1811_01277_amd as P
    P.library()
    return torch, torch.device("cuda:0")


def drawn(torch, dev, n, nbw, nev, seed):
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    hh, tau = W.device_reflectors(torch, n, nbw, dev, g)
    return W.device_block(torch, n, nev, dev, g), hh, tau


# few stripes and long chains take the device form, the others the local one;
# n around multiples of the block (k = 80 / 64) and of the band, ragged columns
@pytest.mark.parametrize("n,nbw,nev", [
    (2, 64, 1), (65, 64, 3), (81, 64, 16), (82, 64, 17), (145, 64, 33), (641, 64, 700),
    (1000, 64, 97), (33, 32, 5), (64, 32, 64), (65, 32, 31), (66, 32, 1), (449, 32, 449),
    (3000, 64, 40), (2500, 32, 17), (2999, 64, 1)])
def test_pipelined_call_equals_launch_schedule(torch_dev, n, nbw, nev):
    torch, dev = torch_dev
    import paper_1811_01277_amd as P
    q, hh, tau = drawn(torch, dev, n, nbw, nev, 7000 + n)
    ref = q.clone()
    print(f"pipelined n={n} nbw={nbw} nev={nev}", flush=True)
    P.hh_trafo(ref, hh, tau, nbw, path=P.PATH_SPLIT, steps=3)
    P.profile_enable(True)
    try:
        P.hh_trafo(q, hh, tau, nbw, path=P.PATH_SPLIT)
        pr = P.profile_last()
    finally:
        P.profile_enable(False)
    torch.cuda.synchronize()
    assert pr["launches"] == 1, pr
    assert torch.equal(q, ref)
    if n <= 700:
        z0 = drawn(torch, dev, n, nbw, nev, 7000 + n)[0].cpu().numpy()
        want = bt.bt_tridiag_to_band(hh.cpu().numpy(), tau.cpu().numpy(), np.asfortranarray(z0),
                                     n, nbw)
        assert checks.max_rel_err(q.cpu().numpy(), want) <= TOL


def test_padded_ldq_and_prepared_device_form(torch_dev):
    """A padded leading dimension (padding untouched), and the device form on a
    prepared call's own counts, run twice."""
    torch, dev = torch_dev
    import paper_1811_01277_amd as P
    n, nbw, nev, ldq = 2600, 64, 35, 2613
    z, hh, tau = drawn(torch, dev, n, nbw, nev, 7100)
    buf = torch.full((nev, ldq), 7.0, dtype=torch.float64, device=dev)
    buf[:, :n] = z.t()
    q = buf.t()[:n]
    ref = z.clone()
    for _ in range(2):
        P.hh_trafo(ref, hh, tau, nbw, path=P.PATH_SPLIT, steps=2)
    b = P.Batch([(q, hh, tau, nbw)])
    b.run()
    b.run()
    torch.cuda.synchronize()
    assert torch.equal(q, ref) and bool((buf[:, n:] == 7.0).all())
    b.close()


@pytest.mark.parametrize("count,n", [(3, 700), (20, 1000), (40, 900), (130, 780)])
def test_batched_waves_per_workgroup(torch_dev, count, n):
    """Batches whose stripes call for eight, four, two and one waves per
    workgroup."""
    torch, dev = torch_dev
    import paper_1811_01277_amd as P
    one = drawn(torch, dev, n, 32, n, 7200)
    probs = [(one[0].clone(), one[1], one[2], 32) for _ in range(count)]
    print(f"batched {count} x n={n}", flush=True)
    P.hh_trafo(one[0], one[1], one[2], 32, path=P.PATH_SPLIT, k=96, steps=4)
    P.hh_trafo_batched(probs, batch=P.BATCH_ONE_LAUNCH)
    torch.cuda.synchronize()
    for p in probs:
        assert torch.equal(p[0], one[0])


# path WY: ragged columns (units of 64, tiles of 16), n around blocks and bands,
# odd and even numbers of sub-groups
@pytest.mark.parametrize("dt,n,nbw,k,nev", [
    ("r32", 98, 64, 96, 1), ("r32", 700, 64, 96, 65), ("r32", 1601, 64, 160, 17),
    ("r32", 513, 32, 96, 130), ("c64", 66, 64, 48, 3), ("c64", 338, 64, 48, 81),
    ("c64", 400, 32, 32, 33), ("r64", 161, 64, 160, 64), ("r64", 1025, 64, 128, 63),
    ("r64", 640, 64, 112, 129), ("r64", 450, 32, 96, 48), ("r64", 3201, 64, 128, 1030)])
def test_wy_units_equal_launch_schedule(torch_dev, dt, n, nbw, k, nev):
    torch, dev = torch_dev
    import paper_1811_01277_amd as P
    q, hh, tau = drawn(torch, dev, n, nbw, nev, 7300 + n)
    if dt == "r32":
        q, hh, tau = q.t().float().t(), hh.float(), tau.float()
    elif dt == "c64":   # unitary: H = I - tau v v^H with real tau and |v| fixed
        ph = torch.polar(torch.ones_like(hh), torch.arange(hh.numel(), device=dev).reshape(
            hh.shape).to(torch.float64))
        hh, tau = hh * ph, tau.to(torch.complex128)
        q = torch.complex(q.t(), q.t().flip(0)).t()
    z = q.clone().cpu().numpy()
    ref = q.t().clone().t()
    print(f"wy units {dt} n={n} nbw={nbw} k={k} nev={nev}", flush=True)
    P.hh_trafo(ref, hh, tau, nbw, path=P.PATH_WY, k=k, steps=2)
    P.profile_enable(True)
    try:
        P.hh_trafo(q, hh, tau, nbw, path=P.PATH_WY, k=k)
        pr = P.profile_last()
    finally:
        P.profile_enable(False)
    torch.cuda.synchronize()
    assert pr["launches"] == 1, pr
    assert torch.equal(q, ref)
    if n <= 700:
        wide = np.complex128 if dt == "c64" else np.float64
        want = bt.bt_tridiag_to_band(hh.cpu().numpy().astype(wide), tau.cpu().numpy().astype(wide),
                                     np.asfortranarray(z.astype(wide)), n, nbw)
        assert checks.max_rel_err(q.cpu().numpy().astype(wide), want) <= (
            5e-5 if dt == "r32" else TOL)


@pytest.mark.parametrize("many", [False, True])
def test_complex_wy_leaves_large_calls_to_the_launch_schedule(torch_dev, many):
    """Complex calls of path WY run in one launch up to 28 units (64 columns of
    a sweep block) per compute unit; past that the diagonal launches, which are
    faster there."""
    torch, dev = torch_dev
    import paper_1811_01277_amd as P
    n, nbw, k = 6000, 64, 48
    blocks = -(-(n - 1) // k)
    cus = torch.cuda.get_device_properties(dev).multi_processor_count
    nev = 64 * (28 * cus // blocks) + (1 if many else 0)
    q, hh, tau = drawn(torch, dev, n, nbw, nev, 7400)
    hh, tau = hh.to(torch.complex128), tau.to(torch.complex128)
    q = q.t().to(torch.complex128).t()
    P.profile_enable(True)
    try:
        P.hh_trafo(q, hh, tau, nbw)
        pr = P.profile_last()
    finally:
        P.profile_enable(False)
    torch.cuda.synchronize()
    print(f"complex n={n} nev={nev}: {pr}", flush=True)
    assert (pr["path"], pr["k"]) == (P.PATH_WY, k)
    assert (pr["launches"] > 1) == many


def test_factors_in_several_launches(torch_dev):
    """Path SPLIT fp64 with more (block, step) groups than one factor launch
    takes (2^16), single (n = 19000) and batched (60 problems of n = 2000 on one
    set of reflectors): against path WY to the parity bar, and bitwise against
    the single launch schedule."""
    torch, dev = torch_dev
    import paper_1811_01277_amd as P
    n = 19000
    assert -(-(n - 1) // 80) * -(-(n - 1) // 64) > 1 << 16
    q, hh, tau = drawn(torch, dev, n, 64, 1, 7500)
    ref = q.clone()
    print(f"factors n={n}", flush=True)
    P.hh_trafo(ref, hh, tau, 64, path=P.PATH_WY, k=160)
    P.hh_trafo(q, hh, tau, 64, path=P.PATH_SPLIT)
    torch.cuda.synchronize()
    assert float((q - ref).abs().max() / ref.abs().max()) <= TOL
    del q, hh, tau, ref
    n, count = 2000, 60
    assert count * -(-(n - 1) // 96) * -(-(n - 1) // 32) > 1 << 16
    q, hh, tau = drawn(torch, dev, n, 32, 3, 7501)
    probs = [(q.t().clone().t(), hh, tau, 32) for _ in range(count)]
    print(f"factors {count} x n={n}", flush=True)
    P.hh_trafo(q, hh, tau, 32, path=P.PATH_SPLIT, k=96, steps=4)
    P.hh_trafo_batched(probs)
    torch.cuda.synchronize()
    for p in probs:
        assert torch.equal(p[0], q)


def test_one_launch_kernels_side_by_side(torch_dev):
    """Kernels whose workgroups wait for one another, two of them in flight on
    two streams at a time (panels, chase, WY and SPLIT units, the local form):
    every result has the bits it has alone, also where the workgroups of one do
    not find room beside the other."""
    torch, dev = torch_dev
    import paper_1811_01277_amd as P
    g = torch.Generator(device=dev)
    g.manual_seed(7600)
    x = torch.randn((1500, 1500), generator=g, device=dev, dtype=torch.float64)
    A = ((x + x.t()) / 2).t()
    B = A.clone()
    P.full_to_band(B, 64)
    sets = {(n, nbw, nev): drawn(torch, dev, n, nbw, nev, 7601 + n)
            for n, nbw, nev in [(3500, 64, 3500), (2600, 64, 700), (400, 32, 400)]}

    def f2b():
        a = A.clone()
        return (a, *P.full_to_band(a, 64))

    def b2t():
        b = B.clone()
        return (b, *P.band_to_tridiag(b, 64))

    def trafo(key, path):
        q, hh, tau = sets[key]
        q = q.t().clone().t()
        P.hh_trafo(q, hh, tau, key[1], path=path)
        return (q,)

    work = {"panels": f2b, "chase": b2t,
            "wy units": lambda: trafo((3500, 64, 3500), P.PATH_WY),
            "split units": lambda: trafo((2600, 64, 700), P.PATH_SPLIT),
            "split local": lambda: trafo((400, 32, 400), P.PATH_SPLIT)}
    alone = {}
    for k, f in work.items():
        alone[k] = f()
        torch.cuda.synchronize()
    s1, s2 = torch.cuda.Stream(dev), torch.cuda.Stream(dev)
    names = list(work)
    for i, a in enumerate(names):
        for b in names[i:]:
            print(f"side by side: {a}, {b}", flush=True)
            got = []
            for _ in range(2):
                with torch.cuda.stream(s1):
                    got.append((a, work[a]()))
                with torch.cuda.stream(s2):
                    got.append((b, work[b]()))
            torch.cuda.synchronize()
            for k, out in got:
                assert all(torch.equal(y, z) for y, z in zip(out, alone[k])), (a, b, k)
