#!/usr/bin/env python3
"""Benchmark of the tridiagonal->band eigenvector back-transformation on one
MI355X.

One step = one elpa_hh_trafo call over the whole workload: every
band->tridiagonal reflector of an n x n problem applied to all nev columns of
Q (inputs resident in HBM).  Default workload: real fp64, n = 20000,
nbw = 64, nev = 20000 (all eigenvectors).  Counted flops per step:
2 n (n-1) nev (real), 8 n (n-1) nev (complex, real flops).

Prints ONE JSON line (rank 0) with the metric, a roofline object for the
kernel (measured live with HIP events on the launch stream) and the CPU oracle
timed on a bounded sample of the same workload.
"""
import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "hh_trafo GFLOP/s & % FP64 MFMA peak at n=20000; solves/sec + p99 latency"
PEAK_TFLOPS = {"r64": 78.6, "c64": 78.6, "r32": 157.3}


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--n", type=int, default=20000)
    ap.add_argument("--nbw", type=int, default=64)
    ap.add_argument("--nev", type=int, default=20000)
    ap.add_argument("--dtype", default="r64", choices=["r64", "r32", "c64"])
    ap.add_argument("--path", type=int, default=0,
                    help="0 auto, 1 reference, 2 one-lane stripe, 3 split (fp64: compact WY with "
                         "the reflectors in place, else two-lane stripe), 4 compact WY")
    ap.add_argument("--k", type=int, default=0, help="sweeps fused per pass (0 = auto)")
    ap.add_argument("--tile-steps", type=int, default=0,
                    help="chase steps per tile of the launch schedule (0 = auto)")
    ap.add_argument("--order", type=int, default=0,
                    help="tile order over workgroup ids: 0 auto, 1 linear, 2 per-XCD runs")
    ap.add_argument("--streams", type=int, default=0,
                    help="stripe groups on concurrent streams (0 = auto)")
    ap.add_argument("--seed", type=int, default=301)
    ap.add_argument("--cpu-seconds", type=float, default=15.0,
                    help="target CPU time of the oracle baseline sample")
    ap.add_argument("--no-cpu", action="store_true", help="skip the CPU baseline leg")
    ap.add_argument("--no-configs", action="store_true",
                    help="skip the table of every stated configuration")
    ap.add_argument("--no-served", action="store_true", help="skip the served SCF stream leg")
    ap.add_argument("--no-batched", action="store_true", help="skip the batched workload leg")
    ap.add_argument("--no-bt2", action="store_true",
                    help="skip the band->full back-transformation leg")
    ap.add_argument("--no-b2t", action="store_true",
                    help="skip the band->tridiagonal reduction leg")
    ap.add_argument("--no-f2b", action="store_true",
                    help="skip the full->band reduction leg")
    ap.add_argument("--no-solve", action="store_true",
                    help="skip the whole-solve leg (every stage of the eigensolver on the device)")
    ap.add_argument("--no-gen", action="store_true",
                    help="skip the generalized-problem leg")
    ap.add_argument("--solve-only", action="store_true",
                    help="instead of the benchmark: only the whole-solve leg (for profiling it on "
                         "its own)")
    ap.add_argument("--bt2-only", action="store_true",
                    help="instead of the benchmark: only the band->full leg at --nev "
                         "(for profiling it on its own)")
    ap.add_argument("--batched-only", action="store_true",
                    help="instead of the benchmark: only the batched workload leg (for profiling "
                         "it on its own)")
    ap.add_argument("--served-rates", default="",
                    help="Poisson arrival rates of the served stream (requests / s; default "
                         "0.8x and 1.25x the plain path's measured capacity)")
    ap.add_argument("--batch-flops", type=float, default=5e10,
                    help="served stream: work bound of a batch (counted flops)")
    ap.add_argument("--call-streams", type=int, default=1,
                    help="served stream: stripe-group streams per call (0: library choice)")
    ap.add_argument("--served-only", action="store_true",
                    help="instead of the benchmark: only the served stream leg")
    ap.add_argument("--peak-probe", action="store_true",
                    help="instead of the benchmark: measured fp64 / fp32 FMA and MFMA issue rates "
                         "(elpa_peak_probe) at 1, 2 and 4 waves per SIMD")
    ap.add_argument("--copy-calibration", type=int, default=0, metavar="MIB",
                    help="instead of the benchmark: copy a MIB-MiB device buffer 3 times "
                         "(reference kernel of known size for the HBM byte counters)")
    return ap.parse_args()


def served_stream(args):
    """The served SCF stream: 64 sequences x 20 solves, n_q ~ U{1000..6000},
    nbw 64, nev = n, Poisson arrivals.  Each sequence keeps its Q, reflectors
    and tau (fp64 and fp32) resident; they are drawn on the device
    (workload.device_*; the upstream stages that would produce them are not
    timed).

    * capacity: the plain one-call-at-a-time path with every request ready at
      once (solves/s);
    * the mixed trace (each request fp32 with probability 0.25) served with
      continuous batching and by the plain path at 0.8x and 1.25x that
      capacity (or at args.served_rates if given);
    * precision switching (the paper's single precision for the first SCF
      steps, double for the rest): fp32 for the first 5 of each sequence's 20
      steps, then fp64, against the same arrivals all in fp64, both served
      and plain, at 0.8x capacity (and served at 1.25x, where the switch
      shows in throughput); a sample of sequences' fp64 buffers are
      checked against the oracle after the served run, and one fresh fp32
      request per sampled sequence is compared with the fp64 oracle."""
    import torch
    import workload as W
    from concurrent.futures import ThreadPoolExecutor
    from oracle import bt, checks
    from paper_1811_01277_amd.serve import Request, Server, latency_stats, run_plain
    import paper_1811_01277_amd as P
    dev = torch.device("cuda:0")
    nseq, steps, switch = 64, 20, 5
    bf, cs = args.batch_flops, args.call_streams
    sizes = W.scf_sequence_sizes(nseq, 1000, 6000, seed=501)
    g = torch.Generator(device=dev)
    g.manual_seed(510000)
    state = []
    for q in range(nseq):
        n = int(sizes[q])
        hh, tau = W.device_reflectors(torch, n, 64, dev, g)
        Z = W.device_block(torch, n, n, dev, g)           # column major
        state.append({"r64": (Z, hh, tau), "r32": (Z.t().float().t(), hh.float(), tau.float())})
    torch.cuda.synchronize()

    def requests(rate, switch_step=None, p32=0.25):
        t, sq, st, f32 = W.scf_trace(nseq, steps, rate=rate, p32=p32, switch_step=switch_step)
        out, last = [], {}
        for i in range(len(t)):
            q = int(sq[i])
            Z, hh, tau = state[q]["r32" if f32[i] else "r64"]
            out.append(Request(rid=i, q=Z, hh=hh, tau=tau, nbw=64, arrival=float(t[i]),
                               after=last.get(q, -1), seq=q, step=int(st[i])))
            last[q] = i
        return out

    warm = requests(1000.0)[:nseq]    # one solve per sequence, untimed
    for r in warm:
        r.arrival, r.after = 0.0, -1
    Server(dev, slots=3, max_batch=32, batch_flops=bf, call_streams=cs).run(warm)
    cap = latency_stats(run_plain(requests(1e9), dev))["solves_per_s"]
    if args.served_rates:
        rates = [float(x) for x in args.served_rates.split(",") if x]
    else:
        rates = [round(0.8 * cap, 1), round(1.25 * cap, 1)]
    # per-sequence graphs of prepared batches (setup, not timed)
    gsrv = Server(dev, slots=3, max_batch=32, batch_flops=bf, call_streams=cs)
    t0 = time.perf_counter()
    gbytes = gsrv.prepare_graphs(requests(1e9))
    gsetup = time.perf_counter() - t0
    runs = []
    for rate in rates:
        srv = Server(dev, slots=3, max_batch=32, batch_flops=bf, call_streams=cs)
        served = latency_stats(srv.run(requests(rate)))
        gsrv.batches, gsrv.replays, gsrv.launch_s = [], 0, 0.0
        with_graphs = latency_stats(gsrv.run(requests(rate)))
        plain = latency_stats(run_plain(requests(rate), dev))
        runs.append({"rate_per_s": rate, "rate_vs_plain_capacity": round(rate / cap, 3),
                     "served": served, "served_graphs": with_graphs, "plain": plain,
                     "solves_per_s_vs_plain": round(served["solves_per_s"] /
                                                    plain["solves_per_s"], 3),
                     "p99_vs_plain": round(served["p99_ms"] / plain["p99_ms"], 3),
                     "graphs_solves_per_s_vs_plain": round(with_graphs["solves_per_s"] /
                                                           plain["solves_per_s"], 3),
                     "graphs_p99_vs_plain": round(with_graphs["p99_ms"] / plain["p99_ms"], 3),
                     "batches": len(srv.batches), "graph_replays": gsrv.replays,
                     "host_launch_s": round(srv.launch_s, 3),
                     "graphs_host_launch_s": round(gsrv.launch_s, 3)})
    gsrv.close_graphs()
    # precision switching at 0.8x capacity; sampled sequences' fp64 buffers
    # checked against the oracle after the served run (each holds its input
    # with one reflector application per fp64 request of the trace)
    rate = round(0.8 * cap, 1)
    sample = sorted({int(np.argmin(sizes)), int(np.argmax(sizes)), 7, 33})
    cols = [0, 1]
    before = {q: state[q]["r64"][0][:, cols].cpu().numpy() for q in sample}
    sw_reqs = requests(rate, switch_step=switch)
    Server(dev, slots=3, max_batch=32, batch_flops=bf, call_streams=cs).run(sw_reqs)
    sw_served = latency_stats(sw_reqs)
    after = {q: state[q]["r64"][0][:, cols].cpu().numpy() for q in sample}
    n64 = {q: sum(1 for r in sw_reqs if r.seq == q and r.q.dtype == torch.float64)
           for q in sample}
    sw_plain = latency_stats(run_plain(requests(rate, switch_step=switch), dev))
    all64_served = latency_stats(Server(dev, slots=3, max_batch=32, batch_flops=bf, call_streams=cs).run(
        requests(rate, switch_step=0)))
    all64_plain = latency_stats(run_plain(requests(rate, switch_step=0), dev))
    # above capacity the switch shows in throughput: fp32 steps finish sooner
    hi = round(1.25 * cap, 1)
    sw_hi = latency_stats(Server(dev, slots=3, max_batch=32, batch_flops=bf, call_streams=cs).run(
        requests(hi, switch_step=switch)))
    all64_hi = latency_stats(Server(dev, slots=3, max_batch=32, batch_flops=bf, call_streams=cs).run(
        requests(hi, switch_step=0)))
    host = {q: (state[q]["r64"][1].cpu().numpy(), state[q]["r64"][2].cpu().numpy())
            for q in sample}

    def replay(q):
        n = int(sizes[q])
        z = before[q]
        for _ in range(n64[q]):
            z = bt.bt_tridiag_to_band(host[q][0], host[q][1], z, n, 64, nthreads=1)
        return q, checks.max_rel_err(after[q], z)

    # fp32 error per request: one fresh fp32 request per sampled sequence
    g2 = torch.Generator(device=dev)
    g2.manual_seed(520000)
    f32_err = {}
    f32_in = {}
    for q in sample:
        n = int(sizes[q])
        hh, tau = W.device_reflectors(torch, n, 64, dev, g2)
        Z = W.device_block(torch, n, 4, dev, g2)          # column major, fp64
        q32 = Z.t().float().t()                            # the fp32 request's Q
        P.hh_trafo(q32, hh.float(), tau.float(), 64)
        torch.cuda.synchronize()
        f32_in[q] = (hh.cpu().numpy(), tau.cpu().numpy(), np.asfortranarray(Z.cpu().numpy()),
                     q32.cpu().numpy().astype(np.float64))
    with ThreadPoolExecutor(max_workers=host_threads()) as ex:
        rep = dict(ex.map(replay, sample))
        futs = {q: ex.submit(bt.bt_tridiag_to_band, v[0], v[1], v[2], int(sizes[q]), 64, 1)
                for q, v in f32_in.items()}
        for q, f in futs.items():
            f32_err[q] = checks.max_rel_err(f32_in[q][3], f.result())
    return {"workload": f"{nseq} sequences x {steps} solves, n ~ U{{1000..6000}}, nbw 64, "
                        f"nev = n, Poisson arrivals; slots 3, max batch 32, "
                        f"batch work bound {bf:.3g} flops, {cs or 'library'} stream(s) per call",
            "plain_capacity_solves_per_s": cap,
            "graphs": {"prepared_batches": 2 * nseq, "device_bytes": gbytes,
                       "setup_s": round(gsetup, 2)},
            "runs": runs,
            "precision_switching": {
                "trace": f"fp32 for steps 0..{switch - 1} of each sequence, fp64 after; "
                         f"{rate} requests/s (0.8x plain capacity)",
                "served": sw_served, "plain": sw_plain,
                "all_fp64_same_arrivals": {"served": all64_served, "plain": all64_plain},
                "solves_per_s_switch_vs_all_fp64_served":
                    round(sw_served["solves_per_s"] / all64_served["solves_per_s"], 3),
                "above_capacity": {"rate_per_s": hi, "served_switch": sw_hi,
                                   "served_all_fp64": all64_hi,
                                   "solves_per_s_switch_vs_all_fp64":
                                       round(sw_hi["solves_per_s"] / all64_hi["solves_per_s"], 3)},
                "fp64_buffers_vs_oracle": {
                    str(q): {"n": int(sizes[q]), "fp64_applications": n64[q],
                             "max_rel_err": float(f"{rep[q]:.3e}")} for q in sample},
                "fp32_request_err_vs_fp64_oracle": {
                    str(q): {"n": int(sizes[q]), "max_rel_err": float(f"{f32_err[q]:.3e}")}
                    for q in sample}}}


def batched_workload(quick=False, order=0, k=0):
    """The batched workload: 256 real fp64 problems, n_i ~ U{200..2000}
    (seed 401), nbw 32, nev = n_i, all back-transforms in one batched call
    (inputs drawn on the device).  Timed with the library's default plan, then
    with the uniform plan the batch tuner picks (kernel family, k, tile height,
    stripe groups) over the whole batch; for comparison, with plans tuned one
    problem at a time per size class of n, and one call per problem."""
    import torch
    import workload as W
    import paper_1811_01277_amd as P
    dev = torch.device("cuda:0")
    sizes = [int(x) for x in W.batched_sizes(256, 200, 2000, seed=401)]
    g = torch.Generator(device=dev)
    g.manual_seed(401000)
    probs = []
    for n in sizes:
        hh, tau = W.device_reflectors(torch, n, 32, dev, g)
        probs.append((W.device_block(torch, n, n, dev, g), hh, tau, 32))
    flops = sum(2 * n * (n - 1) * n for n in sizes)

    def timed(fn, reps=3):
        fn()
        torch.cuda.synchronize()
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        ev[0].record()
        for _ in range(reps):
            fn()
        ev[1].record()
        torch.cuda.synchronize()
        return ev[0].elapsed_time(ev[1]) / reps

    P.tuner_clear()
    P.profile_enable(True)
    t_default = timed(lambda: P.hh_trafo_batched(probs, order=order if quick else 0,
                                                 k=k if quick else 0))
    pr = P.profile_last()
    P.profile_enable(False)
    if quick:
        return {"workload": "256 real fp64 problems, n ~ U{200..2000}, nbw 32, nev = n, one call",
                "gflops_default": round(flops / t_default / 1e6, 1),
                "ms_default": round(t_default, 3), "launches": pr["launches"],
                "kernel_ms": round(pr["kernel_ms"], 3)}
    t_single = timed(lambda: [P.hh_trafo(q, h, t, nbw) for (q, h, t, nbw) in probs], reps=1)
    # the one launch with the stripes in plain problem order (no die grouping)
    t_linear = timed(lambda: P.hh_trafo_batched(probs, order=P.ORDER_LINEAR))
    # one uniform plan timed over the whole batch
    t0 = time.perf_counter()
    plan = P.tune_batched(probs, level=1)
    tune_s = time.perf_counter() - t0
    t_tuned = timed(lambda: P.hh_trafo_batched(probs, **plan))
    # for contrast: plans tuned one problem at a time, per size class of n
    classes = {}
    for i, n in enumerate(sizes):
        classes.setdefault(int(np.floor(4 * np.log2(n) + 1e-9)), i)
    for i in classes.values():
        q, h, t, nbw = probs[i]
        P.tune(q, h, t, nbw, level=1)
    t_class = timed(lambda: P.hh_trafo_batched(probs))
    P.tuner_clear()
    return {"workload": "256 real fp64 problems, n ~ U{200..2000}, nbw 32, nev = n, one call",
            "gflops_default": round(flops / t_default / 1e6, 1),
            "ms_default": round(t_default, 3), "launches_default": pr["launches"],
            "kernel_ms_default": round(pr["kernel_ms"], 3),
            "ms_linear_order": round(t_linear, 3),
            "gflops_tuned": round(flops / t_tuned / 1e6, 1), "ms_tuned": round(t_tuned, 3),
            "tuned_plan": plan, "tuning_s": round(tune_s, 1),
            "gflops_per_class_single_call_plans": round(flops / t_class / 1e6, 1),
            "gflops_one_call_per_problem": round(flops / t_single / 1e6, 1)}


# The stated back-transformation configurations: (label, n, nbw, nev, dtype).
# Reflectors and eigenvector blocks are drawn on the device with the seeded
# generators of workload (synthetic reflectors with the bulge chase's slot
# structure stand in for the oracle's reduction of the stated matrices).
CONFIGS = [("C1", 512, 32, 512, "r64")] + \
    [("C2", 8192, 64, e, "r64") for e in (819, 4096, 8192)] + \
    [("C3", 20000, 64, e, dt) for dt in ("r64", "r32", "c64") for e in (2000, 10000, 20000)]


def configs_leg(args):
    """Every stated configuration timed in the library's default plan: ms per
    call (median of the timed calls, HIP events on the launch stream, after
    one untimed call), counted TFLOP/s, the fraction of the dtype's peak, and
    the max-abs relative error of one call against the fp64 oracle on sampled
    columns (fp32: the error of the fp32 path against the oracle of the
    unrounded fp64 inputs, and against the oracle of the rounded inputs, the
    5e-5 parity bar).  The oracle runs per column in a thread pool while the
    GPU times the next configurations."""
    import torch
    import workload as W
    import paper_1811_01277_amd as P
    from concurrent.futures import ThreadPoolExecutor
    from oracle import bt, checks
    dev = torch.device("cuda:0")
    pool = ThreadPoolExecutor(max_workers=host_threads())
    rows, pending = [], []
    groups = {}
    for c in CONFIGS:
        groups.setdefault((c[1], c[2], c[4]), []).append(c)
    for gi, ((n, nbw, dt), cfgs) in enumerate(groups.items()):
        cplx = dt == "c64"
        wide = np.complex128 if cplx else np.float64
        g = torch.Generator(device=dev)
        g.manual_seed(args.seed + 1000 + gi)
        hh64, tau64 = W.device_reflectors(torch, n, nbw, dev, g, complex_=cplx)
        Z64 = W.device_block(torch, n, max(c[3] for c in cfgs), dev, g, complex_=cplx)
        hh_h, tau_h = hh64.cpu().numpy(), tau64.cpu().numpy()
        if dt == "r32":
            hh, tau = hh64.float(), tau64.float()
            hh_r = hh.cpu().numpy().astype(np.float64)
            tau_r = tau.cpu().numpy().astype(np.float64)
            del hh64, tau64
        else:
            hh, tau = hh64, tau64
        for (label, _, _, nev, _) in cfgs:
            print(f"config {label} n={n} nbw={nbw} nev={nev} {dt}", file=sys.stderr, flush=True)
            Zs = Z64[:, :nev]
            src = Zs.t().float().t() if dt == "r32" else Zs
            q = src.t().clone().t()
            cols = sorted({0, 31, 32, nev // 2, nev - 1})
            Zc = Zs[:, cols].cpu().numpy()
            stream = torch.cuda.current_stream(dev)
            P.hh_trafo(q, hh, tau, nbw, stream=stream)
            got = q[:, cols].cpu().numpy().astype(wide)
            reps = 20 if n * n * nev <= 8192 ** 3 else 3
            ev = [torch.cuda.Event(enable_timing=True) for _ in range(2 * reps)]
            for i in range(reps):
                ev[2 * i].record(stream)
                P.hh_trafo(q, hh, tau, nbw, stream=stream)
                ev[2 * i + 1].record(stream)
            torch.cuda.synchronize()
            ms = float(np.median([ev[2 * i].elapsed_time(ev[2 * i + 1]) for i in range(reps)]))
            fl = counted_flops(n, nev, dt)
            tf = fl / (ms * 1e-3) / 1e12
            row = {"config": label, "n": n, "nbw": nbw, "nev": nev, "dtype": dt,
                   "ms": round(ms, 3), "tflops": round(tf, 2),
                   "frac_peak": round(tf / PEAK_TFLOPS[dt], 4), "peak_tflops": PEAK_TFLOPS[dt],
                   "calls_timed": reps, "sampled_columns": len(cols)}
            if dt == "r32":
                row["frac_fp64_peak"] = round(tf / PEAK_TFLOPS["r64"], 4)
            rows.append(row)

            def one(hh_, tau_, z, c):
                return bt.bt_tridiag_to_band(hh_, tau_, z[:, c:c + 1], n, nbw, nthreads=1)

            def err_of(futs, got_):
                ref = np.concatenate([f.result() for f in futs], axis=1)
                return float(f"{checks.max_rel_err(got_, ref):.3e}")

            f64 = [pool.submit(one, hh_h, tau_h, Zc, i) for i in range(len(cols))]
            pending.append((row, "max_rel_err_vs_fp64_oracle", f64, got))
            if dt == "r32":
                Zr = Zc.astype(np.float32).astype(np.float64)
                f32 = [pool.submit(one, hh_r, tau_r, Zr, i) for i in range(len(cols))]
                pending.append((row, "max_rel_err_vs_oracle_rounded_inputs", f32, got))
            del q, src, Zs
        del hh, tau, Z64
        torch.cuda.empty_cache()
    for row, key, futs, got in pending:
        row[key] = err_of(futs, got)
    pool.shutdown()
    for row in rows:
        tol = 5e-5 if row["dtype"] == "r32" else 1e-12
        key = "max_rel_err_vs_oracle_rounded_inputs" if row["dtype"] == "r32" else \
            "max_rel_err_vs_fp64_oracle"
        row["within_parity_bar"] = bool(row[key] <= tol)
    return {"measure": "default plan; ms = median HIP-event time per call on the launch stream; "
                       "tflops = counted flops (2 n (n-1) nev real, 8 n (n-1) nev complex) / ms; "
                       "errors: max |gpu - oracle| / max |oracle| on sampled columns of one call",
            "rows": rows}


def bt2_leg(args, nevs=None):
    """Band -> full back-transformation (elpa_bt2_trafo) on the same n and
    nev: synthetic first-stage reflectors (workload.synthetic_stage1, nbw 64),
    real fp64, the library's default block; counted flops 2 nev N (N+1) with
    N = n - nbw (4 (n - c - nbw) nev per reflector c).  The products run on the
    fp64 matrix cores, so the roofline is the 78.6 TFLOP/s MFMA peak."""
    import torch
    import workload as W
    import paper_1811_01277_amd as P
    dev = torch.device("cuda:0")
    n, nbw = args.n, 64
    out = {"workload": f"band->full back-transform, n={n}, nbw={nbw}, r64, synthetic "
                       f"first-stage reflectors", "runs": []}
    V, tau = W.synthetic_stage1(n, nbw, seed=args.seed + 7)
    v = torch.from_numpy(np.ascontiguousarray(V.T)).to(dev).t()
    t = torch.from_numpy(tau).to(dev)
    del V
    N = n - nbw
    for nev in nevs or sorted({args.nev, min(args.nev, 2000)}, reverse=True):
        g = torch.Generator(device=dev)
        g.manual_seed(args.seed + 8)
        q = torch.randn(nev, n, device=dev, dtype=torch.float64, generator=g).t()
        P.bt2_trafo(q, v, t, nbw)
        torch.cuda.synchronize()
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        reps = 2
        ev[0].record()
        for _ in range(reps):
            P.bt2_trafo(q, v, t, nbw)
        ev[1].record()
        torch.cuda.synchronize()
        ms = ev[0].elapsed_time(ev[1]) / reps
        fl = 2.0 * nev * N * (N + 1)
        out["runs"].append({"nev": nev, "ms": round(ms, 3), "gflops": round(fl / ms / 1e6, 1),
                            "frac_fp64_mfma_peak": round(fl / ms / 1e9 / 78.6, 4)})
        del q
        torch.cuda.empty_cache()
    return out


def b2t_leg(args):
    """Band -> tridiagonal reduction (elpa_band_to_tridiag) on a random
    symmetric band matrix of the same n, nbw 64, real fp64, drawn on the
    device.  One launch for bands this wide; bound by the latency of a sweep's
    hand-overs, so the figures are time, chase steps per second and time per
    sweep."""
    import torch
    import paper_1811_01277_amd as P
    dev = torch.device("cuda:0")
    n, b = args.n, 64
    g = torch.Generator(device=dev)
    g.manual_seed(args.seed + 9)
    G = torch.randn(n, n, device=dev, dtype=torch.float64, generator=g)
    B = (G + G.t()) * 0.5
    del G
    i = torch.arange(n, device=dev)
    B.masked_fill_((i[:, None] - i[None, :]).abs() > b, 0.0)
    steps = P.num_reflectors(n, b)
    times = []
    for _ in range(2):
        a = B.clone().t()   # symmetric: the column-major view holds the same matrix
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        P.band_to_tridiag(a, b)
        torch.cuda.synchronize()
        times.append(time.perf_counter() - t0)
        del a
    del B
    torch.cuda.empty_cache()
    t = min(times)
    return {"workload": f"band->tridiagonal reduction, n={n}, nbw={b}, r64, random band "
                        f"matrix", "s": round(t, 3), "chase_steps": steps,
            "steps_per_s": round(steps / t), "sweeps": n - 1,
            "us_per_sweep": round(t / (n - 1) * 1e6, 2)}


def f2b_leg(args):
    """Full -> band reduction (elpa_full_to_band) of a random symmetric matrix
    of the same n, nbw 64, real fp64, drawn on the device.  Counted flops
    4 n^3 / 3, the usual count of a symmetric two-sided reduction; executed
    about 2 n^3 (A22 V and one rank-2k product over both triangles per
    panel)."""
    import torch
    import paper_1811_01277_amd as P
    dev = torch.device("cuda:0")
    n, b = args.n, 64
    g = torch.Generator(device=dev)
    g.manual_seed(args.seed + 11)
    G = torch.randn(n, n, device=dev, dtype=torch.float64, generator=g)
    A = (G + G.t()) * 0.5
    del G
    times = []
    for _ in range(2):
        a = A.clone().t()   # symmetric: the column-major view holds the same matrix
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        v, tau = P.full_to_band(a, b)
        torch.cuda.synchronize()
        times.append(time.perf_counter() - t0)
        del a, v, tau
    del A
    torch.cuda.empty_cache()
    t = min(times)
    return {"workload": f"full->band reduction, n={n}, nbw={b}, r64, random symmetric "
                        f"matrix", "s": round(t, 3),
            "tflops_4n3_3": round(4.0 * n ** 3 / 3 / t / 1e12, 2),
            "tflops_executed_2n3": round(2.0 * n ** 3 / t / 1e12, 2)}


def solve_leg(args):
    """The whole standard eigensolver on the device for a random symmetric
    matrix of the same n, nbw 64, real fp64, the eigenvectors of the nev
    smallest eigenvalues: full -> band, band -> tridiagonal, tridiagonal
    divide and conquer, tridiagonal -> band, band -> full.  Stage times with
    a synchronisation after each, and the residual ratio
    ||A z - lambda z||_1 / (||A||_1 n eps) on sampled columns."""
    import torch
    import paper_1811_01277_amd as P
    dev = torch.device("cuda:0")
    n, b, nev = args.n, 64, args.nev
    g = torch.Generator(device=dev)
    g.manual_seed(args.seed + 13)
    A = torch.randn(n, n, device=dev, dtype=torch.float64, generator=g)
    A = (A + A.t()) * 0.5
    a = A.clone().t()
    marks = []

    def mark():
        torch.cuda.synchronize()
        marks.append(time.perf_counter())

    mark()
    v, t1 = P.full_to_band(a, b)
    mark()
    d, e, hh, tau = P.band_to_tridiag(a, b)
    mark()
    lam, q = P.tridiag_eigh(d, e, nev)
    mark()
    P.hh_trafo(q, hh, tau, b)
    mark()
    P.bt2_trafo(q, v, t1, b)
    mark()
    idx = torch.tensor([0, nev // 2, nev - 1], device=dev)
    Z = q[:, idx]
    R = A @ Z - Z * lam[idx]
    eps = 2.0 ** -52
    res = float(R.abs().sum(0).max()) / (float(A.abs().sum(0).max()) * n * eps)
    del A, a, v, t1, d, e, hh, tau, lam, q, Z, R
    torch.cuda.empty_cache()
    st = [marks[i + 1] - marks[i] for i in range(5)]
    return {"workload": f"standard eigensolver on the device, n={n}, nbw={b}, nev={nev}, r64, "
                        f"random symmetric matrix",
            "s": round(marks[-1] - marks[0], 3),
            "stages_s": {"full_to_band": round(st[0], 3), "band_to_tridiag": round(st[1], 3),
                         "tridiag_eigh": round(st[2], 3), "hh_trafo": round(st[3], 3),
                         "bt2_trafo": round(st[4], 3)},
            "residual_ratio_sampled": round(res, 4)}


def gen_leg(args):
    """The generalized problem's own steps at the same n, real fp64: the
    inverted Cholesky factor of a random symmetric positive definite B
    (n^3/3 + n^3/3 flops: factorisation and triangular inverse), the forward
    transformation Linv A Linv^H (2 n^3: two triangular products) and the
    back-transformation Linv^H Q for nev columns (n^2 nev)."""
    import torch
    import paper_1811_01277_amd as P
    dev = torch.device("cuda:0")
    n, nev = args.n, args.nev
    g = torch.Generator(device=dev)
    g.manual_seed(args.seed + 17)
    X = torch.randn(n, n, device=dev, dtype=torch.float64, generator=g)
    B = X @ X.t() / n
    B.diagonal().add_(1.0)
    A = (X + X.t()) * 0.5
    del X
    q = torch.randn(nev, n, device=dev, dtype=torch.float64, generator=g).t()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    P.cholesky_inverse(B.t())          # symmetric: the column-major view is B
    t1 = time.perf_counter()           # (cholesky_inverse synchronises to check info)
    P.generalized_to_standard(A.t(), B.t())
    torch.cuda.synchronize()
    t2 = time.perf_counter()
    P.generalized_back(q, B.t())
    torch.cuda.synchronize()
    t3 = time.perf_counter()
    del A, B, q
    torch.cuda.empty_cache()
    c, f, b = t1 - t0, t2 - t1, t3 - t2
    return {"workload": f"generalized steps, n={n}, nev={nev}, r64, random SPD B",
            "cholesky_inverse_s": round(c, 3), "cholesky_inverse_tflops": round(2 * n ** 3 / 3 / c / 1e12, 2),
            "to_standard_s": round(f, 3), "to_standard_tflops": round(2 * n ** 3 / f / 1e12, 2),
            "back_s": round(b, 3), "back_tflops": round(n * n * nev / b / 1e12, 2)}


def recorded_traffic(workload):
    """HBM bytes per launch of the dominant kernel from the committed rocprofv3
    FETCH_SIZE / WRITE_SIZE passes (profiles/*_traffic.json), if they were taken
    for this workload and plan with the kernel sources as they are now; else
    None."""
    import glob
    import hashlib
    for f in sorted(glob.glob(os.path.join(ROOT, "profiles", "*_traffic.json"))):
        side = json.load(open(f))
        if side.get("workload") != workload:
            continue
        h = hashlib.sha256()
        for src in side["kernel_sources"]:
            h.update(open(os.path.join(ROOT, src), "rb").read())
        if h.hexdigest() == side["kernel_sources_sha256"]:
            return side["bytes_per_launch"]
    return None


def copy_calibration(mib):
    """A plain device-to-device copy of known size (read mib MiB, write mib MiB).
    Under rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE its counters give the factor
    from counter units to bytes for this GPU."""
    import torch
    dev = torch.device("cuda:0")
    n = mib * (1 << 20) // 8
    a = torch.empty(n, dtype=torch.float64, device=dev).uniform_()
    b = torch.empty_like(a)
    torch.cuda.synchronize()
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
    ev[0].record()
    for i in range(3):
        b.copy_(a)
        ev[i + 1].record()
    torch.cuda.synchronize()
    ms = [ev[i].elapsed_time(ev[i + 1]) for i in range(3)]
    print(json.dumps({"copy_bytes_read": n * 8, "copy_bytes_written": n * 8,
                      "ms": [round(x, 4) for x in ms],
                      "GBps_read_plus_write": round(2 * n * 8 / (min(ms) * 1e-3) / 1e9, 1)}),
          flush=True)


def peak_probe():
    """Measured issue rates of the arithmetic units (include/elpa_probe.h)."""
    import ctypes as C
    import torch
    import paper_1811_01277_amd as P
    torch.cuda.init()
    L = P.library()
    L.elpa_peak_probe.argtypes = [C.c_int32, C.c_int32, C.c_int64, C.POINTER(C.c_double),
                                  C.POINTER(C.c_double)]
    L.elpa_peak_probe.restype = C.c_int
    names = {0: "fp64 vector FMA", 1: "fp64 MFMA 16x16x4", 2: "fp32 MFMA 16x16x4",
             3: "fp32 vector FMA (no packed)"}
    iters = {0: 800000, 1: 40000, 2: 80000, 3: 800000}
    vendor = {0: 78.6, 1: 78.6, 2: 157.3, 3: 78.6}
    rows = []
    for kind in range(4):
        for w in (1, 2, 4):
            tf, ms = C.c_double(), C.c_double()
            rc = L.elpa_peak_probe(kind, w, iters[kind], C.byref(tf), C.byref(ms))
            if rc != 0:
                raise RuntimeError(P.strerror(rc))
            rows.append({"unit": names[kind], "waves_per_simd": w, "tflops": round(tf.value, 2),
                         "ms": round(ms.value, 2), "vendor_peak_tflops": vendor[kind]})
    print(json.dumps({"peak_probe": rows}), flush=True)


def counted_flops(n, nev, dt):
    return (8 if dt == "c64" else 2) * n * (n - 1) * nev


def host_threads():
    """Host threads this process may use: the cores of its CPU affinity mask,
    capped by OMP_NUM_THREADS when that is set (the host's share for this
    job)."""
    try:
        c = len(os.sched_getaffinity(0))
    except AttributeError:
        c = os.cpu_count() or 1
    env = os.environ.get("OMP_NUM_THREADS")
    if env and env.isdigit():
        c = min(c, int(env))
    return max(1, c)


def host_info():
    model = None
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    try:
        aff = len(os.sched_getaffinity(0))
    except AttributeError:
        aff = None
    return {"nproc": os.cpu_count(), "affinity_cores": aff,
            "omp_num_threads": os.environ.get("OMP_NUM_THREADS"), "cpu_model": model}


def cpu_baseline(args, hh, tau, Z):
    """The oracle (oracle/csrc/oracle.c, unchanged) on a column sample."""
    from oracle import bt
    n, nbw = args.n, args.nbw
    thr = host_threads()
    per_col = counted_flops(n, 1, args.dtype)
    # calibrate on one block of 8 columns per thread, then scale to ~cpu_seconds
    ncal = 8 * thr
    t0 = time.perf_counter()
    bt.bt_tridiag_to_band(hh, tau, np.asfortranarray(Z[:, :ncal]), n, nbw, nthreads=thr)
    tcal = time.perf_counter() - t0
    ncols = int(min(Z.shape[1], max(ncal, ncal * args.cpu_seconds / max(tcal, 1e-3))))
    ncols = max(ncal, (ncols // (8 * thr)) * 8 * thr)
    ncols = min(ncols, Z.shape[1])
    t0 = time.perf_counter()
    ref = bt.bt_tridiag_to_band(hh, tau, np.asfortranarray(Z[:, :ncols]), n, nbw, nthreads=thr)
    dt = time.perf_counter() - t0
    # one core: one 8-column block (the oracle's unit of work)
    t0 = time.perf_counter()
    bt.bt_tridiag_to_band(hh, tau, np.asfortranarray(Z[:, :8]), n, nbw, nthreads=1)
    dt1 = time.perf_counter() - t0
    return {"value": round(per_col * ncols / dt / 1e9, 3), "unit": "GFLOP/s", "cores": thr,
            "kind": "oracle",
            "sample": f"{ncols} of {Z.shape[1]} columns, all {n}x{n} nbw={nbw} reflectors, "
                      f"{dt:.1f} s, fp64 C oracle (OpenMP over 8-column blocks)",
            "one_core": {"value": round(per_col * 8 / dt1 / 1e9, 3), "unit": "GFLOP/s",
                         "sample": f"8 of {Z.shape[1]} columns, {dt1:.1f} s, 1 thread"},
            "host": host_info()}, ref


def accuracy(gpu_cols, ref, dt):
    """The GPU result of one call in the timed configuration against the
    oracle on the cpu_baseline leg's columns (fp64 inputs; for fp32 this is the
    fp32 error against the fp64 oracle)."""
    from oracle import checks
    m = min(gpu_cols.shape[1], ref.shape[1])
    err = checks.max_rel_err(gpu_cols[:, :m].astype(ref.dtype), ref[:, :m])
    out = {"columns": m, "max_rel_err_vs_fp64_oracle": float(f"{err:.3e}"),
           "measure": "max |gpu - oracle| / max |oracle| over the sampled columns"}
    if dt == "r32":
        out["note"] = ("fp32 inputs are the fp64 ones rounded; the 5e-5 parity bound of the "
                       "tests applies against the oracle on the rounded inputs")
    else:
        out["tol"] = 1e-12
    return out


def main():
    args = parse()
    if args.copy_calibration:
        copy_calibration(args.copy_calibration)
        return
    if args.peak_probe:
        peak_probe()
        return
    if args.solve_only:
        print(json.dumps({"solve": solve_leg(args)}), flush=True)
        if not args.no_gen:
            print(json.dumps({"generalized": gen_leg(args)}), flush=True)
        return
    if args.served_only:
        print(json.dumps({"served_stream": served_stream(args)}), flush=True)
        return
    if args.batched_only:
        print(json.dumps({"batched_workload": batched_workload(quick=True, order=args.order,
                                                               k=args.k)}),
              flush=True)
        return
    if args.bt2_only:
        print(json.dumps({"bt2": bt2_leg(args, [args.nev])}), flush=True)
        return
    if args.gpus != 1:
        print(json.dumps({"error": "the benchmark runs on one GPU only; --gpus must be 1 "
                                   "(the path shards by columns across GPUs by design, "
                                   "but no multi-GPU run exists)"}))
        sys.exit(2)
    import torch
    import paper_1811_01277_amd as P
    import workload as W

    dev = torch.device("cuda:0")
    n, nbw, nev, dt = args.n, args.nbw, args.nev, args.dtype
    cplx = dt == "c64"
    tdt = {"r64": torch.float64, "r32": torch.float32, "c64": torch.complex128}[dt]
    npdt = {"r64": np.float64, "r32": np.float32, "c64": np.complex128}[dt]
    hh, tau = W.synthetic_reflectors(n, nbw, complex_=cplx, seed=args.seed)
    Z = W.gaussian_block(n, nev, complex_=cplx, seed=args.seed + 1)
    q = torch.from_numpy(np.ascontiguousarray(Z.T).astype(npdt)).to(dev).t()
    h = torch.from_numpy(hh.astype(npdt)).to(dev)
    t = torch.from_numpy(tau.astype(npdt)).to(dev)
    torch.cuda.synchronize()
    stream = torch.cuda.current_stream(dev)

    plan = dict(path=args.path, k=args.k, steps=args.tile_steps, streams=args.streams,
                order=args.order)
    for _ in range(args.warmup):
        P.hh_trafo(q, h, t, nbw, stream=stream, **plan)
    torch.cuda.synchronize()
    # library-side HIP events on the launch stream around the main kernel
    # sequence of every call (the latest call's figures are read below)
    P.profile_enable(True)

    starts = [torch.cuda.Event(enable_timing=True) for _ in range(args.steps)]
    ends = [torch.cuda.Event(enable_timing=True) for _ in range(args.steps)]
    torch.cuda.synchronize()
    w0 = time.perf_counter()
    for i in range(args.steps):
        starts[i].record(stream)
        P.hh_trafo(q, h, t, nbw, stream=stream, **plan)
        ends[i].record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - w0
    prof = P.profile_last()  # last timed step: main kernel sequence
    P.profile_enable(False)
    per = [s.elapsed_time(e) for s, e in zip(starts, ends)]  # ms per call
    ms = wall * 1e3 / args.steps
    flops = counted_flops(n, nev, dt)
    # algorithmic flops per launch / average launch duration, times the
    # launches in flight (stripe groups on concurrent streams overlap their
    # launches): the dominant kernel's device-wide rate, flops / sequence time
    launches = max(1, prof["launches"])
    avg_launch_ms = prof["sum_launch_ms"] / launches
    in_flight = prof["sum_launch_ms"] / prof["kernel_ms"]
    achieved = (flops / launches) / (avg_launch_ms * 1e-3) * in_flight / 1e12
    peak = PEAK_TFLOPS[dt]
    direct = prof["path"] == 3 and dt == "r64"
    one = prof["launches"] == 1 and prof["steps"] == 0   # the sweep blocks in one launch
    kname = {1: "k_ref", 2: "k_diag",
             3: ("k_wyd_local / k_wyd_units" if one else "k_wyd") if direct else "k_split",
             4: "k_wy_units" if one else "k_wy"}.get(prof["path"], "?")
    # the compact-WY kernels run on the matrix cores and execute (nbw+16)/nbw
    # times the counted flops (their sub-groups' parallelograms padded to whole
    # 16-row tiles; path 3 applies T by itself, 8 more rows' worth); the VALU
    # kernels execute the counted flops
    mfma = prof["path"] == 4 or direct
    executed = achieved * ((nbw + (24 if direct else 16)) / nbw if mfma else 1.0)
    traffic = recorded_traffic({"n": n, "nbw": nbw, "nev": nev, "dtype": dt, "path": prof["path"],
                                "k": prof["k"], "tile_steps": prof["steps"],
                                "streams": prof["streams"]})
    value = flops / (ms * 1e-3) / 1e9
    out = {
        "metric": METRIC, "value": round(value, 2), "unit": "GFLOP/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(ms, 3),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": {"r64": "f64", "r32": "f32", "c64": "c128"}[dt], "data": "synthetic",
        "config": {"workload": f"tridiag->band back-transform, n={n}, nbw={nbw}, nev={nev}, "
                               f"{dt}, synthetic reflectors", "n": n, "nbw": nbw, "nev": nev,
                   "plan": {"path": prof["path"], "k": prof["k"], "tile_steps": prof["steps"],
                            "streams": prof["streams"]}},
        # the headline fraction from the same whole-call time as value; the
        # dominant kernel's own rate is roofline.achieved
        "pct_peak_whole_call": round(100.0 * value / 1e3 / peak, 2),
        "peak_tflops": peak,
        "roofline": {"bound": "mfma" if mfma else "alu", "achieved": round(achieved, 3),
                     "peak": peak, "achieved_executed": round(executed, 3),
                     "frac_executed": round(executed / peak, 4),
                     "unit": "TFLOP/s", "frac": round(achieved / peak, 4),
                     "traffic": None if traffic is None else round(traffic),
                     "kernel": kname, "launches": prof["launches"],
                     "avg_launch_us": round(avg_launch_ms * 1e3, 2),
                     "launches_in_flight": round(in_flight, 3),
                     "sequence_ms": round(prof["kernel_ms"], 3),
                     "flops_per_launch": flops / launches,
                     "call_ms": [round(x, 3) for x in per]},
    }
    gpu_cols = None
    if not args.no_cpu:
        # one fresh call in the timed configuration; its first columns are
        # checked against the oracle run of the cpu_baseline leg
        q.copy_(torch.from_numpy(np.ascontiguousarray(Z.T).astype(npdt)).t())
        P.hh_trafo(q, h, t, nbw, stream=stream, **plan)
        torch.cuda.synchronize()
        gpu_cols = q[:, :min(nev, 4096)].cpu().numpy()
    del q, h, t
    torch.cuda.empty_cache()
    if not args.no_configs:
        out["configs"] = configs_leg(args)
        torch.cuda.empty_cache()
    if not args.no_batched:
        out["batched_workload"] = batched_workload()
        torch.cuda.empty_cache()
    if not args.no_bt2:
        out["bt2"] = bt2_leg(args)
        torch.cuda.empty_cache()
    if not args.no_b2t:
        out["b2t"] = b2t_leg(args)
    if not args.no_f2b:
        out["f2b"] = f2b_leg(args)
    if not args.no_solve:
        out["solve"] = solve_leg(args)
    if not args.no_gen:
        out["generalized"] = gen_leg(args)
        torch.cuda.empty_cache()
    if not args.no_served:
        out["served_stream"] = served_stream(args)
        torch.cuda.empty_cache()
    if not args.no_cpu:
        out["cpu_baseline"], ref = cpu_baseline(args, hh, tau, Z)
        out["accuracy"] = accuracy(gpu_cols, ref, dt)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
