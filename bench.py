"""Benchmark of the split pressure-gradient projection step on one MI355X.

A step is one pass of the whole hot path -- ppe_solve + ppe_correct: right-hand
side (Eq. 29), real FFT in x, FFT in z, tridiagonal sweeps in y, inverse FFTs,
refinement sweeps when the precision is mixed, projection (Eq. 28) and its
continuity check -- over one synthetic two-phase sheet whose fields are
resident in HBM before the timed region starts.  Prints ONE JSON line.

  python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload NAME]

The roofline entry is measured live: a second pass over the same steps runs
with the library's per-kernel HIP-event timing (events on the plan's stream)
and the kernel with the largest total time is reported against the MI355X HBM
peak, with its algorithmic bytes per launch.  `traffic` is taken from the
committed rocprofv3 counter summary when it was collected from the current
kernel sources, else null.  The CPU baseline times the FP64 oracle (numpy /
scipy) on the same workload on the host.
"""

from __future__ import annotations

import argparse
import glob
import hashlib
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

# name -> (synth builder, precision, max_refine, description)
WORKLOADS = {
    "sheet_256x128x256_fp64": ("sheet_256", 0, 0,
                               "FP64 direct solve, 256x128x256 liquid sheet rho 640/100, Taylor-Green u* + 1% noise"),
    "sheet_512x256x512_mixed": ("sheet_512", 1, 1,
                                "FP32 spectra + FP64 refinement to 1e-12, 512x256x512 sheet rho 640/60"),
    "sheet_512x256x512_fp64": ("sheet_512", 0, 0, "FP64 direct solve, 512x256x512 sheet rho 640/60"),
    "sheet_32_fp64": ("sheet_32", 0, 0, "FP64 direct solve, 32^3 sheet rho 640/100"),
    "sheet_src_256x128x256_fp64": ("sheet_256", 0, 0,
                                   "FP64: target divergence from Eq. (26) inputs (phase compressibilities, "
                                   "interface mass flux, under-resolved block) + direct solve + correction, "
                                   "256x128x256 liquid sheet rho 640/100"),
    "fullstep_256x128x256_fp64": ("sheet_256", 0, 0,
                                  "FP64 flow step from u^n: predictor (Eq. 23: SMART convection, viscous stress, "
                                  "CSF) + target divergence (Eq. 26) + direct solve + correction, 256x128x256 "
                                  "liquid sheet rho 640/100"),
    "timeloop_256x128x256_fp64": ("sheet_256", 0, 0,
                                  "FP64 direct solve + correction in a time loop: p^n, p^{n-1} resident in a "
                                  "device ring, 256x128x256 liquid sheet rho 640/100"),
    "varcoef_256x128x256_fp64": ("sheet_256", 0, 0,
                                 "FP64 variable-coefficient pressure (Eq. 25) by the split fixed point to a "
                                 "1e-10 relative residual, then the variable-density projection, "
                                 "256x128x256 liquid sheet rho 640/100"),
    "jet_256x128x256_fp64": ("jet_256", 0, 0, "FP64 direct solve, 256x128x256 half jet over a symmetry plane "
                                               "with an outflow (p = 0) top, rho 640/100"),
    "batch_48_mixed": ("batch_48", 1, 1, "48 independent sheets of uneven sizes {64^3, 96x64x96, 128x64x128, "
                                          "192x96x192}, rho ratio U(3,12), FP32 spectra + FP64 refinement, "
                                          "same-shape instances batched per launch"),
    "batch_48_fp64": ("batch_48", 0, 0, "the same 48 sheets as batch_48_mixed through the FP64 direct solve, "
                                         "same-shape instances batched per launch"),
    "serve_fp64": ("serve", 0, 0, "the serve_mixed request stream through the FP64 direct solve"),
    "serve_mixed": ("serve", 1, 1, "Poisson-arrival stream of sheets over {32^3 .. 256x128x256}, FP32 spectra + "
                                   "FP64 refinement to 1e-12, each request's inputs copied into memory of its own "
                                   "at admission, inputs + outputs + plans admitted against a 64 GB HBM budget, "
                                   "plans cached, continuous "
                                   "batching on 4 streams"),
}

PEAK_HBM_GBS = 8000.0  # MI355X HBM3E, vendor figure

# kernels of the spectral chain, which may run in several kx chunks per pass
CHAIN_KERNELS = ("k_fft_z_fwd", "k_tri", "k_fft_z_inv")


def source_hash() -> str:
    """Hash of the kernel sources (counter summaries are valid for one hash)."""
    h = hashlib.sha256()
    for f in sorted(glob.glob(os.path.join(ROOT, "paper_2103_01874_amd", "csrc", "*"))):
        if f.endswith((".hip", ".hpp", ".inc", ".cpp")):
            h.update(open(f, "rb").read())
    return h.hexdigest()[:16]


def algorithmic_bytes(kernel: str, nx: int, ny: int, nz: int, precision: int, mode_update: bool = False,
                      n_iface: int = 0, ctx: dict | None = None) -> float:
    """Bytes one launch must move for one instance (the compulsory traffic).

    N cells, Nv = nx (ny+1) nz v-faces, Ns = (nx/2+1) ny nz spectral values of
    cs bytes (16 FP64, 8 FP32); n_iface interface cells (0 < C < 1) for the
    target-divergence pass.  `ctx` says how the workload launches a kernel:
    split (k_rhs with the p_hat term; False in the Eq. (25) iteration, which
    assembles only c), p_aliased (k_correct given one array for p, p^n and
    p^{n-1}), first_frac (the share of k_resid_var launches that form p_0 from
    p^n, p^{n-1}), viscous_separate (predictor given its own viscous-term
    velocities), one_march (the predictor's components share one pass over the
    inputs).  mode_update: for k_c2r the refinement launch (p read and
    written), for k_r2c the refinement launch (the residual as its source, in
    the spectrum's precision)."""
    ctx = ctx or {}
    N = nx * ny * nz
    Nv = nx * (ny + 1) * nz
    Ns = (nx // 2 + 1) * ny * nz
    cs = 16 if precision == 0 else 8
    split = ctx.get("split", True)
    first = ctx.get("first_frac", 0.0)
    pred_in = 8 * (8 * N + Nv) + (8 * (2 * N + Nv) if ctx.get("viscous_separate", False) else 0)
    table = {
        # u*, v*, w*, rho, p^n, p^{n-1}, S -> b; without the split term u*, v*, w*, S -> c
        "k_rhs": (8 * (6 * N + Nv) if split else 8 * (3 * N + Nv)) + 8 * N,
        # b, or the refinement residual (spectrum precision) -> half spectrum
        "k_r2c": (cs // 2 if mode_update else 8) * N + cs * Ns,
        "k_fft_z_fwd": 2 * cs * Ns,
        "k_fft_z_inv": 2 * cs * Ns,
        "k_tri": 2 * cs * Ns,
        "k_c2r": cs * Ns + 8 * N + (8 * N if mode_update else 0),
        "k_resid": 16 * N + (cs // 2) * N,             # b, p -> r (spectrum precision)
        # c, rho, p -> r; the first sweep reads p^n, p^{n-1} instead of p and also writes p
        "k_resid_var": (1 - first) * 32 * N + first * 48 * N,
        # u*,v*,w*,rho,p^n,p^{n-1},p,S -> u,v,w (one pressure array when aliased)
        "k_correct": 8 * ((5 if ctx.get("p_aliased", False) else 7) * N + Nv) + 8 * (2 * N + Nv),
        # C and one phase divergence -> S everywhere; interface cells also read
        # the other divergence, m', A/V0, rho_g, rho_l (8 B each) and the mask (1 B)
        "k_source": 24 * N + 41 * n_iface,
        # each component reads u^n, v^n, w^n, rho^n, rho^{n+1}, mu, C, sigma,
        # kappa (and the viscous-term velocities if separate), writes its own
        "k_predict_u": pred_in + 8 * N,
        "k_predict_v": pred_in + 8 * Nv,
        "k_predict_w": pred_in + 8 * N,
        # the three components in one launch: three passes, or one march
        "k_predict": (1 if ctx.get("one_march", False) else 3) * pred_in + 16 * N + 8 * Nv,
    }
    return float(table.get(kernel, 0.0))


def copy_gbs(dev, nbytes: int = 1 << 30, reps: int = 5) -> float:
    """Rate of a plain device-to-device copy of nbytes (read + write bytes / time)."""
    import torch

    src = torch.ones(nbytes // 8, dtype=torch.float64, device=dev)
    dst = torch.empty_like(src)
    dst.copy_(src)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record()
    for _ in range(reps):
        dst.copy_(src)
    b.record()
    torch.cuda.synchronize()
    ms = a.elapsed_time(b) / reps
    del src, dst
    return 2 * nbytes / (ms * 1e-3) / 1e9


def cpu_model() -> str:
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def cpu_baseline(pr, budget_s: float = 12.0, single_budget_s: float = 6.0):
    """The FP64 oracle on the same workload, timed on the host: with up to 16
    FFT workers, and again with one."""
    import oracle as O

    g = O.Grid(pr.nx, pr.ny, pr.nz, pr.lx, pr.ly, pr.lz, ybc=pr.ybc)

    def timed(workers, budget):
        steps = 0
        t0 = time.perf_counter()
        while True:
            O.ppe_step(g, pr.rho0, pr.dt, *pr.fields(), workers=workers)
            steps += 1
            el = time.perf_counter() - t0
            if el >= budget or steps >= 20:
                return steps, el

    workers = max(1, min(16, os.cpu_count() or 1))
    steps, el = timed(workers, budget_s)
    s1, e1 = timed(1, single_budget_s)
    return {"value": pr.npts * steps / el, "unit": "points/s", "cores": workers, "kind": "oracle",
            "sample": f"{steps} full step(s) of the same workload ({pr.nx}x{pr.ny}x{pr.nz}) in {el:.1f} s; "
                      f"scipy.fft with {workers} workers, numpy elementwise work on one thread",
            "single_worker": {"value": pr.npts * s1 / e1, "unit": "points/s", "cores": 1,
                              "sample": f"{s1} full step(s) in {e1:.1f} s, scipy.fft with 1 worker"},
            "cpu_model": cpu_model(), "host_cpus": os.cpu_count()}


def counter_traffic(workload: str, kernel: str):
    """HBM bytes per launch of `kernel` from profiles/counters_<workload>.json,
    if those counters were taken from the current kernel sources."""
    path = os.path.join(ROOT, "profiles", f"counters_{workload}.json")
    if not os.path.exists(path):
        return None
    try:
        d = json.load(open(path))
    except Exception:
        return None
    if d.get("source_hash") != source_hash():
        return None
    k = d.get("kernels", {}).get(kernel)
    if not k:
        return None
    return k.get("hbm_bytes_per_launch")


def run_batch(args, precision, max_refine, desc):
    """48 instances of uneven sizes; a step is one batched launch sequence per
    shape group, groups on separate streams."""
    import torch

    from paper_2103_01874_amd import binding, synth
    from paper_2103_01874_amd.serve import GpuBackend, Request, group_by_shape

    probs = synth.batch_48()
    dev = torch.device("cuda", 0)
    torch.cuda.set_device(dev)
    be = GpuBackend(n_slots=4, precision=precision, tol=1e-12, max_refine=max_refine)
    reqs = [Request(rid=i, shape=(p.nx, p.ny, p.nz), inputs=binding.to_device(p, dev), rho0=p.rho0, dt=p.dt,
                    arrival=0.0) for i, p in enumerate(probs)]
    groups = group_by_shape(reqs, binding.MAX_BATCH)
    plans = [be.make_plan(i % 4, g[0].shape, len(g), g[0].lengths) for i, g in enumerate(groups)]
    outs = [[{"p": torch.empty_like(r.inputs["rho"]), "u": torch.empty_like(r.inputs["us"]),
              "v": torch.empty_like(r.inputs["vs"]), "w": torch.empty_like(r.inputs["ws"])} for r in g]
            for g in groups]
    infos = [pl.new_info() for pl in plans]

    def one_step():
        for i, (pl, g) in enumerate(zip(plans, groups)):
            with torch.cuda.stream(be.streams[i % 4]):
                binding.step(pl, [r.inputs for r in g], [r.rho0 for r in g], [r.dt for r in g], outs[i], infos[i])

    for _ in range(args.warmup):
        one_step()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        one_step()
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1e3 / args.steps
    recs = [rec for inf in infos for rec in binding.decode_info(inf)]
    pts = sum(r.npts for r in reqs)
    kernels = None
    roofline = None
    if not args.no_profile:
        for pl in plans:
            pl.profile(True)
        # one group at a time, so that each launch's event bracket holds that
        # kernel alone (the timed steps above overlap the groups on 4 streams)
        for i, (pl, g) in enumerate(zip(plans, groups)):
            binding.step(pl, [r.inputs for r in g], [r.rho0 for r in g], [r.dt for r in g], outs[i], infos[i])
            torch.cuda.synchronize()
        tot = {}
        for pl, g in zip(plans, groups):
            nx, ny, nz = g[0].shape
            prof = pl.profile_read()
            for k, v in prof.items():
                b = algorithmic_bytes(k, nx, ny, nz, precision) * len(g)
                if k in ("k_c2r", "k_r2c") and max_refine > 0:
                    b = 0.5 * len(g) * (algorithmic_bytes(k, nx, ny, nz, precision, False)
                                        + algorithmic_bytes(k, nx, ny, nz, precision, True))
                # full passes: a chunked chain pass is one k_c2r launch
                n = prof["k_c2r"]["launches"] if k in CHAIN_KERNELS and "k_c2r" in prof else v["launches"]
                t = tot.setdefault(k, [0.0, 0.0])
                t[0] += v["total_ms"]
                t[1] += b * n
            pl.profile(False)
        kname, (tms, tb) = max(tot.items(), key=lambda kv: kv[1][0])
        achieved = tb / (tms * 1e-3) / 1e9
        roofline = {"bound": "hbm", "achieved": achieved, "peak": PEAK_HBM_GBS, "unit": "GB/s",
                    "frac": achieved / PEAK_HBM_GBS, "traffic": None, "kernel": kname,
                    "note": "summed over the shape groups of one step, timed with the groups run one "
                            "after another (the timed steps overlap them on 4 streams)"}
        kernels = {k: round(v[0], 4) for k, v in sorted(tot.items(), key=lambda kv: -kv[1][0])}
    for pl in plans:
        pl.close()
    return {"ms": ms, "points": pts, "recs": recs, "roofline": roofline, "kernels_total_ms": kernels,
            "extra": {"instances": len(reqs), "groups": [[list(g[0].shape), len(g)] for g in groups],
                      "eps_div_max": max(r["res_rel"] for r in recs),
                      "iters_max": max(r["iters"] for r in recs),
                      "status_nonzero": sum(1 for r in recs if r["status"] != 0)}}


def run_serve(args, precision, max_refine, desc, n_requests=500):
    """Poisson stream served with continuous batching; saturated throughput,
    then p50/p99 latency at 0.5x and 0.8x of it."""
    import numpy as np
    import torch

    from paper_2103_01874_amd import binding, synth
    from paper_2103_01874_amd.serve import GpuBackend, Request, Server, poisson_arrivals

    dev = torch.device("cuda", 0)
    torch.cuda.set_device(dev)
    max_points = args.max_points if args.max_points > 0 else None
    pool = {}
    for si, shape in enumerate(synth.SERVE_SHAPES):
        pool[shape] = []
        for k in range(2):
            pr = synth.mixed_instance(5000 + 10 * si + k, shape=shape)
            pool[shape].append((pr, binding.to_device(pr, dev)))
    rng = np.random.default_rng(5000)
    picks = [(synth.SERVE_SHAPES[int(rng.integers(0, len(synth.SERVE_SHAPES)))], int(rng.integers(0, 2)))
             for _ in range(n_requests)]

    def requests(arrivals):
        # every request gets device inputs of its own, copied from the pool at
        # admission and charged against the budget until it completes
        out = []
        for i, ((shape, k), a) in enumerate(zip(picks, arrivals)):
            pr, f = pool[shape][k]
            out.append(Request(rid=i, shape=shape, inputs=None, source=f, rho0=pr.rho0, dt=pr.dt,
                               arrival=float(a)))
        return out

    be = GpuBackend(n_slots=4, precision=precision, tol=1e-12, max_refine=max_refine)
    budget = 64 << 30
    # warm the plan cache and the kernels once
    warm = Server(be, budget, n_slots=4, max_group=8, max_points=max_points)
    warm.run(requests([0.0] * n_requests))
    results = {}
    srv = Server(be, budget, n_slots=4, max_group=8, max_points=max_points)
    srv.plans, srv.used = warm.plans, sum(v[1] for v in warm.plans.values())
    m = srv.run(requests([0.0] * n_requests))
    results["saturated"] = m
    rate_sat = m["requests_per_s"]
    for frac in (0.5, 0.8):
        reqs = requests(poisson_arrivals(n_requests, frac * rate_sat, 77))
        srv2 = Server(be, budget, n_slots=4, max_group=8, max_points=max_points)
        srv2.plans, srv2.used = srv.plans, sum(v[1] for v in srv.plans.values())
        results[f"poisson_{frac}"] = dict(srv2.run(reqs), rate_per_s=frac * rate_sat)
        bad = [r for r in reqs if r.status != 0]
        results[f"poisson_{frac}"]["status_nonzero"] = len(bad)
        results[f"poisson_{frac}"]["eps_div_max"] = max(r.info["res_rel"] for r in reqs if r.info)
    for plan, _ in srv.plans.values():
        plan.close()
    return results


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--workload", default="sheet_512x256x512_fp64", choices=sorted(WORKLOADS))
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-profile", action="store_true", help="skip the event-timed roofline pass")
    ap.add_argument("--max-points", type=int, default=256 * 128 * 256,
                    help="serving: cap on the grid points of one batched group (0: none); the default, one "
                         "256x128x256 instance, cut p99 by a fifth to a third against no cap")
    ap.add_argument("--copy-bytes", type=int, default=0,
                    help="also run a plain device copy of this many bytes 3 times (counter calibration)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(json.dumps({"error": "one GPU only: a projection step of one grid runs on one MI355X here; "
                                   "sharding across GPUs is described in the design notes, not built",
                          "n_gpus": args.gpus}), flush=True)
        sys.exit(2)

    import torch

    import numpy as np

    from paper_2103_01874_amd import binding, synth

    builder, precision, max_refine, desc = WORKLOADS[args.workload]
    if builder in ("batch_48", "serve"):
        base = {"metric": "PPE grid points/s (projection step: solve + correction) at 1e-12 relative divergence "
                          "residual", "unit": "points/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
                "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
                "dtype": "f64" if precision == 0 else "f32+f64", "data": "synthetic"}
        if builder == "batch_48":
            r = run_batch(args, precision, max_refine, desc)
            out = dict(base, value=r["points"] / (r["ms"] * 1e-3), ms_per_step=r["ms"],
                       config={"workload": args.workload, "description": desc, "points": r["points"],
                               "precision": "fp64" if precision == 0 else "mixed", "max_refine": max_refine,
                               "parallelism": "single GPU"},
                       result=r["extra"], roofline=r["roofline"], cpu_baseline=None,
                       kernels_total_ms=r["kernels_total_ms"], source_hash=source_hash())
        else:
            r = run_serve(args, precision, max_refine, desc)
            sat = r["saturated"]
            out = dict(base, value=sat["points_per_s"], ms_per_step=None,
                       config={"workload": args.workload, "description": desc, "requests": sat["served"],
                               "precision": "fp64" if precision == 0 else "mixed", "max_refine": max_refine,
                               "parallelism": "single GPU"},
                       serving=r, roofline=None, cpu_baseline=None, source_hash=source_hash())
        print(json.dumps(out), flush=True)
        return
    pr = getattr(synth, builder)()
    dev = torch.device("cuda", 0)
    torch.cuda.set_device(dev)
    stream = torch.cuda.Stream(dev)
    with torch.cuda.stream(stream):
        plan = binding.Plan(pr.nx, pr.ny, pr.nz, pr.lx, pr.ly, pr.lz, precision=precision, tol=1e-12,
                            max_refine=max_refine, stream=stream, ybc=pr.ybc,
                            flags=binding.PPE_FLAG_VARCOEF if args.workload.startswith("varcoef") else 0)
        fields = binding.to_device(pr, dev)
        outs = {"p": torch.empty_like(fields["rho"]), "u": torch.empty_like(fields["us"]),
                "v": torch.empty_like(fields["vs"]), "w": torch.empty_like(fields["ws"])}
        info = plan.new_info()
    torch.cuda.synchronize()
    g = lambda k: [fields[k]]
    o = lambda k: [outs[k]]
    src_dev = None
    pred_dev = None
    n_iface = 0
    if args.workload.startswith("fullstep"):
        rin = synth.predictor_inputs(pr, pr.meta["seed"] + 53)
        with torch.cuda.stream(stream):
            pred_dev = {k: (torch.from_numpy(np.ascontiguousarray(v)).to(dev) if isinstance(v, np.ndarray) else v)
                        for k, v in rin.items()}
        torch.cuda.synchronize()
    if "_src_" in args.workload or args.workload.startswith("fullstep"):
        # Eq. (26) inputs around the same interface as the density field
        rl, rg = pr.meta["rho_l"], pr.meta["rho_g"]
        C = (pr.rho - rg) / (rl - rg)
        src = synth.interface_inputs(np.random.default_rng(pr.meta["seed"] + 31), C, pr.lx, pr.ly, pr.lz, rl, rg)
        n_iface = int(((src.C > 0) & (src.C < 1)).sum())
        with torch.cuda.stream(stream):
            src_dev = binding.sources_to_device(src, dev)
        torch.cuda.synchronize()

    ring = None
    if args.workload.startswith("timeloop"):
        with torch.cuda.stream(stream):
            ring = binding.Ring(plan, g("pn"), g("pnm1"))
        torch.cuda.synchronize()

        def one_step():
            ring.step([pr.rho0], [pr.dt], g("us"), g("vs"), g("ws"), g("rho"), g("S"), o("u"), o("v"), o("w"), info)
    elif args.workload.startswith("varcoef"):
        def one_step():
            plan.solve_varcoef([pr.rho0], [pr.dt], g("us"), g("vs"), g("ws"), g("rho"), g("pn"), g("pnm1"), g("S"),
                               o("p"), 1000, 1e-10, info=info)
            plan.correct([pr.dt], g("us"), g("vs"), g("ws"), g("rho"), o("p"), o("p"), o("p"), g("S"), o("u"),
                         o("v"), o("w"), info)
    else:
        one_step = None

    def split_step():
        if pred_dev is not None:
            # u^p into the u* buffers of the projection
            plan.predict([pred_dev], g("us"), g("vs"), g("ws"))
        if src_dev is not None:
            plan.source([src_dev], g("S"))
        plan.solve([pr.rho0], [pr.dt], g("us"), g("vs"), g("ws"), g("rho"), g("pn"), g("pnm1"), g("S"), o("p"),
                   info)
        plan.correct([pr.dt], g("us"), g("vs"), g("ws"), g("rho"), g("pn"), g("pnm1"), o("p"), g("S"), o("u"),
                     o("v"), o("w"), info)

    if one_step is None:
        one_step = split_step
    for _ in range(args.warmup):
        one_step()
    torch.cuda.synchronize()
    start = torch.cuda.Event(enable_timing=True)
    stop = torch.cuda.Event(enable_timing=True)
    t0 = time.perf_counter()
    start.record(stream)
    for _ in range(args.steps):
        one_step()
    stop.record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    ms = start.elapsed_time(stop) / args.steps
    rec = binding.decode_info(info)[0]
    npts = pr.npts
    print(f"# timed {args.steps} steps: {ms:.4f} ms/step, eps_div={rec['res_rel']:.3e} iters={rec['iters']}",
          file=sys.stderr, flush=True)

    roofline = None
    kernels = None
    if not args.no_profile:
        plan.profile(True)
        for _ in range(args.steps):
            one_step()
        kernels = plan.profile_read()
        plan.profile(False)
        dom = max(kernels.items(), key=lambda kv: kv[1]["total_ms"])
        kname, kv = dom
        varcoef = args.workload.startswith("varcoef")
        ctx = {"split": not varcoef, "p_aliased": varcoef, "one_march": True,
               "first_frac": 1.0 / (rec["iters"] + 1) if varcoef else 0.0}

        def launch_bytes(k):
            if k == "k_c2r" and varcoef:  # every sweep updates p
                return algorithmic_bytes(k, pr.nx, pr.ny, pr.nz, precision, True, ctx=ctx)
            if k in ("k_c2r", "k_r2c") and max_refine > 0:
                # the first launch solves for p, the refinement launches correct it: average
                nu = min(max_refine, rec["iters"])
                return (algorithmic_bytes(k, pr.nx, pr.ny, pr.nz, precision, False, ctx=ctx)
                        + nu * algorithmic_bytes(k, pr.nx, pr.ny, pr.nz, precision, True, ctx=ctx)) / (1 + nu)
            return algorithmic_bytes(k, pr.nx, pr.ny, pr.nz, precision, n_iface=n_iface, ctx=ctx)

        # the spectral chain may run in kx chunks (one launch per chunk and
        # pass); a full pass of its kernels is one k_c2r launch
        def full_us(k):
            v = kernels[k]
            n = kernels["k_c2r"]["launches"] if k in CHAIN_KERNELS and "k_c2r" in kernels else v["launches"]
            return 1e3 * v["total_ms"] / max(1, n)

        per_launch = launch_bytes(kname)
        achieved = per_launch / (full_us(kname) * 1e-6) / 1e9
        traffic = counter_traffic(args.workload, kname)
        roofline = {"bound": "hbm", "achieved": achieved, "peak": PEAK_HBM_GBS, "unit": "GB/s",
                    "frac": achieved / PEAK_HBM_GBS, "traffic": traffic, "kernel": kname,
                    "avg_launch_us": full_us(kname), "bytes_per_launch": per_launch}
        # every kernel's algorithmic rate, for the per-kernel view
        kernels_gbs = {}
        for k, v in kernels.items():
            bpl = launch_bytes(k)
            if bpl > 0:
                kernels_gbs[k] = round(bpl / (full_us(k) * 1e-6) / 1e9, 1)
        roofline["kernels_gbs"] = kernels_gbs
        # the same box's plain device copy, for scale next to the vendor peak
        cg = copy_gbs(dev)
        roofline["copy_gbs"] = round(cg, 1)
        roofline["frac_of_copy"] = achieved / cg
        kernels = {k: round(full_us(k), 2) for k, v in sorted(kernels.items(), key=lambda kv: -kv[1]["total_ms"])}

    if args.copy_bytes > 0:
        n = args.copy_bytes // 8
        src = torch.ones(n, dtype=torch.float64, device=dev)
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        for _ in range(3):
            torch.mul(src, 1.0, out=dst)
        torch.cuda.synchronize()
        del src, dst

    cpu = None
    if not args.no_cpu_baseline:
        cpu = cpu_baseline(pr)

    out = {
        "metric": "PPE grid points/s (projection step: solve + correction) at 1e-12 relative divergence residual",
        "value": npts / (ms * 1e-3),
        "unit": "points/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64" if precision == 0 else "f32+f64",
        "data": "synthetic",
        "config": {"workload": args.workload, "description": desc, "grid": [pr.nx, pr.ny, pr.nz],
                   "points": npts, "precision": "fp64" if precision == 0 else "mixed",
                   "y_boundaries": "walls" if pr.ybc == 0 else "symmetry bottom, outflow top",
                   "max_refine": max_refine, "parallelism": "single GPU"},
        "result": {"eps_div": rec["res_rel"], "iters": rec["iters"], "status": rec["status"],
                   **({"ms_per_sweep": ms / max(1, rec["iters"] + 1)} if args.workload.startswith("varcoef")
                      else {})},
        "roofline": roofline,
        "cpu_baseline": cpu,
        "kernels_avg_us": kernels,
        "wall_s": wall,
        "source_hash": source_hash(),
    }
    print(json.dumps(out), flush=True)
    if ring is not None:
        ring.close()
    plan.close()


if __name__ == "__main__":
    main()
