#!/usr/bin/env python3
"""Benchmark of the chi0 band sum on one MI355X.

Default workload (the largest configuration that fits one GPU): the 256-atom-MgO-shaped
polarizability -- 128^3 FFT grid, 137,065-plane-wave wavefunction sphere, 512 valence bands and
25,000 conduction bands of which those above E0 = 30 eV are grouped into 1 eV windows (Eqs. (chi02)
and (energyintegration): 8,451 explicit columns + 30 window representatives, 4.34 M band pairs),
8,000 G-vectors in the dielectric sphere, q = (0.01, 0, 0), static.  Seeded synthetic inputs
(orthonormal random coefficients, sqrt(E) conduction spectrum) stand in for the paper's MgO
wavefunctions.

One step = one gw_chi0_build (band transforms, pair transforms, weights, contraction) followed by
gw_eps_inv of the result (float64), every input already in HBM.  The headline (`value`) is the
mixed-precision path (split-BF16x3 contraction with float32 accumulation on float32 pair
densities; float64 weights, accumulation across chunks and eps^-1); one float64 step is timed
beside it and gives the error of the mixed path.  A bounded sample of the same workload runs
through the CPU oracle as a reported baseline (its full-size time extrapolated linearly in band
pairs, and labelled so).  The 64-atom workload (72^3, 128 x 4,000, NG 2,000) is reported beside it
in float64, float32 and split-BF16x3.  Prints one JSON line on stdout; progress goes to stderr.
"""
import argparse
import json
import math
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "chi0 build TFLOP/s + band-pairs/s, FP64 vs mixed vs oracle, err vs FP64"
PEAK = {"fp64_vec": 78.6, "fp64_mfma": 78.6, "fp32_mfma": 157.3, "fp32_vec_nopk": 78.6, "bf16_mfma": 2500.0,
        "hbm": 8000.0}


T_START = time.time()


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def within_budget(args, seconds, what):
    """True if a leg of about `seconds` still ends inside the run's time budget (the timed steps
    are never cut; only the legs reported beside them are skipped, and say so)."""
    left = args.budget_s - (time.time() - T_START)
    if seconds <= left:
        return True
    log(f"{what}: skipped, about {seconds:.0f} s needed and {left:.0f} s of the {args.budget_s:.0f} s budget left")
    return False


def transform_grid(nd, gw, gc):
    """Points per axis of the library's transforms: the smallest alias-free multiple of 4."""
    rw, rc = int(np.abs(gw).max()), int(np.abs(gc).max())
    return min(nd, -(-max(2 * rw + rc + 1, 2 * rc + 1, 16) // 4) * 4)


def flops_model(nd, k, ng, npair, nband, with_inverse=True):
    """Algorithmic flop counts of a build on an nd^3 grid (the GPU's: transform_grid, the grid its
    transforms run on; the oracle's: the stated grid): pruned forward transform per pair (three passes over
    N, N K/N_d and N K^2/N_d^2 points at 5 n log2 n), the product (6 N), the band
    transforms (5 N log2 N each), the Hermitian contraction (4 NG^2 per pair) and the static
    inverse by Hermitian sweeps (a rank-64 update of the lower triangle per 64 pivots, 4 NG^3)."""
    n = nd ** 3
    lg = math.log2(nd)
    planes = 5.0 * n * lg * (1.0 + k / nd) + 6.0 * n
    finish = 5.0 * n * lg * (k * k / nd ** 2)
    band = 5.0 * n * math.log2(n)
    contract = 4.0 * ng * ng
    inverse = 4.0 * ng ** 3 if with_inverse else 0.0
    return {"planes": planes * npair, "finish": finish * npair, "band": band * nband, "contract": contract * npair,
            "eps_inv": inverse, "total": (planes + finish + contract) * npair + band * nband + inverse}


KERNEL_OF_STAGE = {"planes": ("pair_transform.hip", ("k_pair_planes<{t}, 7", "k_pair_planes_mfma<7")),
                   "finish": ("pair_transform.hip", "k_pair_finish<{t}, 7"),
                   "contract": ("contract.hip", "k_contract_batch<{m},")}


def sources_unchanged(tr, src):
    """True when the kernel's source file and the shared device headers recorded beside it are
    byte-identical to the ones the counters were taken with."""
    import hashlib
    for name in [src] + [n for n in tr["sources"] if n.endswith(".h")]:
        with open(os.path.join(ROOT, "paper_1601_06767_amd", "csrc", name), "rb") as f:
            if hashlib.sha256(f.read()).hexdigest() != tr["sources"][name]:
                return False
    return True


def measured_traffic(stage, mode):
    """HBM bytes per launch of the stage's kernel from the committed FETCH_SIZE / WRITE_SIZE
    summary, or None when that kernel's source changed since the counters were taken."""
    try:
        with open(os.path.join(ROOT, "profiles", "traffic.json")) as f:
            tr = json.load(f)
        src, pat = KERNEL_OF_STAGE[stage]
        if not sources_unchanged(tr, src):
            return None
        pats = pat if isinstance(pat, tuple) else (pat,)
        if stage == "planes":   # float64 and float32 have a kernel each
            pats = pats[:1] if mode == "fp64" else pats[1:]
        keys = tuple(p.format(t="double" if mode == "fp64" else "float", m={"fp64": 0, "fp32": 1, "bf16x3": 2}[mode])
                     for p in pats)
        if stage == "contract" and mode == "bf16x3":
            keys = ("k_contract_img",)   # the static split-BF16x3 contraction
        for k, v in tr["kernels"].items():
            if k.startswith(keys):
                return {"read_bytes": v["read_bytes_per_dispatch"], "write_bytes": v["write_bytes_per_dispatch"],
                        "bytes": v["read_bytes_per_dispatch"] + v["write_bytes_per_dispatch"],
                        "kernel": k, "source": v.get("profile", "profiles/traffic.json")}
    except (OSError, KeyError, ValueError):
        pass
    return None


def traffic_for(prefixes, src):
    """HBM bytes per dispatch of the first kernel in profiles/traffic.json whose name starts with
    one of the prefixes, or None when its source file changed since the counters were taken."""
    try:
        with open(os.path.join(ROOT, "profiles", "traffic.json")) as f:
            tr = json.load(f)
        if not sources_unchanged(tr, src):
            return None
        for k, v in tr["kernels"].items():
            if k.startswith(tuple(prefixes)):
                return {"read_bytes": v["read_bytes_per_dispatch"], "write_bytes": v["write_bytes_per_dispatch"],
                        "bytes": v["read_bytes_per_dispatch"] + v["write_bytes_per_dispatch"],
                        "kernel": k, "source": v.get("profile", "profiles/traffic.json")}
    except (OSError, KeyError, ValueError):
        pass
    return None


def timed_steps(p, ctx, torch, run, steps, warmup, label):
    """warmup untimed calls, then steps timed between two events on the current stream with the
    library's stage timers on: (ms per step, wall seconds, stage ms per step, launches per step)."""
    for _ in range(warmup):
        run()
    torch.cuda.synchronize()
    p.gw_ctx_stage_times(ctx, reset=True)
    p.gw_ctx_set_timing(ctx, True)
    stream = torch.cuda.current_stream()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    tw = time.perf_counter()
    e0.record(stream)
    for i in range(steps):
        run()
        log(f"{label}: step {i + 1}/{steps} enqueued")
    e1.record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - tw
    p.gw_ctx_set_timing(ctx, False)
    stages = p.gw_ctx_stage_times(ctx, reset=True)
    ms = e0.elapsed_time(e1) / steps
    return (ms, wall, {k: v[0] / steps for k, v in stages.items() if v[1]},
            {k: v[1] / steps for k, v in stages.items() if v[1]})


def run_headline(args, torch, synth, p, dev):
    """The 256-atom-shaped grouped workload in mixed precision (timed steps), one float64 step,
    the oracle on a bounded sample, and the 64-atom workload beside it."""
    cfg = synth.config(4)
    hev = synth.HARTREE_EV
    nd = cfg.nd
    gw = synth.wf_sphere(nd)
    gc = synth.chi_sphere(cfg.ng[0], cfg.qs[0], cfg.cell)
    e_all = synth.conduction_energies(cfg)
    nwin = int(round((cfg.emax_ev - cfg.e0_ev) / cfg.de_ev))
    col, e_col, n_col, n0 = p.gw_group_windows(e_all, cfg.e0_ev / hev, cfg.de_ev / hev, nwin)
    t0 = time.time()
    workers = max(1, min(16, len(os.sched_getaffinity(0))))
    bands_idx = np.concatenate([np.arange(cfg.nv), cfg.nv + np.asarray(col)])
    rows = synth.gaussian_columns_threaded(cfg.index, 0, bands_idx, len(gw), workers)
    log(f"headline: {len(bands_idx)} coefficient rows of {len(gw)} plane waves in {time.time() - t0:.1f}s")
    qd = synth.orthonormalize_on_device(rows, "cuda")
    del rows
    cv = qd[:cfg.nv].contiguous()
    cc = qd[cfg.nv:].contiguous()
    del qd
    torch.cuda.synchronize()
    ev_host = synth.valence_energies(cfg, 0)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    ev, ecol, ncol = t(ev_host), t(e_col), t(n_col)
    log(f"headline inputs: {nd}^3, npw={len(gw)}, nv={cfg.nv}, {cfg.nc} bands -> {len(col)} columns ({n0} explicit "
        f"+ {len(col) - n0} windows), NG={len(gc)}, ready in {time.time() - t0:.1f}s")
    ctx = p.gw_ctx_create(0)
    p.gw_ctx_set_overlap(ctx, 0 if args.no_overlap else 1)
    geom = p.gw_geom_create(ctx, (nd,) * 3, gw, gc, cfg.cell, cfg.qs[0])
    prob = p.make_problem(geom, cv, ev, cc, ecol, ncol)
    ng = len(gc)
    vcoul = t(synth.coulomb(gc, cfg.qs[0], cfg.cell))
    k = 2 * int(np.abs(gc).max()) + 1
    npair = cfg.nv * len(col)
    fl = flops_model(transform_grid(nd, gw, gc), k, ng, npair, cfg.nv + len(col))
    head = args.head_mode
    modes = [head] + ([] if args.no_fp64_step or head == "fp64" else ["fp64"])
    wsb = max(p.gw_chi0_workspace_size(ctx, [prob], 1, p.PRECISIONS[m]) for m in modes)
    ws = torch.empty(wsb, dtype=torch.uint8, device=dev)
    ws_inv = torch.empty(p.gw_eps_inv_workspace_size(ctx, ng, 1), dtype=torch.uint8, device=dev)
    log(f"workspace {wsb / 2**30:.1f} GiB")
    results, chis, zs = {}, {}, {}
    skipped = {}
    for m in modes:
        if m != head and not within_budget(args, 3.2 * results[head]["ms_per_step"] * 1e-3 + 10, f"{m} step"):
            skipped[m] = "time budget"
            continue
        out = torch.empty(ng * ng, dtype=torch.complex128, device=dev)     # one output per mode
        zout = torch.empty((ng, ng), dtype=torch.complex128, device=dev)

        def run():
            p.gw_chi0_build(ctx, [prob], [ng], [0.0], 0.0, p.PRECISIONS[m], workspace=ws, out=out)
            p.gw_eps_inv(ctx, vcoul, out.view(ng, ng), workspace=ws_inv, out=zout, hermitian=True)
        steps, warm = (args.steps, args.warmup) if m == head else (1, 0)
        ms, wall, st, nl = timed_steps(p, ctx, torch, run, steps, warm, m)
        p.gw_eps_inv_status(ctx)
        chis[m], zs[m] = out.view(ng, ng), zout
        results[m] = {"ms_per_step": ms, "steps": steps, "warmup": warm, "wall_s": wall,
                      "tflops": fl["total"] / (ms * 1e-3) / 1e12, "band_pairs_per_s": npair / (ms * 1e-3),
                      "stages_ms_per_step": st, "stage_launches_per_step": nl}
        log(f"{m}: {ms:.1f} ms/step, {results[m]['tflops']:.2f} TFLOP/s, stages {st}")
    if "fp64" in chis:
        ref, zref = chis["fp64"], zs["fp64"]
        rmax, zmax = ref.abs().max(), zref.abs().max()
        for m in chis:
            d = chis[m] - ref
            dz = zs[m] - zref
            results[m]["err_vs_fp64"] = float(torch.linalg.norm(d) / torch.linalg.norm(ref))
            results[m]["max_err_vs_fp64"] = float(d.abs().max() / rmax)
            results[m]["eps_inv_max_err_vs_fp64"] = float(dz.abs().max() / zmax)
            # without the head row and column: at q -> 0 the head of chi0 is zero in exact
            # arithmetic (orthogonal bands), and the float32 pair densities leave <v|c> ~ 1e-7 there,
            # which v(q) of the head multiplies
            results[m]["eps_inv_max_err_vs_fp64_wings_excluded"] = float(dz[1:, 1:].abs().max() / zmax)
            results[m]["eps_inf"] = float(1.0 / zs[m][0, 0].real)
            del d, dz
        results["fp64"]["hermitian_residual"] = float((ref - ref.conj().T).abs().max() / rmax)
        if head != "fp64":
            results[head]["speedup_vs_fp64"] = results["fp64"]["ms_per_step"] / results[head]["ms_per_step"]
    del chis, zs
    hr = results[head]
    # dominant kernel of the timed mode against its roofline
    st = hr["stages_ms_per_step"]
    dom = max(st, key=st.get)
    launches = hr["stage_launches_per_step"][dom]
    avg_ms = st[dom] / launches
    fp = "double" if head == "fp64" else "float"
    if dom == "contract":
        bound = "mfma"
        peak = {"fp64": PEAK["fp64_mfma"], "fp32": PEAK["fp32_mfma"], "bf16x3": PEAK["bf16_mfma"]}[head]
        work = fl["contract"] / launches
        traffic = traffic_for(["k_contract_img" if head == "bf16x3" else
                               f"k_contract_batch<{ {'fp64': 0, 'fp32': 1}[head] },"], "contract.hip")
        basis = f"{head} matrix-core peak (split products not counted as work)"
    else:
        bound = "alu"
        peak = PEAK["fp64_vec"] if head == "fp64" else PEAK["fp32_vec_nopk"]
        work = fl[dom] / launches
        rc = (k - 1) // 2
        kern = {"planes": [f"k_pair_planes<double, {rc}," if head == "fp64" else f"k_pair_planes_mfma<{rc},"],
                "finish": [f"k_pair_finish<{fp}, {rc}"], "band": [f"k_band_ab<{fp},"]}.get(dom, [dom])
        traffic = traffic_for(kern,
                              "pair_transform.hip" if dom in ("planes", "finish") else "band_fft.hip")
        basis = ("256 CU x 4 SIMD x 16 lanes x 2 flop (FMA) x 2.4 GHz: the float64 vector rate, and the float32 "
                 "rate without packed instructions, which the library is compiled without")
    achieved = work / (avg_ms * 1e-3) / 1e12
    roofline = {"bound": bound, "kernel": dom, "achieved": achieved, "peak": peak, "unit": "TFLOP/s",
                "frac": achieved / peak, "traffic": traffic, "avg_launch_ms": avg_ms,
                "algorithmic_work_per_launch": work, "peak_basis": basis}
    # the oracle on a bounded sample of the same workload (full grid and sphere)
    cpu = None
    nvs, ncs = (int(x) for x in args.cpu_pairs.split("x"))
    want_cpu = args.cpu_sample > 0 and nvs > 0 and ncs > 0
    if want_cpu and not within_budget(args, 45, "oracle sample"):
        skipped["cpu_baseline"] = "time budget"
        want_cpu = False
    if want_cpu:
        import oracle
        cores = len(os.sched_getaffinity(0))
        vs = np.linspace(0, cfg.nv - 1, nvs).astype(int)
        cs = np.linspace(0, len(col) - 1, ncs).astype(int)
        cv_s = cv[torch.from_numpy(vs).to(dev)].cpu().numpy()
        cc_s = cc[torch.from_numpy(cs).to(dev)].cpu().numpy()
        t1 = time.perf_counter()
        ref_s = oracle.chi0_bands(cv_s, ev_host[vs], cc_s, e_col[cs], gw, gc, (nd,) * 3, n_col=n_col[cs])[0]
        dt = time.perf_counter() - t1
        sp = len(vs) * len(cs)
        fs = flops_model(nd, k, ng, sp, len(vs) + len(cs), with_inverse=False)
        sub = p.make_problem(geom, t(cv_s), t(ev_host[vs]), t(cc_s), t(e_col[cs]), t(n_col[cs]))
        gchi = p.gw_chi0_build(ctx, [sub], [ng], [0.0], 0.0, p.GW_FP64)[0][0].cpu().numpy()
        rate = (fs["total"] - fs["eps_inv"]) / dt / 1e12
        cpu = {"value": rate, "unit": "TFLOP/s", "cores": cores, "kind": "oracle",
               "band_pairs_per_s": sp / dt, "seconds": dt,
               "sample": f"{len(vs)} valence x {len(cs)} columns ({sp} pairs) of the same workload, full 128^3 grid "
                         f"and 8000-G sphere, scipy.fft workers={cores}",
               "full_build_s_extrapolated": npair / (sp / dt),
               "extrapolation": "linear in band pairs (the sum's cost is per pair plus per band)",
               "gpu_fp64_err_on_sample": float(np.linalg.norm(gchi - ref_s) / np.linalg.norm(ref_s))}
        log(f"oracle sample: {sp} pairs in {dt:.1f}s ({cpu['value'] * 1e3:.3f} GFLOP/s); GPU fp64 on the sample "
            f"{cpu['gpu_fp64_err_on_sample']:.1e} from it")
    c2 = None
    if not args.no_c2:
        if within_budget(args, 40, "72^3 workload"):
            c2 = run_c2_beside(args, torch, synth, p, dev, ctx)
        else:
            skipped["mgo64_static_72cube"] = "time budget"
    line = {"metric": METRIC, "value": hr["tflops"], "unit": "TFLOP/s", "n_gpus": 1, "steps": args.steps,
            "warmup": args.warmup, "ms_per_step": hr["ms_per_step"], "higher_is_better": True, "scaling": "weak",
            "vs_baseline": None, "dtype": {"fp64": "f64", "fp32": "f32", "bf16x3": "bf16x3"}[head],
            "data": "synthetic",
            "config": {"workload": cfg.name, "grid": nd, "transform_grid": transform_grid(nd, gw, gc), "npw": len(gw),
                       "nv": cfg.nv, "nc_generated": cfg.nc,
                       "ncol": len(col), "explicit": n0, "windows": len(col) - n0, "ng": ng, "pairs": npair,
                       "q": list(cfg.qs[0]), "omega": 0.0, "e0_ev": cfg.e0_ev, "de_ev": cfg.de_ev,
                       "precision": head},
            "band_pairs_per_s": hr["band_pairs_per_s"], "modes": results, "roofline": roofline,
            "cpu_baseline": cpu, "mgo64_static_72cube": c2, "skipped": skipped or None,
            "run_s": time.time() - T_START}
    print(json.dumps(line))


def run_chunk(args, torch, synth, p, dev):
    """One conduction chunk of a configuration's shape for profiler and counter runs: random
    coefficient rows (the kernels' cost does not depend on their values), one build (or backward)
    per call, chunk overlap off so that every kernel runs on the context's stream."""
    if args.copy_calibration:
        x = torch.ones(1 << 28, dtype=torch.float32, device=dev)
        y = torch.empty_like(x)
        torch.mul(x, 2.0, out=y)
        torch.cuda.synchronize()
        log("copy calibration: 1 GiB read + 1 GiB written by one elementwise kernel")
        del x, y
    parts = args.chunk.split(":")
    cfg_i, mode, nv, ncol = int(parts[0]), parts[1], int(parts[2]), int(parts[3])
    backward = len(parts) > 4 and parts[4] == "backward"
    cfg = synth.config(cfg_i)
    gw = synth.wf_sphere(cfg.nd)
    gc = synth.chi_sphere(cfg.ng[0], cfg.qs[0], cfg.cell)
    g = torch.Generator(device=dev)
    g.manual_seed(1)
    cv = torch.randn((nv, len(gw)), dtype=torch.complex128, device=dev, generator=g) / np.sqrt(len(gw))
    cc = torch.randn((ncol, len(gw)), dtype=torch.complex128, device=dev, generator=g) / np.sqrt(len(gw))
    ev = torch.linspace(-0.4, -0.01, nv, dtype=torch.float64, device=dev)
    ec = torch.linspace(0.2, 2.0, ncol, dtype=torch.float64, device=dev)
    ctx = p.gw_ctx_create(0)
    p.gw_ctx_set_overlap(ctx, 0)
    geom = p.gw_geom_create(ctx, (cfg.nd,) * 3, gw, gc, cfg.cell, cfg.qs[0])
    prob = p.make_problem(geom, cv, ev, cc, ec)
    ng = len(gc)
    prec = p.PRECISIONS[mode]
    ws = torch.empty(p.gw_chi0_workspace_size(ctx, [prob], 1, prec), dtype=torch.uint8, device=dev)
    if backward:
        gb = torch.randn((1, ng, ng), dtype=torch.complex128, device=dev, generator=g)
        gb = (gb + gb.conj().transpose(1, 2)).contiguous()
    log(f"chunk: {cfg.name}, {mode}, {nv} x {ncol} pairs, NG {ng}, {'backward' if backward else 'build'}")
    for r in range(args.reps):
        t0 = time.time()
        if backward:
            p.gw_chi0_backward(ctx, [prob], [0.0], 0.0, prec, gb, workspace=ws)
        else:
            p.gw_chi0_build(ctx, [prob], [ng], [0.0], 0.0, prec, workspace=ws)
        torch.cuda.synchronize()
        log(f"call {r + 1}/{args.reps}: {time.time() - t0:.3f} s")
    p.gw_geom_destroy(geom)
    p.gw_ctx_destroy(ctx)


def run_c2_beside(args, torch, synth, p, dev, ctx):
    """The 64-atom workload (72^3, 128 x 4000, NG 2000, exact sum) in float64, float32 and
    split-BF16x3, a few timed steps each, errors against float64."""
    cfg = synth.config(1)
    nd = cfg.nd
    gw = synth.wf_sphere(nd)
    gc = synth.chi_sphere(cfg.ng[0], cfg.qs[0], cfg.cell)
    t0 = time.time()
    rows = synth.gaussian_columns_threaded(cfg.index, 0, np.arange(cfg.nv + cfg.nc), len(gw),
                                           max(1, min(16, len(os.sched_getaffinity(0)))))
    qd = synth.orthonormalize_on_device(rows, "cuda")
    del rows
    cv, cc = qd[:cfg.nv].contiguous(), qd[cfg.nv:].contiguous()
    del qd
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    ev, ec = t(synth.valence_energies(cfg, 0)), t(synth.conduction_energies(cfg))
    geom = p.gw_geom_create(ctx, (nd,) * 3, gw, gc, cfg.cell, cfg.qs[0])
    prob = p.make_problem(geom, cv, ev, cc, ec)
    ng = len(gc)
    vcoul = t(synth.coulomb(gc, cfg.qs[0], cfg.cell))
    k = 2 * int(np.abs(gc).max()) + 1
    npair = cfg.nv * cfg.nc
    fl = flops_model(transform_grid(nd, gw, gc), k, ng, npair, cfg.nv + cfg.nc)
    modes = ["fp64", "fp32", "bf16x3"]
    ws = torch.empty(max(p.gw_chi0_workspace_size(ctx, [prob], 1, p.PRECISIONS[m]) for m in modes), dtype=torch.uint8,
                     device=dev)
    ws_inv = torch.empty(p.gw_eps_inv_workspace_size(ctx, ng, 1), dtype=torch.uint8, device=dev)
    out = torch.empty(ng * ng, dtype=torch.complex128, device=dev)
    zout = torch.empty((ng, ng), dtype=torch.complex128, device=dev)
    log(f"72^3 workload beside: inputs in {time.time() - t0:.1f}s")
    steps = max(1, min(args.steps, 3))
    res, chis = {}, {}
    for m in modes:
        def run():
            p.gw_chi0_build(ctx, [prob], [ng], [0.0], 0.0, p.PRECISIONS[m], workspace=ws, out=out)
            p.gw_eps_inv(ctx, vcoul, out.view(ng, ng), workspace=ws_inv, out=zout, hermitian=True)
        ms, _, st, _ = timed_steps(p, ctx, torch, run, steps, 1, f"72^3 {m}")
        chis[m] = out.view(ng, ng).cpu().numpy()
        res[m] = {"ms_per_step": ms, "tflops": fl["total"] / (ms * 1e-3) / 1e12, "band_pairs_per_s": npair / (ms * 1e-3),
                  "stages_ms_per_step": st}
    ref = chis["fp64"]
    for m in modes:
        res[m]["err_vs_fp64"] = float(np.linalg.norm(chis[m] - ref) / np.linalg.norm(ref))
    p.gw_geom_destroy(geom)
    log("72^3: " + ", ".join(f"{m} {res[m]['ms_per_step']:.1f} ms" for m in modes))
    return {"workload": cfg.name, "steps": steps, "warmup": 1, "pairs": npair, "ng": ng, "modes": res}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--modes", default="fp64,fp32")
    ap.add_argument("--cpu-sample", type=int, default=16, help="valence bands in the oracle sample (0 = skip)")
    ap.add_argument("--cpu-cols", type=int, default=800)
    ap.add_argument("--tune", action="store_true", help="run the launch-shape tuner before timing each mode")
    ap.add_argument("--inputs-cache", default=None,
                    help="npz file for the generated inputs: loaded if present, written otherwise")
    ap.add_argument("--workload", default="headline",
                    choices=["headline", "static", "batched", "grouped", "adjoint", "grouping-study", "extensions",
                             "reduced-box", "chunk"],
                    help="headline (default): the 128^3 / 512 x 25000 grouped / NG 8000 build, mixed precision "
                         "with a float64 step and the 72^3 workload beside it; "
                         "static: the 72^3 / 128x4000 / NG 2000 build; batched: 8 q-points x 16 "
                         "frequencies, 128x6000 bands, NG 800..3000, one persistent launch per chunk; grouped: "
                         "96^3, 256 x 16000 bands grouped above 30 eV into 1 eV windows, NG 4000, with eps^-1; "
                         "adjoint: 128^3, 512 x 25000 bands grouped the same way, NG 8000, build + eps^-1 + "
                         "their adjoints down to the energy gradients; grouping-study: the 96^3 spectrum summed "
                         "exactly and grouped on several energy grids (accuracy and time against the exact sum); "
                         "extensions: the k-point sum, the static COH self-energy and the plasmon-pole "
                         "eps^-1(w); reduced-box: the static inputs with the stated 72^3 grid and with 48^3 "
                         "stated (both run on the smallest alias-free grid), beside the metric, never as it; chunk: "
                         "one conduction chunk of a configuration's shape (--chunk), a short driver for "
                         "profiler and counter runs, no JSON line")
    ap.add_argument("--grid", type=int, default=0,
                    help="grouped / adjoint workloads: FFT grid N^3 to run on instead of the stated one (an "
                         "alias-free smaller box gives the same chi0: 64 for the 96^3 workload, 96 for the "
                         "128^3 one); reported with reduced_box true, beside the metric, never as it")
    ap.add_argument("--no-reduced-box", action="store_true",
                    help="static workload: skip the extra head-mode steps on the 48^3 alias-free grid")
    ap.add_argument("--no-overlap", action="store_true",
                    help="run every conduction chunk's contraction on the context's stream (no second stream)")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="also run a plain 1 GiB read + 1 GiB write elementwise kernel (counter calibration)")
    ap.add_argument("--head-mode", default="bf16x3", choices=["bf16x3", "fp32", "fp64"],
                    help="headline workload: the precision of the timed steps")
    ap.add_argument("--no-fp64-step", action="store_true", help="headline workload: skip the float64 step")
    ap.add_argument("--no-c2", action="store_true", help="headline workload: skip the 72^3 workload beside it")
    ap.add_argument("--budget-s", type=float, default=540.0,
                    help="headline workload: wall-clock budget of the whole run; the legs beside the timed steps "
                         "(float64 step, oracle sample, 72^3 workload) are skipped when they would overrun it")
    ap.add_argument("--chunk", default="4:bf16x3:64:512",
                    help="chunk workload: CONFIG:MODE:NV:NCOL[:backward], configuration index (0..4), precision, "
                         "valence rows and columns (one chunk: NV x NCOL <= 32768 pairs), and the adjoint "
                         "instead of the build")
    ap.add_argument("--reps", type=int, default=1, help="chunk workload: calls")
    ap.add_argument("--cpu-pairs", default="8x160",
                    help="headline workload: oracle sample, valence x columns of the full-size workload")
    args = ap.parse_args()
    if args.gpus != 1:
        print(json.dumps({"error": "this benchmark runs on one GPU; --gpus must be 1 (the band sum shards over "
                                   "pairs, see the design notes)"}))
        sys.exit(2)

    import torch
    import synth
    import paper_1601_06767_amd as p

    dev = torch.device("cuda", 0)
    torch.cuda.set_device(dev)
    if args.workload == "headline":
        run_headline(args, torch, synth, p, dev)
        return
    if args.workload == "chunk":
        run_chunk(args, torch, synth, p, dev)
        return
    if args.workload == "batched":
        run_batched(args, torch, synth, p, dev)
        return
    if args.workload in ("grouped", "adjoint"):
        run_grouped(args, torch, synth, p, dev, args.workload == "adjoint")
        return
    if args.workload == "grouping-study":
        run_grouping_study(args, torch, synth, p, dev)
        return
    if args.workload == "extensions":
        run_extensions(args, torch, synth, p, dev)
        return
    if args.workload == "reduced-box":
        run_reduced_box(args, torch, synth, p, dev)
        return
    cfg = synth.config(1)
    nd = cfg.nd
    gw = synth.wf_sphere(nd)
    gc = synth.chi_sphere(cfg.ng[0], cfg.qs[0], cfg.cell)
    t0 = time.time()
    if args.inputs_cache and os.path.exists(args.inputs_cache):
        z = np.load(args.inputs_cache)
        bands = synth.Bands(z["coef_v"], z["e_v"], z["coef_c"], z["e_c"], z["v_index"], z["c_index"])
        log(f"inputs loaded from {args.inputs_cache}")
    else:
        bands = synth.make_bands(cfg, gvec_wf=gw, device="cuda")
        if args.inputs_cache:
            np.savez(args.inputs_cache, coef_v=bands.coef_v, e_v=bands.e_v, coef_c=bands.coef_c, e_c=bands.e_c,
                     v_index=bands.v_index, c_index=bands.c_index)
    log(f"inputs: npw={len(gw)} ng={len(gc)} nv={cfg.nv} nc={cfg.nc} ready in {time.time() - t0:.1f}s")

    ctx = p.gw_ctx_create(0)
    p.gw_ctx_set_overlap(ctx, 0 if args.no_overlap else 1)
    geom = p.gw_geom_create(ctx, (nd,) * 3, gw, gc, cfg.cell, cfg.qs[0])
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    cv, ev, cc, ec = t(bands.coef_v), t(bands.e_v), t(bands.coef_c), t(bands.e_c)
    prob = p.make_problem(geom, cv, ev, cc, ec)
    ng = len(gc)
    vcoul = t(synth.coulomb(gc, cfg.qs[0], cfg.cell))
    k = 2 * int(np.abs(gc).max()) + 1
    npair = cfg.nv * cfg.nc
    fl = flops_model(transform_grid(nd, gw, gc), k, ng, npair, cfg.nv + cfg.nc)
    modes = [m for m in args.modes.split(",") if m]
    wsb = max(p.gw_chi0_workspace_size(ctx, [prob], 1, p.PRECISIONS[m]) for m in modes)
    ws = torch.empty(wsb, dtype=torch.uint8, device=dev)
    ws_inv = torch.empty(p.gw_eps_inv_workspace_size(ctx, ng, 1), dtype=torch.uint8, device=dev)
    zout = torch.empty((ng, ng), dtype=torch.complex128, device=dev)
    log(f"workspace {wsb / 2**30:.2f} GiB")
    results = {}
    chis = {}
    stream = torch.cuda.current_stream()
    for m in modes:
        out = torch.empty(ng * ng, dtype=torch.complex128, device=dev)
        if args.tune:
            p.gw_tune(ctx, [prob], 1, p.PRECISIONS[m], workspace=ws)
            log(f"{m}: tuned (pair-kernel form, contraction splits) = {p.gw_tune_get(ctx, prob, p.PRECISIONS[m])}")

        def run():
            p.gw_chi0_build(ctx, [prob], [ng], [0.0], 0.0, p.PRECISIONS[m], workspace=ws, out=out)
            p.gw_eps_inv(ctx, vcoul, out.view(ng, ng), workspace=ws_inv, out=zout, hermitian=True)
        for _ in range(args.warmup):
            run()
        torch.cuda.synchronize()
        p.gw_ctx_stage_times(ctx, reset=True)
        p.gw_ctx_set_timing(ctx, True)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        tw = time.perf_counter()
        e0.record(stream)
        for i in range(args.steps):
            run()
            log(f"{m}: step {i + 1}/{args.steps} enqueued")
        e1.record(stream)
        torch.cuda.synchronize()
        wall = time.perf_counter() - tw
        p.gw_ctx_set_timing(ctx, False)
        stages = p.gw_ctx_stage_times(ctx, reset=True)
        ms = e0.elapsed_time(e1) / args.steps
        p.gw_eps_inv_status(ctx)
        chis[m] = out.view(ng, ng).cpu().numpy()
        zs = zout.cpu().numpy()
        results[m] = {"ms_per_step": ms, "wall_s": wall, "tflops": fl["total"] / (ms * 1e-3) / 1e12,
                      "band_pairs_per_s": npair / (ms * 1e-3),
                      "stages_ms_per_step": {s: v[0] / args.steps for s, v in stages.items() if v[1]},
                      "stage_launches_per_step": {s: v[1] / args.steps for s, v in stages.items() if v[1]},
                      "eps_inf": float(1.0 / zs[0, 0].real)}
        log(f"{m}: {ms:.1f} ms/step, {results[m]['tflops']:.2f} TFLOP/s, stages {results[m]['stages_ms_per_step']}")
    if "fp64" in chis:
        ref = chis["fp64"]
        nrm = np.linalg.norm(ref)
        for m in chis:
            results[m]["err_vs_fp64"] = float(np.linalg.norm(chis[m] - ref) / nrm)
        results["fp64"]["hermitian_residual"] = float(np.abs(ref - ref.conj().T).max() / np.abs(ref).max())

    head = modes[0]
    hr = results[head]
    # the head mode on the smallest supported alias-free grid (2 * 18 + 7 < 48): the same chi0
    # with less work, reported beside the metric (which stays on the stated grid)
    reduced = None
    if not args.no_reduced_box:
        geom_s = p.gw_geom_create(ctx, (48,) * 3, gw, gc)
        prob_s = p.make_problem(geom_s, cv, ev, cc, ec)
        need = p.gw_chi0_workspace_size(ctx, [prob_s], 1, p.PRECISIONS[head])
        ws_s = ws if need <= wsb else torch.empty(need, dtype=torch.uint8, device=dev)
        out_s = torch.empty(ng * ng, dtype=torch.complex128, device=dev)

        def run_s():
            p.gw_chi0_build(ctx, [prob_s], [ng], [0.0], 0.0, p.PRECISIONS[head], workspace=ws_s, out=out_s)
            p.gw_eps_inv(ctx, vcoul, out_s.view(ng, ng), workspace=ws_inv, out=zout, hermitian=True)
        for _ in range(max(1, args.warmup)):
            run_s()
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(stream)
        for _ in range(args.steps):
            run_s()
        e1.record(stream)
        torch.cuda.synchronize()
        p.gw_eps_inv_status(ctx)
        ms_s = e0.elapsed_time(e1) / args.steps
        chi_s = out_s.view(ng, ng).cpu().numpy()
        reduced = {"grid": 48, "mode": head, "ms_per_step": ms_s, "speedup_vs_stated_grid": hr["ms_per_step"] / ms_s,
                   "max_rel_diff_vs_stated_grid": float(np.abs(chi_s - chis[head]).max() / np.abs(chis[head]).max()),
                   "note": "same chi0 on the smallest supported alias-free grid; beside the metric, not it"}
        log(f"{head} on 48^3: {ms_s:.1f} ms/step ({reduced['speedup_vs_stated_grid']:.2f}x), "
            f"max rel diff {reduced['max_rel_diff_vs_stated_grid']:.1e}")
        p.gw_geom_destroy(geom_s)
        del ws_s, out_s
    # dominant kernel of the headline mode and its roofline
    st = hr["stages_ms_per_step"]
    dom = max(st, key=st.get)
    launches = hr["stage_launches_per_step"][dom]
    avg_ms = st[dom] / launches
    if dom == "contract":
        bound = "mfma"
        peak = {"fp64": PEAK["fp64_mfma"], "fp32": PEAK["fp32_mfma"], "bf16x3": PEAK["bf16_mfma"]}[head]
        work = fl["contract"] / launches
    else:
        bound, peak = "alu", (PEAK["fp64_vec"] if head == "fp64" else PEAK["fp32_vec_nopk"])
        work = fl[dom if dom in fl else "planes"] / launches
    achieved = work / (avg_ms * 1e-3) / 1e12
    roofline = {"bound": bound, "kernel": dom, "achieved": achieved, "peak": peak, "unit": "TFLOP/s",
                "frac": achieved / peak, "traffic": measured_traffic(dom, head), "avg_launch_ms": avg_ms,
                "algorithmic_work_per_launch": work}

    if args.copy_calibration:
        x = torch.ones(1 << 28, dtype=torch.float32, device=dev)
        y = torch.empty_like(x)
        torch.mul(x, 2.0, out=y)
        torch.cuda.synchronize()
        log("copy calibration: 1 GiB read + 1 GiB written by one elementwise kernel")
        del x, y

    cpu = None
    if args.cpu_sample > 0:
        import oracle
        cores = len(os.sched_getaffinity(0))
        vs = np.linspace(0, cfg.nv - 1, args.cpu_sample).astype(int)
        cs = np.arange(args.cpu_cols) * (cfg.nc // args.cpu_cols)
        t1 = time.perf_counter()
        ref = oracle.chi0_bands(bands.coef_v[vs], bands.e_v[vs], bands.coef_c[cs], bands.e_c[cs], gw, gc,
                                (nd,) * 3)[0]
        dt = time.perf_counter() - t1
        sp = len(vs) * len(cs)
        fs = flops_model(nd, k, ng, sp, len(vs) + len(cs), with_inverse=False)
        # the same sample through the GPU path
        sub = p.make_problem(geom, t(bands.coef_v[vs]), t(bands.e_v[vs]), t(bands.coef_c[cs]), t(bands.e_c[cs]))
        gchi = p.gw_chi0_build(ctx, [sub], [ng], [0.0], 0.0, p.GW_FP64)[0][0].cpu().numpy()
        cpu = {"value": (fs["total"] - fs["eps_inv"]) / dt / 1e12, "unit": "TFLOP/s", "cores": cores, "kind": "oracle",
               "band_pairs_per_s": sp / dt, "seconds": dt,
               "sample": f"{len(vs)} valence x {len(cs)} conduction bands ({sp} pairs) of the same workload, "
                         f"full grid and dielectric sphere, scipy.fft workers={cores}",
               "gpu_fp64_err_on_sample": float(np.linalg.norm(gchi - ref) / np.linalg.norm(ref))}
        log(f"oracle sample: {dt:.1f}s, {cpu['value'] * 1e3:.3f} GFLOP/s")

    line = {"metric": METRIC, "value": hr["tflops"], "unit": "TFLOP/s", "n_gpus": 1, "steps": args.steps,
            "warmup": args.warmup, "ms_per_step": hr["ms_per_step"], "higher_is_better": True, "scaling": "weak",
            "vs_baseline": None, "dtype": {"fp64": "f64", "fp32": "f32", "bf16x3": "bf16x3"}[head], "data": "synthetic",
            "config": {"workload": cfg.name, "grid": nd, "npw": len(gw), "nv": cfg.nv, "ncol": cfg.nc, "ng": ng,
                       "pairs": npair, "q": list(cfg.qs[0]), "omega": 0.0},
            "band_pairs_per_s": hr["band_pairs_per_s"], "modes": results, "roofline": roofline,
            "cpu_baseline": cpu, "reduced_box": reduced}
    print(json.dumps(line))


def run_batched(args, torch, synth, p, dev):
    """The batched frequency-dependent workload: every q-point is one problem of the same
    build call (uneven dielectric spheres), all frequencies with broadening in each call."""
    cfg = synth.config(3)
    nd = cfg.nd
    gw = synth.wf_sphere(nd)
    om = synth.omegas(cfg)
    delta = synth.delta(cfg)
    t0 = time.time()
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    ctx = p.gw_ctx_create(0)
    p.gw_ctx_set_overlap(ctx, 0 if args.no_overlap else 1)
    probs, ngs, keep = [], [], []
    cc = ec = None
    for iq in range(len(cfg.qs)):
        gc = synth.chi_sphere(cfg.ng[iq], cfg.qs[iq], cfg.cell)
        b = synth.make_bands(cfg, gvec_wf=gw, iq=iq, device="cuda")
        if cc is None:   # the conduction set (at k) is the same for every q-point
            cc, ec = t(b.coef_c), t(b.e_c)
        geom = p.gw_geom_create(ctx, (nd,) * 3, gw, gc, cfg.cell, cfg.qs[iq])
        cv, ev = t(b.coef_v), t(b.e_v)
        keep += [cv, ev]
        probs.append(p.make_problem(geom, cv, ev, cc, ec))
        ngs.append(len(gc))
        del b
    log(f"batched inputs: {len(probs)} q-points, NG {ngs}, {len(om)} frequencies, ready in {time.time() - t0:.1f}s")
    modes = [m for m in args.modes.split(",") if m]
    npair = cfg.nv * cfg.nc
    k = [2 * int(np.abs(synth.chi_sphere(n, q, cfg.cell)).max()) + 1 for n, q in zip(cfg.ng, cfg.qs)]
    work = {"planes": 0.0, "finish": 0.0, "contract": 0.0, "band": 0.0}
    for n, kk in zip(ngs, k):
        # the spheres of nd // 4 and (kk - 1) / 2 on their transform grid
        f = flops_model(transform_grid(nd, np.array([nd // 4]), np.array([(kk - 1) // 2])), kk, n, npair, cfg.nv + cfg.nc, with_inverse=False)
        work["planes"] += f["planes"]
        work["finish"] += f["finish"]
        work["band"] += f["band"]
        work["contract"] += 2.0 * f["contract"] * len(om)     # 8 NG^2 per pair per frequency
    total = sum(work.values())
    results = {}
    for m in modes:
        wsb = p.gw_chi0_workspace_size(ctx, probs, len(om), p.PRECISIONS[m])
        ws = torch.empty(wsb, dtype=torch.uint8, device=dev)
        out = torch.empty(sum(len(om) * n * n for n in ngs), dtype=torch.complex128, device=dev)
        log(f"{m}: workspace {wsb / 2**30:.1f} GiB")

        def run():
            p.gw_chi0_build(ctx, probs, ngs, om, delta, p.PRECISIONS[m], workspace=ws, out=out)
        for _ in range(args.warmup):
            run()
        torch.cuda.synchronize()
        p.gw_ctx_stage_times(ctx, reset=True)
        p.gw_ctx_set_timing(ctx, True)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        e0.record(torch.cuda.current_stream())
        for i in range(args.steps):
            run()
            log(f"{m}: step {i + 1}/{args.steps} enqueued")
        e1.record(torch.cuda.current_stream())
        torch.cuda.synchronize()
        p.gw_ctx_set_timing(ctx, False)
        stages = p.gw_ctx_stage_times(ctx, reset=True)
        ms = e0.elapsed_time(e1) / args.steps
        st = {s_: v[0] / args.steps for s_, v in stages.items() if v[1]}
        nl = {s_: v[1] / args.steps for s_, v in stages.items() if v[1]}
        results[m] = {"ms_per_step": ms, "tflops": total / (ms * 1e-3) / 1e12,
                      "band_pairs_per_s": npair * len(ngs) / (ms * 1e-3), "stages_ms_per_step": st,
                      "stage_launches_per_step": nl,
                      "contract_tflops": work["contract"] / (st.get("contract", ms) * 1e-3) / 1e12}
        log(f"{m}: {ms:.1f} ms/step, {results[m]['tflops']:.2f} TFLOP/s, stages {st}")
        del ws, out
    head = modes[0]
    hr = results[head]
    st = hr["stages_ms_per_step"]
    peak = PEAK["fp64_mfma"] if head == "fp64" else PEAK["fp32_mfma"] if head == "fp32" else PEAK["bf16_mfma"]
    avg = st["contract"] / hr["stage_launches_per_step"]["contract"]
    per = work["contract"] / hr["stage_launches_per_step"]["contract"]
    roofline = {"bound": "mfma", "kernel": "contract", "achieved": per / (avg * 1e-3) / 1e12, "peak": peak,
                "unit": "TFLOP/s", "frac": per / (avg * 1e-3) / 1e12 / peak, "traffic": None, "avg_launch_ms": avg,
                "algorithmic_work_per_launch": per}
    line = {"metric": METRIC, "value": hr["tflops"], "unit": "TFLOP/s", "n_gpus": 1, "steps": args.steps,
            "warmup": args.warmup, "ms_per_step": hr["ms_per_step"], "higher_is_better": True, "scaling": "weak",
            "vs_baseline": None, "dtype": {"fp64": "f64", "fp32": "f32", "bf16x3": "bf16x3"}[head],
            "data": "synthetic",
            "config": {"workload": cfg.name, "grid": nd, "npw": len(gw), "nv": cfg.nv, "ncol": cfg.nc, "ng": ngs,
                       "pairs_per_q": npair, "q": [list(q) for q in cfg.qs], "omegas": len(om),
                       "delta_ev": cfg.delta_ev},
            "band_pairs_per_s": hr["band_pairs_per_s"], "modes": results, "roofline": roofline,
            "cpu_baseline": None}
    print(json.dumps(line))


def make_bands_logged(synth, cfg, c_index, gw, e_all):
    """synth.make_bands (q = 0) in steps that each report progress: the Gaussian rows in
    blocks of bands, then the orthonormalisation on the GPU."""
    npw = len(gw)
    bands_idx = np.concatenate([np.arange(cfg.nv), cfg.nv + np.asarray(c_index)])
    rows = np.empty((len(bands_idx), npw), dtype=np.complex128)
    for b0 in range(0, len(bands_idx), 1024):
        rows[b0:b0 + 1024] = synth.gaussian_columns(cfg.index, 0, bands_idx[b0:b0 + 1024], npw)
        log(f"  coefficient rows {min(b0 + 1024, len(bands_idx))}/{len(bands_idx)}")
    q = synth.orthonormalize(rows, "cuda")
    del rows
    log("  orthonormalised")
    ev = synth.valence_energies(cfg, 0)
    return synth.Bands(q[:cfg.nv], ev[:cfg.nv], q[cfg.nv:], e_all[np.asarray(c_index)], np.arange(cfg.nv),
                       np.asarray(c_index))


def run_grouped(args, torch, synth, p, dev, backward):
    """The grouped workloads (Eq. (energyintegration)): explicit bands up to E0 = 30 eV and
    one representative per 1 eV window above, static.  With backward, one step is also the
    adjoint of L = Re sum over the 27-G head block of eps^-1: gw_eps_inv_backward, then
    gw_chi0_backward down to dL/dE_v, dL/dE_col and dL/dn_col (the pair densities are
    recomputed)."""
    cfg = synth.config(4 if backward else 2)
    nd = args.grid or cfg.nd   # FFT grid; the spheres stay those of the stated grid
    ev_ = synth.HARTREE_EV
    gw = synth.wf_sphere(cfg.nd)
    gc = synth.chi_sphere(cfg.ng[0], cfg.qs[0], cfg.cell)
    e_all = synth.conduction_energies(cfg)
    nwin = int(round((cfg.emax_ev - cfg.e0_ev) / cfg.de_ev))
    col, e_col, n_col, n0 = p.gw_group_windows(e_all, cfg.e0_ev / ev_, cfg.de_ev / ev_, nwin)
    t0 = time.time()
    bands = make_bands_logged(synth, cfg, col, gw, e_all)
    log(f"grouped inputs: {nd}^3, npw={len(gw)}, nv={cfg.nv}, {cfg.nc} bands -> {len(col)} columns "
        f"({n0} explicit + {len(col) - n0} windows), NG={len(gc)}, ready in {time.time() - t0:.1f}s")
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    ctx = p.gw_ctx_create(0)
    p.gw_ctx_set_overlap(ctx, 0 if args.no_overlap else 1)
    geom = p.gw_geom_create(ctx, (nd,) * 3, gw, gc, cfg.cell, cfg.qs[0])
    cv, ev, cc = t(bands.coef_v), t(bands.e_v), t(bands.coef_c)
    del bands
    ecol, ncol = t(e_col), t(n_col)
    prob = p.make_problem(geom, cv, ev, cc, ecol, ncol)
    ng = len(gc)
    vcoul = t(synth.coulomb(gc, cfg.qs[0], cfg.cell))
    head = torch.from_numpy(synth.loss_head_block(gc)).to(dev)
    k = 2 * int(np.abs(gc).max()) + 1
    npair = cfg.nv * len(col)
    fl = flops_model(transform_grid(nd, gw, gc), k, ng, npair, cfg.nv + len(col))
    # the adjoint recomputes the pair densities and forms Y = M L^T, L a lower triangle (4 NG^2 per pair),
    # and Zbar -> chi0bar (two NG^3 complex products, 16 NG^3)
    bw = fl["planes"] + fl["finish"] + fl["band"] + fl["contract"] + 2.0 * fl["eps_inv"] if backward else 0.0
    modes = [m for m in args.modes.split(",") if m]
    wsb = max(p.gw_chi0_workspace_size(ctx, [prob], 1, p.PRECISIONS[m]) for m in modes)
    ws = torch.empty(wsb, dtype=torch.uint8, device=dev)
    ws_inv = torch.empty(p.gw_eps_inv_workspace_size(ctx, ng, 1), dtype=torch.uint8, device=dev)
    zout = torch.empty((ng, ng), dtype=torch.complex128, device=dev)
    zbar = torch.zeros((ng, ng), dtype=torch.complex128, device=dev)
    zbar[head, head] = 1.0
    gchi = torch.empty((ng, ng), dtype=torch.complex128, device=dev)
    log(f"workspace {wsb / 2**30:.1f} GiB")
    stream = torch.cuda.current_stream()
    results, chis, grads = {}, {}, {}
    for m in modes:
        out = torch.empty(ng * ng, dtype=torch.complex128, device=dev)
        g = [None, None, None]
        if args.tune:
            p.gw_tune(ctx, [prob], 1, p.PRECISIONS[m], workspace=ws)
            log(f"{m}: tuned (pair-kernel form, contraction splits) = {p.gw_tune_get(ctx, prob, p.PRECISIONS[m])}")

        def run():
            p.gw_chi0_build(ctx, [prob], [ng], [0.0], 0.0, p.PRECISIONS[m], workspace=ws, out=out)
            p.gw_eps_inv(ctx, vcoul, out.view(ng, ng), workspace=ws_inv, out=zout, hermitian=True)
            if backward:
                p.gw_eps_inv_backward(ctx, vcoul, zout, zbar, workspace=ws_inv, out=gchi)
                g[:] = p.gw_chi0_backward(ctx, [prob], [0.0], 0.0, p.PRECISIONS[m], gchi.view(1, ng, ng),
                                          workspace=ws)
        for _ in range(args.warmup):
            run()
        torch.cuda.synchronize()
        p.gw_ctx_stage_times(ctx, reset=True)
        p.gw_ctx_set_timing(ctx, True)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        e0.record(stream)
        for i in range(args.steps):
            run()
            log(f"{m}: step {i + 1}/{args.steps} enqueued")
        e1.record(stream)
        torch.cuda.synchronize()
        p.gw_ctx_set_timing(ctx, False)
        stages = p.gw_ctx_stage_times(ctx, reset=True)
        ms = e0.elapsed_time(e1) / args.steps
        p.gw_eps_inv_status(ctx)
        chis[m] = out.view(ng, ng).cpu().numpy()
        if backward:
            grads[m] = [x.cpu().numpy() for x in g]
        results[m] = {"ms_per_step": ms, "tflops": (fl["total"] + bw) / (ms * 1e-3) / 1e12,
                      "band_pairs_per_s": npair / (ms * 1e-3),
                      "stages_ms_per_step": {s_: v[0] / args.steps for s_, v in stages.items() if v[1]},
                      "stage_launches_per_step": {s_: v[1] / args.steps for s_, v in stages.items() if v[1]},
                      "eps_inf": float(1.0 / zout[0, 0].real.item())}
        log(f"{m}: {ms:.1f} ms/step, {results[m]['tflops']:.2f} TFLOP/s, stages {results[m]['stages_ms_per_step']}")
        del out
    if "fp64" in chis:
        ref = chis["fp64"]
        nrm = np.linalg.norm(ref)
        for m in chis:
            results[m]["err_vs_fp64"] = float(np.linalg.norm(chis[m] - ref) / nrm)
            if backward:
                results[m]["grad_err_vs_fp64"] = [float(np.abs(a - b).max() / np.abs(b).max())
                                                  for a, b in zip(grads[m], grads["fp64"])]
    head_m = modes[0]
    hr = results[head_m]
    st = hr["stages_ms_per_step"]
    launches = hr["stage_launches_per_step"]["contract"]
    avg = st["contract"] / launches
    per = fl["contract"] / launches
    peak = PEAK["fp64_mfma"] if head_m == "fp64" else PEAK["fp32_mfma"] if head_m == "fp32" else PEAK["bf16_mfma"]
    roofline = {"bound": "mfma", "kernel": "contract", "achieved": per / (avg * 1e-3) / 1e12, "peak": peak,
                "unit": "TFLOP/s", "frac": per / (avg * 1e-3) / 1e12 / peak, "traffic": None, "avg_launch_ms": avg,
                "algorithmic_work_per_launch": per}
    line = {"metric": METRIC, "value": hr["tflops"], "unit": "TFLOP/s", "n_gpus": 1, "steps": args.steps,
            "warmup": args.warmup, "ms_per_step": hr["ms_per_step"], "higher_is_better": True, "scaling": "weak",
            "vs_baseline": None, "dtype": {"fp64": "f64", "fp32": "f32", "bf16x3": "bf16x3"}[head_m],
            "data": "synthetic",
            "config": {"workload": cfg.name + ("-with-adjoint" if backward else ""), "grid": nd,
                       "reduced_box": nd != cfg.nd, "npw": len(gw),
                       "nv": cfg.nv, "nc_generated": cfg.nc, "ncol": len(col), "explicit": n0, "ng": ng,
                       "pairs": npair, "q": list(cfg.qs[0]), "omega": 0.0, "e0_ev": cfg.e0_ev, "de_ev": cfg.de_ev},
            "band_pairs_per_s": hr["band_pairs_per_s"], "modes": results, "roofline": roofline,
            "cpu_baseline": None}
    print(json.dumps(line))


def run_grouping_study(args, torch, synth, p, dev):
    """Accuracy and cost of the energy integration (Eqs. (chi02), (energyintegration)) on the
    96^3 spectrum (256 valence, 16,000 conduction bands with density ~ sqrt(E) on 5..60 eV,
    NG 4000): chi0 of the exact band sum against grouped sums above E0 = 30 eV on uniform
    grids of dE = 1..5 eV (band-count weights), with density weights g(E) dE under the
    midpoint and the two-point Gauss rule, on two nonuniform grids (geometric windows;
    windows of equal band count), and with E0 lowered to 20, 15 and 10 eV.  Per grid: N0 + N_E, the paper's speed-up N_c / (N0 + N_E),
    the measured build-time ratio, ||chi_grp - chi_exact||_F / ||chi_exact||_F, the change
    of L = Re sum over the 27-G head block of eps^-1, and the static COH self-energy of the
    band-edge states (Eq. (sigmach), the same grouping over all bands) with its gap term
    Sigma_cb - Sigma_vb against the exact sum."""
    cfg = synth.config(2)
    nd = cfg.nd
    hev = synth.HARTREE_EV
    gw = synth.wf_sphere(nd)
    gc = synth.chi_sphere(cfg.ng[0], cfg.qs[0], cfg.cell)
    e_all = synth.conduction_energies(cfg)
    t0 = time.time()
    bands = make_bands_logged(synth, cfg, np.arange(cfg.nc), gw, e_all)
    log(f"study inputs: {nd}^3, npw={len(gw)}, nv={cfg.nv}, nc={cfg.nc}, NG={len(gc)}, ready in "
        f"{time.time() - t0:.1f}s")
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    ctx = p.gw_ctx_create(0)
    geom = p.gw_geom_create(ctx, (nd,) * 3, gw, gc, cfg.cell, cfg.qs[0])
    cv, ev, cc = t(bands.coef_v), t(bands.e_v), t(bands.coef_c)
    del bands
    ng = len(gc)
    vcoul = t(synth.coulomb(gc, cfg.qs[0], cfg.cell))
    head = torch.from_numpy(synth.loss_head_block(gc)).to(dev)
    mode = [m for m in args.modes.split(",") if m][0]
    prec = p.PRECISIONS[mode]
    e0 = cfg.e0_ev / hev
    top = cfg.emax_ev / hev
    # density of the generator's spectrum, dN/dE = A sqrt(E) (A per Hartree^(3/2))
    dos_a = 1.5 * cfg.nc / (cfg.emax_ev ** 1.5 - 5.0 ** 1.5) * hev ** 1.5
    above = np.sort(e_all[e_all > e0])
    grids = [(f"uniform dE={de:g} eV, counts", np.append(np.arange(e0, top - 1e-12, de / hev), top), 0, 0)
             for de in (1.0, 1.5, 2.0, 2.5, 3.0, 3.5, 4.0, 5.0)]
    for de in (2.0, 4.0):
        edges = np.append(np.arange(e0, top - 1e-12, de / hev), top)
        grids.append((f"uniform dE={de:g} eV, g(E) dE midpoint", edges, 1, 0))
        grids.append((f"uniform dE={de:g} eV, g(E) dE two-point Gauss", edges, 1, 1))
    geo = [e0]
    while geo[-1] < top:
        geo.append(geo[-1] + (0.5 / hev) * 1.15 ** (len(geo) - 1))
    geo[-1] = top
    grids.append(("geometric dE 0.5 eV x 1.15^i, counts", np.array(geo), 0, 0))
    q = np.quantile(above, np.linspace(0.0, 1.0, 31)[1:-1])
    grids.append(("30 windows of equal band count, counts", np.concatenate([[e0], q, [top]]), 0, 0))
    for e0_ev in (20.0, 15.0, 10.0):   # fewer explicit bands: the regime of the paper's N0 = 8 per atom
        grids.append((f"E0={e0_ev:g} eV, uniform dE=2 eV, counts",
                      np.append(np.arange(e0_ev / hev, top - 1e-12, 2.0 / hev), top), 0, 0))

    ws = torch.empty(p.gw_chi0_workspace_size(ctx, [p.make_problem(geom, cv, ev, cc, t(e_all))], 1, prec),
                     dtype=torch.uint8, device=dev)
    ws_inv = torch.empty(p.gw_eps_inv_workspace_size(ctx, ng, 1), dtype=torch.uint8, device=dev)
    out = torch.empty(ng * ng, dtype=torch.complex128, device=dev)
    z = torch.empty((ng, ng), dtype=torch.complex128, device=dev)

    def build(prob):
        torch.cuda.synchronize()
        a = time.perf_counter()
        p.gw_chi0_build(ctx, [prob], [ng], [0.0], 0.0, prec, workspace=ws, out=out)
        torch.cuda.synchronize()
        dt = time.perf_counter() - a
        p.gw_eps_inv(ctx, vcoul, out.view(ng, ng), workspace=ws_inv, out=z, hermitian=True)
        p.gw_eps_inv_status(ctx)
        return dt, out.view(ng, ng).clone(), float(z[head, head].real.sum().item())

    # static COH self-energy of the 4 highest valence and 4 lowest conduction states over
    # every valence band plus the conduction columns (the same grouping, Eq. (sigmach))
    call = torch.cat([cv, cc])
    states = torch.cat([cv[cfg.nv - 4:], cc[:4]]).contiguous()
    st_e = t(np.zeros(8))

    def coh(col, n_col):
        cols = np.concatenate([np.arange(cfg.nv), cfg.nv + np.asarray(col)]).astype(np.int32)
        w = np.concatenate([np.ones(cfg.nv), n_col])
        prob = p.make_problem(geom, states, st_e, call, t(np.zeros(len(cols))), t(w), t(cols))
        torch.cuda.synchronize()
        a = time.perf_counter()
        s_ = p.gw_sigma_coh_static(ctx, prob, vcoul, z)
        torch.cuda.synchronize()
        return time.perf_counter() - a, s_.cpu().numpy()

    exact_prob = p.make_problem(geom, cv, ev, cc, t(e_all))
    build(exact_prob)   # warm-up
    t_ex, chi_ex, l_ex = build(exact_prob)
    tc_ex, s_ex = coh(np.arange(cfg.nc), np.ones(cfg.nc))
    gap_ex = float((s_ex[4, 4].real - s_ex[3, 3].real) * hev)
    nrm = float(torch.linalg.norm(chi_ex).item())
    log(f"exact: {cfg.nc} columns, {t_ex:.2f} s, L = {l_ex:.6f}; COH {tc_ex:.2f} s, "
        f"Sigma_cb - Sigma_vb = {gap_ex:.4f} eV")
    rows = [{"grid": "exact band sum", "columns": cfg.nc, "explicit": cfg.nc, "speedup_predicted": 1.0,
             "build_s": t_ex, "speedup_measured": 1.0, "chi_rel_err": 0.0, "head_trace": l_ex, "head_trace_rel": 0.0,
             "coh_s": tc_ex, "coh_gap_ev": gap_ex, "coh_gap_shift_ev": 0.0, "coh_rel_err": 0.0}]
    for name, edges, md, rule in grids:
        col, e_col, n_col, n0 = p.gw_group_windows_edges(e_all, edges, md, rule, dos_a, 0.0)
        prob = p.make_problem(geom, cv, ev, cc, t(e_col), t(n_col), t(col))
        dt, chi, l_g = build(prob)
        err = float(torch.linalg.norm(chi - chi_ex).item()) / nrm
        tc, s_g = coh(col, n_col)
        gap = float((s_g[4, 4].real - s_g[3, 3].real) * hev)
        row = {"grid": name, "columns": len(col), "explicit": n0, "speedup_predicted": cfg.nc / len(col),
               "build_s": dt, "speedup_measured": t_ex / dt, "chi_rel_err": err, "head_trace": l_g,
               "head_trace_rel": (l_g - l_ex) / abs(l_ex), "coh_s": tc, "coh_gap_ev": gap,
               "coh_gap_shift_ev": gap - gap_ex,
               "coh_rel_err": float(np.linalg.norm(s_g - s_ex) / np.linalg.norm(s_ex))}
        rows.append(row)
        log(f"{name}: {len(col)} columns ({n0} explicit), {dt:.2f} s, speed-up {t_ex / dt:.2f} "
            f"(N_c/(N0+N_E) = {cfg.nc / len(col):.2f}), chi err {err:.3e}, L rel {row['head_trace_rel']:+.3e}, "
            f"COH {tc:.2f} s, gap shift {gap - gap_ex:+.4f} eV, Sigma err {row['coh_rel_err']:.3e}")
    print(json.dumps({"metric": METRIC, "workload": "grouping-study-" + cfg.name, "dtype": mode,
                      "data": "synthetic", "grid": nd, "nv": cfg.nv, "nc": cfg.nc, "ng": ng, "e0_ev": cfg.e0_ev,
                      "rows": rows}))


def run_reduced_box(args, torch, synth, p, dev):
    """The static 72^3 workload's inputs built on the stated grid and on 48^3.  The product
    of two bands of the wavefunction sphere (|n| <= 18 per axis) has components up to 36, so
    with the chi sphere's |n| <= 7 every grid with N > 43 gives the same pair densities
    (Eq. (chi0)'s sum over r is exact on any grid where the product is unaliased on the
    chi sphere).  The metric stays on the stated grid; this line reports the time a smaller
    box saves and the difference of the two results."""
    cfg = synth.config(1)
    gw = synth.wf_sphere(cfg.nd)
    gc = synth.chi_sphere(cfg.ng[0], cfg.qs[0], cfg.cell)
    t0 = time.time()
    if args.inputs_cache and os.path.exists(args.inputs_cache):
        z = np.load(args.inputs_cache)
        bands = synth.Bands(z["coef_v"], z["e_v"], z["coef_c"], z["e_c"], z["v_index"], z["c_index"])
    else:
        bands = synth.make_bands(cfg, gvec_wf=gw, device="cuda")
    log(f"inputs ready in {time.time() - t0:.1f}s")
    ctx = p.gw_ctx_create(0)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    cv, ev, cc, ec = t(bands.coef_v), t(bands.e_v), t(bands.coef_c), t(bands.e_c)
    ng = len(gc)
    vcoul = t(synth.coulomb(gc, cfg.qs[0], cfg.cell))
    ws_inv = torch.empty(p.gw_eps_inv_workspace_size(ctx, ng, 1), dtype=torch.uint8, device=dev)
    zout = torch.empty((ng, ng), dtype=torch.complex128, device=dev)
    stream = torch.cuda.current_stream()
    modes = [m for m in args.modes.split(",") if m]
    res = {}
    for m in modes:
        res[m] = {}
        chis = {}
        for nd in (cfg.nd, 48):
            geom = p.gw_geom_create(ctx, (nd,) * 3, gw, gc, cfg.cell, cfg.qs[0])
            prob = p.make_problem(geom, cv, ev, cc, ec)
            ws = torch.empty(p.gw_chi0_workspace_size(ctx, [prob], 1, p.PRECISIONS[m]), dtype=torch.uint8, device=dev)
            out = torch.empty(ng * ng, dtype=torch.complex128, device=dev)

            def run():
                p.gw_chi0_build(ctx, [prob], [ng], [0.0], 0.0, p.PRECISIONS[m], workspace=ws, out=out)
                p.gw_eps_inv(ctx, vcoul, out.view(ng, ng), workspace=ws_inv, out=zout, hermitian=True)
            for _ in range(max(1, args.warmup)):
                run()
            torch.cuda.synchronize()
            p.gw_ctx_stage_times(ctx, reset=True)
            p.gw_ctx_set_timing(ctx, True)
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record(stream)
            for _ in range(args.steps):
                run()
            e1.record(stream)
            torch.cuda.synchronize()
            p.gw_ctx_set_timing(ctx, False)
            st = p.gw_ctx_stage_times(ctx, reset=True)
            p.gw_eps_inv_status(ctx)
            ms = e0.elapsed_time(e1) / args.steps
            chis[nd] = out.view(ng, ng).cpu().numpy()
            res[m][f"{nd}^3"] = {"ms_per_step": ms, "band_pairs_per_s": cfg.nv * cfg.nc / (ms * 1e-3),
                                 "stages_ms_per_step": {s: v[0] / args.steps for s, v in st.items() if v[1]}}
            log(f"{m} {nd}^3: {ms:.1f} ms/step, stages {res[m][f'{nd}^3']['stages_ms_per_step']}")
            p.gw_geom_destroy(geom)
            del ws, out
        a, b = chis[cfg.nd], chis[48]
        res[m]["speedup"] = res[m][f"{cfg.nd}^3"]["ms_per_step"] / res[m]["48^3"]["ms_per_step"]
        res[m]["rel_diff_48_vs_72"] = float(np.abs(a - b).max() / np.abs(a).max())
    print(json.dumps({"metric": METRIC, "workload": "reduced-box", "data": "synthetic",
                      "config": {"workload": cfg.name, "grids": [cfg.nd, 48], "ng": ng, "pairs": cfg.nv * cfg.nc,
                                 "alias_free_min": int(2 * np.abs(gw).max() + np.abs(gc).max() + 1)},
                      "results": res}))


def run_extensions(args, torch, synth, p, dev):
    """Throughput of the paths beside the band sum, each on inputs shaped like the 72^3 /
    NG 2000 workload: (1) the k-point sum of Eq. (chi0) on a 2x2x2 grid (q = (1/2, 0, 0), 128
    valence x 500 conduction bands per k: 512,000 pairs as in the static workload), (2) the
    static COH self-energy of 8 band-edge states over 128 + 4,000 bands, (3) the plasmon-pole
    eps^-1(w) at NG 8000 for 16 frequencies (reads eps^-1(0) once, writes every frequency)."""
    ctx = p.gw_ctx_create(0)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    mode = [m for m in args.modes.split(",") if m][0]
    prec = p.PRECISIONS[mode]
    out = {}

    def timed(fn, reps=None):
        reps = reps or max(1, args.steps)
        for _ in range(args.warmup):
            fn()
        torch.cuda.synchronize()
        a = time.perf_counter()
        for _ in range(reps):
            r = fn()
        torch.cuda.synchronize()
        return (time.perf_counter() - a) / reps, r

    # (1) k-point sum
    cfg = synth.config(1)
    kp = synth.kpoint_grid(2)
    q = (0.5, 0.0, 0.0)
    t0 = time.time()
    kb = synth.make_kbands(11, kp, cfg.nd / 4.0, 128, 500)
    gc = synth.chi_sphere(cfg.ng[0], q, cfg.cell)
    idx, g0 = p.gw_kq_map(kp, q)
    # valence rows relabelled to k + q (entry g holds c_{v,k''}(g + G0)): one geometry and
    # the dielectric sphere's own width
    u = np.unique(np.concatenate(list(kb.gw) + [kb.gw[idx[k]] - g0[k] for k in range(len(kp))]), axis=0)
    u = np.ascontiguousarray(u[np.lexsort((u[:, 2], u[:, 1], u[:, 0], (u * u).sum(1)))].astype(np.int32))
    pos = {tuple(x): i for i, x in enumerate(u.tolist())}

    def embed(rows, gw):
        e = np.zeros((rows.shape[0], len(u)), dtype=np.complex128)
        e[:, [pos[tuple(x)] for x in gw.tolist()]] = rows
        return e
    geoms = {(): p.gw_geom_create(ctx, (cfg.nd,) * 3, u, gc)}
    probs = []
    for k in range(len(kp)):
        kk = idx[k]
        probs.append(p.make_problem(geoms[()], t(embed(kb.coef_v[kk], kb.gw[kk] - g0[k])), t(kb.e_v[kk]),
                                    t(embed(kb.coef_c[k], kb.gw[k])), t(kb.e_c[k])))
    log(f"k-point inputs: {len(kp)} k, union sphere {len(u)}, NG {len(gc)}, ready in {time.time() - t0:.1f}s")
    ws = torch.empty(p.gw_chi0_workspace_size(ctx, probs, 1, prec), dtype=torch.uint8, device=dev)
    chi = torch.empty((1, len(gc), len(gc)), dtype=torch.complex128, device=dev)
    dt, _ = timed(lambda: p.gw_chi0_build_ksum(ctx, probs, len(gc), [0.0], 0.0, prec, workspace=ws, out=chi))
    k = 2 * int(np.abs(gc).max()) + 1
    npair = 128 * 500 * len(kp)
    fl = flops_model(transform_grid(cfg.nd, u, gc), k, len(gc), npair, len(kp) * 628, with_inverse=False)
    out["ksum"] = {"k_points": len(kp), "pairs": npair, "ng": len(gc), "seconds": dt,
                   "tflops": fl["total"] / dt / 1e12, "band_pairs_per_s": npair / dt}
    log(f"k-point sum: {dt * 1e3:.1f} ms, {out['ksum']['tflops']:.2f} TFLOP/s")
    del ws, chi, probs
    for gm in geoms.values():
        p.gw_geom_destroy(gm)

    # (2) static COH of 8 band-edge states over every band of the static workload
    gw = synth.wf_sphere(cfg.nd)
    gc0 = synth.chi_sphere(cfg.ng[0], cfg.qs[0], cfg.cell)
    bands = synth.make_bands(cfg, gvec_wf=gw, device="cuda")
    geom = p.gw_geom_create(ctx, (cfg.nd,) * 3, gw, gc0)
    cv, cc = t(bands.coef_v), t(bands.coef_c)
    ng = len(gc0)
    prob = p.make_problem(geom, cv, t(bands.e_v), cc, t(bands.e_c))
    chi0 = p.gw_chi0_build(ctx, [prob], [ng], [0.0], 0.0, p.GW_FP64)[0][0]
    vc = t(synth.coulomb(gc0, cfg.qs[0], cfg.cell))
    z = p.gw_eps_inv(ctx, vc, chi0, hermitian=True)
    call = torch.cat([cv, cc])
    states = torch.cat([cv[-4:], cc[:4]]).contiguous()
    ncols = cfg.nv + cfg.nc
    sprob = p.make_problem(geom, states, t(np.zeros(8)), call, t(np.zeros(ncols)))
    sws = torch.empty(p.gw_sigma_coh_workspace_size(ctx, sprob), dtype=torch.uint8, device=dev)
    dt, _ = timed(lambda: p.gw_sigma_coh_static(ctx, sprob, vc, z, workspace=sws))
    ngp = (ng + 127) // 128 * 128
    gemm = 8.0 * ngp * ngp * 8 * ncols
    out["sigma_coh_static"] = {"states": 8, "columns": ncols, "ng": ng, "seconds": dt,
                               "gemm_tflops": gemm / dt / 1e12}
    log(f"static COH: {dt * 1e3:.1f} ms for 8 states x {ncols} columns ({gemm / dt / 1e12:.1f} TFLOP/s of GEMM)")
    del sws, call, cv, cc, bands

    # (3) plasmon-pole eps^-1(w) at NG 8000
    c5 = synth.config(4)
    gc5 = synth.chi_sphere(c5.ng[0], c5.qs[0], c5.cell)
    n5 = len(gc5)
    rz = np.random.default_rng(5)
    z5 = torch.eye(n5, dtype=torch.complex128, device=dev) * 0.8
    z5 += 0.01 * torch.from_numpy(rz.standard_normal((n5, n5))).to(dev)
    half = int((gc5.max(0) - gc5.min(0)).max())
    box = t(synth.density_box(half, c5.cell, 2.0 * c5.nv))
    om = np.linspace(0.0, 40.0, 16) / synth.HARTREE_EV
    b5 = synth.recip(c5.cell)
    dt, _ = timed(lambda: p.gw_gpp_eps_inv(ctx, gc5, c5.qs[0], b5, box, z5, om, 0.1 / synth.HARTREE_EV))
    nbytes = 16.0 * n5 * n5 * (1 + len(om))
    out["plasmon_pole"] = {"ng": n5, "frequencies": len(om), "seconds": dt, "bytes": nbytes,
                           "gb_per_s": nbytes / dt / 1e9, "hbm_frac": nbytes / dt / 8e12}
    log(f"plasmon pole: {dt * 1e3:.1f} ms at NG {n5} x {len(om)} frequencies, {nbytes / dt / 1e9:.0f} GB/s")
    print(json.dumps({"metric": METRIC, "workload": "extensions", "dtype": mode, "data": "synthetic",
                      "results": out}))


if __name__ == "__main__":
    main()
