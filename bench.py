"""Benchmark of the Schwarz-HMC hot path on one MI355X.

One step = one application of the even-odd Wilson hop D_eo (Sec. 1, eq. 2 restricted to
one output parity, the operator the even-odd solvers apply four times per iteration) to
the 12 right-hand sides of the 24^3 x 48 workload (kappa = 0.158, links exp(i 0.35 H)) in
FP32 storage, the configuration of the batched block solves; inputs resident in HBM.
The value is the Dslash bandwidth: algorithmic bytes of one launch (every link once,
4 V x 72 B, plus each rhs's input and output half field, 2 x 48 B per site) divided by
the time per launch, timed with HIP events on the stream the kernel runs on.

Also printed in the same JSON line: the single-rhs FP64 / FP32 / FP16 even-odd hop and the
full operator M (apply_M, 960 / 480 / 248 B per site) with their own roofline fractions, the HBM
ceilings of plain kernels on this GPU, the CPU oracle baseline on a bounded sample, and
(unless --skip-solve) the block-solve comparison: mixed-precision batched vs plain FP64
solves to a verified 1e-10 residual.

Usage: python bench.py [--gpus 1] [--steps K] [--warmup W]
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

METRIC = "Dslash GB/s (% HBM peak); mixed vs FP64 block-solve time to 1e-10 residual"
WORKLOAD = "batched_24x24x24x48"
HBM_PEAK_GBS = 8000.0
REAL = {"f64": 8, "f32": 4, "f16": 2}
FLOP_PER_SITE = 1320      # hop of eq. 2 per output site and rhs (secondary figure)
# hop mappings of the timed 12-rhs even-odd launches (one kernel per line, profile and
# counter set); the full-size parity test sets the same ones
HEADLINE_MAPS = {"f32": "slabd", "f64": "slab1w", "f16": "slabd"}
ROTATE = 3                # contexts the single-rhs operators rotate over


def hop_map_id(sap, name):
    return sap.HOP_MAP_NAMES.index(name)


def spinor_site_bytes(prec):
    """Bytes of one stored spinor site: 24 reals, plus the FP32 site norm in FP16 storage."""
    return 24 * REAL[prec] + (4 if prec == "f16" else 0)


def eo_bytes(V, prec, nrhs):
    """Algorithmic bytes of one even-odd hop launch: all 4V links (18 reals) once, and per
    rhs the input half field and the output half field (V/2 sites each)."""
    return 4 * V * 18 * REAL[prec] + nrhs * 2 * (V // 2) * spinor_site_bytes(prec)


def apply_M_bytes(V, prec):
    """Algorithmic bytes of apply_M on one rhs: 4 links per site once, spinor in and out
    (960 / 480 / 248 B per site in FP64 / FP32 / FP16)."""
    return V * (4 * 18 * REAL[prec] + 2 * spinor_site_bytes(prec))


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--op", choices=["eo", "M"], default="eo",
                    help="operator timed by --only-dslash (profiler runs)")
    ap.add_argument("--prec", choices=["f64", "f32", "f16"], default="f32")
    ap.add_argument("--nrhs", type=int, default=12)
    ap.add_argument("--hop-map", default="",
                    help="with --only-dslash: comma-separated hop mappings (names or HOP_MAP_* numbers) "
                         "timed one after the other instead of the tuned one")
    ap.add_argument("--skip-solve", action="store_true")
    ap.add_argument("--skip-cpu", action="store_true")
    ap.add_argument("--cpu-extended", action="store_true",
                    help="also time the oracle's apply_M / apply_W1 / CGLS iterations on the host")
    ap.add_argument("--only-dslash", action="store_true",
                    help="time only the Dslash loop (for profiler runs)")
    ap.add_argument("--only-solve", choices=["cg_f32", "bicgstab_f32", "cg_f16", "bicgstab_f16", "cg_f64",
                                             "bicgstab_f64"],
                    help="run only this batched block solve of both levels once (for profiler runs)")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="also run a plain device copy of known size (counter calibration)")
    ap.add_argument("--only-force", action="store_true",
                    help="run only the force-kernel timings (for profiler runs)")
    return ap.parse_args()


def _oracle_hop_worker(task):
    """One application of the FP64 oracle's even-odd hop (output parity 0) to one rhs, in a
    worker process started fresh (spawn: nothing of the GPU process is inherited); the
    fields are memory-mapped from the .npy files the parent wrote. Returns the CPU seconds."""
    import numpy as np
    from oracle import dirac, lattice
    udir, r = task
    U = np.load(os.path.join(udir, "U.npy"), mmap_mode="r")
    psi = np.load(os.path.join(udir, "psi.npy"), mmap_mode="r")[r]
    par = lattice.parity(U.shape[:4])
    m_in, m_out = lattice.site_mask(U.shape[:4], par == 1), lattice.site_mask(U.shape[:4], par == 0)
    c0 = time.process_time()
    dirac.hop(np.asarray(U), psi * m_in) * m_out
    return time.process_time() - c0


def _worker_ready(_):
    import oracle.dirac  # noqa: F401  (imports done before the timed passes)
    return os.getpid()


def cpu_baseline(U, psi, V, rounds=2):
    """The FP64 oracle's even-odd hop on the benchmark's own workload, the 12 rhs of
    24^3x48, on the host cores: one worker process per rhs (the oracle as it stands, applied
    to independent rhs in parallel), `rounds` passes over the 12 rhs. GB/s over the
    algorithmic bytes of the FP64 12-rhs launch."""
    import multiprocessing as mp
    import shutil
    import tempfile
    import numpy as np
    nrhs = psi.shape[0]
    ncpu = len(os.sched_getaffinity(0)) if hasattr(os, "sched_getaffinity") else os.cpu_count()
    workers = max(1, min(nrhs, ncpu))
    udir = tempfile.mkdtemp(prefix="sap_oracle_")
    try:
        np.save(os.path.join(udir, "U.npy"), U)
        np.save(os.path.join(udir, "psi.npy"), psi)
        with mp.get_context("spawn").Pool(workers) as pool:
            pool.map(_worker_ready, range(workers))
            w0 = time.perf_counter()
            cpu = 0.0
            for _ in range(rounds):
                cpu += sum(pool.map(_oracle_hop_worker, [(udir, r) for r in range(nrhs)], chunksize=1))
            wall = time.perf_counter() - w0
    finally:
        shutil.rmtree(udir, ignore_errors=True)
    per = wall / rounds
    return {"value": round(eo_bytes(V, "f64", nrhs) / per / 1e9, 3), "unit": "GB/s",
            "cores": workers, "kind": "oracle",
            "sample": f"{rounds} passes of the even-odd hop (FP64 numpy oracle) over the {nrhs} rhs of 24^3x48, "
                      f"one worker process per rhs on {workers} of {ncpu} host CPUs: {per:.2f} s wall per "
                      f"12-rhs pass ({cpu / rounds / nrhs:.2f} s CPU per rhs); GB/s over the FP64 12-rhs "
                      f"launch's algorithmic bytes"}


def cpu_extended():
    """Further timings of the FP64 oracle on the host cores (opt-in, about a minute):
    apply_M and apply_W1 on the 16^3x32 and 24^3x48 workloads, and the cost of one CGLS
    iteration of the even-odd solve on 16^3x32 for one 16^3x4 block and for the full
    lattice (10 iterations timed, less the set-up; whole solves take 100-200 iterations).
    The oracle works on full-lattice arrays, so its block iteration costs full-lattice
    operator applications."""
    import numpy as np
    import synth
    from oracle import dirac, lattice, solvers

    def timed(fn):
        c0, w0 = time.process_time(), time.perf_counter()
        fn()
        w = time.perf_counter() - w0
        return w, max(1, round((time.process_time() - c0) / w))

    res = {"host_cpus": os.cpu_count()}
    for name in ("plain_16x16x16x32", "batched_24x24x24x48"):
        cfg = synth.CONFIGS[name]
        L, k, l0 = cfg["L"], cfg["kappa"], cfg["l0"]
        U = synth.gauge_field(L, cfg["eps"], cfg["seed_gauge"])
        psi = synth.gaussian_spinor(L, cfg["seed_src"])
        tm, cm = timed(lambda: dirac.apply_M(U, psi, k))
        tw, cw = timed(lambda: dirac.apply_W(U, psi, k, l0))
        res[name] = {"apply_M_seconds": round(tm, 3), "apply_W1_seconds": round(tw, 3), "cores": max(cm, cw)}
        print(f"[bench] oracle {name}: apply_M {tm:.2f} s, apply_W1 {tw:.2f} s", file=sys.stderr, flush=True)
        if name == "plain_16x16x16x32":
            even = dirac.parity_masks(L)[0]

            def per_iteration(lb, src):
                A = lambda v: dirac.apply_Mhat(U, v, k, lb, False)
                Ad = lambda v: dirac.apply_Mhat(U, v, k, lb, True)
                t10, c = timed(lambda: solvers.cgls(A, Ad, even * src, tol=1e-30, maxiter=10, max_restarts=0))
                t0, _ = timed(lambda: solvers.cgls(A, Ad, even * src, tol=1e-30, maxiter=0, max_restarts=0))
                return (t10 - t0) / 10, c

            tb, cb = per_iteration(l0, psi * lattice.site_mask(L, lattice.single_block_mask(L, l0, 0)))
            tf, cf = per_iteration(None, psi)
            res[name].update({"block_cg_seconds_per_iteration": round(tb, 3),
                              "full_cg_seconds_per_iteration": round(tf, 3), "solve_cores": max(cb, cf)})
            print(f"[bench] oracle {name}: CGLS iteration, one block {tb:.2f} s, full {tf:.2f} s",
                  file=sys.stderr, flush=True)
    return res


def hbm_probe(sap, torch, gib=2):
    """Bandwidth a plain streaming kernel reaches on this GPU (the library's own probe:
    16-byte accesses, grid-stride): copy, copy with non-temporal stores and read-only
    reduction of 2 GiB (best of 5 each), for context next to the 8 TB/s peak."""
    n = gib * (1 << 30)
    a = torch.ones(n // 4, dtype=torch.float32, device="cuda")
    b = torch.empty_like(a)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    res = {}
    for name, mode, moved in (("copy_gbs", 0, 2 * n), ("copy_nt_gbs", 1, 2 * n), ("read_gbs", 2, n)):
        best = 1e9
        for _ in range(5):
            e0.record()
            sap.sap_stream_probe(b, a, n, mode)
            e1.record()
            torch.cuda.synchronize()
            best = min(best, e0.elapsed_time(e1))
        res[name] = round(moved / best / 1e6, 1)
    del a, b
    res["bytes"] = n
    return res


KERNEL_SOURCES = ("dslash.hip", "half.hip", "split.hip", "split.h", "site_io.h", "device_common.h", "internal.h")


def kernel_source_hash():
    import hashlib
    h = hashlib.sha256()
    for f in KERNEL_SOURCES:
        with open(os.path.join(ROOT, "paper_0710_0066_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def committed_traffic(key):
    """HBM bytes per hop launch measured with rocprofv3 FETCH_SIZE / WRITE_SIZE (scaled by
    a plain copy of known size) for the hop kernel source it was taken on; None when the
    kernel source has changed since."""
    path = os.path.join(ROOT, "profiles", "hop_traffic_24x24x24x48.json")
    if not os.path.exists(path):
        return None
    with open(path) as fh:
        rec = json.load(fh)
    if rec.get("kernel_source_hash") != kernel_source_hash():
        return None
    entry = rec.get(key)
    return None if entry is None else entry["traffic_bytes_per_launch"]


def block_solve_comparison(sap, torch, ctx, cfg, L, repeats=5):
    """Wall time (call to verified return) of the block solves of the 24^3x48 workload:
    level 1 (12 blocks of 24^3x4) and level 2 (24 blocks of 24^3x2), 12 Gaussian
    right-hand sides each, to ||b - W x|| / ||b|| <= 1e-10 recomputed in FP64.
      mixed_batched       FP32 inner solves inside the FP64 defect correction, every block
                          and rhs of a level in one batched solve;
      fp64_batched        the same batching, FP64 inner solve (the precision gain alone);
      fp64_batched_bicgstab  the same with BiCGstab (the precision gain of that method);
      fp64_rhs_loop       FP64, one rhs per call, the blocks of a level together;
      fp64_per_block_loop FP64, one block and one rhs per call (the plain, unbatched
                          solve: 432 calls, timed once);
      mixed_batched_by_method  the mixed batched solve with the inner CG replaced by
                          BiCGstab and by the geometric series (Sec. 3's block-term solver);
      mixed_f16_storage_by_method  inner CG / BiCGstab on FP16-storage fields (FP32
                          arithmetic) to a relative residual of 2e-3 per correction."""
    import numpy as np
    import synth
    nrhs = cfg["nrhs"]
    b = synth.gaussian_spinor(L, cfg["seed_src"], nrhs=nrhs)
    fb = ctx.new_field(nrhs)
    ctx.pack_spinor(fb, torch.from_numpy(b).cuda(), nrhs)
    del b
    fx = ctx.new_field(nrhs)
    one = ctx.field_bytes(1) // 8
    mixed = sap.solve_opts(tol=1e-10, inner_prec=sap.SAP_F32, inner_tol=1e-5)
    plain = sap.solve_opts(tol=1e-10, inner_prec=sap.SAP_F64, inner_tol=0.0)

    def run(opts, mode, reps):
        ts, worst, iters = [], 0.0, 0
        for _ in range(reps):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            infos = []
            for level in (1, 2):
                nb = ctx.nblocks(level)
                if mode == "batched":
                    infos += sap.solve_blocks(ctx, fx, fb, nrhs, level, sap.SAP_ALL, opts)
                    continue
                for r in range(nrhs):
                    xr, br = fx[r * one:(r + 1) * one], fb[r * one:(r + 1) * one]
                    if mode == "rhs":
                        infos += sap.solve_blocks(ctx, xr, br, 1, level, sap.SAP_ALL, opts)
                    else:
                        for blk in range(nb):
                            inf = sap.solve_blocks(ctx, xr, br, 1, level, sap.SAP_ALL, opts, block=blk)
                            infos.append(inf[blk])
            ts.append(time.perf_counter() - t0)
            worst = max(e.true_rel_res for e in infos if e.iters > 0)
            iters = max(e.iters for e in infos)
        # the first call of a configuration also captures its iteration graphs
        return {"seconds": float(np.median(ts)), "first_call_seconds": ts[0], "runs": reps,
                "max_true_rel_res": worst, "max_iters": iters}

    print("[bench] block solves: mixed batched", file=sys.stderr, flush=True)
    m = run(mixed, "batched", repeats)
    methods = {"cg": m}
    for name, meth in (("bicgstab", sap.SAP_BICGSTAB), ("geometric_series", sap.SAP_GEOM)):
        print(f"[bench] block solves: mixed batched {name}", file=sys.stderr, flush=True)
        o = sap.solve_opts(tol=1e-10, inner_prec=sap.SAP_F32, inner_tol=1e-5, method=meth)
        try:
            methods[name] = run(o, "batched", repeats)
        except sap.SapError as e:
            methods[name] = {"error": str(e)}
    half = {}
    for name, meth in (("cg", sap.SAP_CG), ("bicgstab", sap.SAP_BICGSTAB)):
        print(f"[bench] block solves: FP16-storage inner {name}", file=sys.stderr, flush=True)
        o = sap.solve_opts(tol=1e-10, inner_prec=sap.SAP_F16, inner_tol=2e-3, method=meth)
        try:
            half[name] = run(o, "batched", repeats)
        except sap.SapError as e:
            half[name] = {"error": str(e)}
    print("[bench] block solves: fp64 batched", file=sys.stderr, flush=True)
    f = run(plain, "batched", repeats)
    print("[bench] block solves: fp64 batched bicgstab", file=sys.stderr, flush=True)
    try:
        fbi = run(sap.solve_opts(tol=1e-10, inner_prec=sap.SAP_F64, inner_tol=0.0, method=sap.SAP_BICGSTAB),
                  "batched", repeats)
    except sap.SapError as e:
        fbi = {"error": str(e)}
    print("[bench] block solves: fp64 one rhs per call", file=sys.stderr, flush=True)
    fl = run(plain, "rhs", 1)
    print("[bench] block solves: fp64 one block and rhs per call", file=sys.stderr, flush=True)
    fb1 = run(plain, "block", 1)
    return {"systems": f"{nrhs} rhs x (12 blocks 24^3x4 + 24 blocks 24^3x2) = {nrhs * 36}",
            "tol": 1e-10, "mixed_batched": m, "fp64_batched": f, "fp64_rhs_loop": fl,
            "fp64_per_block_loop": fb1, "fp64_batched_bicgstab": fbi, "mixed_batched_by_method": methods,
            "mixed_f16_storage_by_method": half,
            "speedup_vs_fp64_batched": f["seconds"] / m["seconds"],
            "speedup_bicgstab_vs_fp64_batched_bicgstab":
                fbi["seconds"] / methods["bicgstab"]["seconds"]
                if "seconds" in fbi and "seconds" in methods["bicgstab"] else None,
            "speedup_vs_fp64_rhs_loop": fl["seconds"] / m["seconds"],
            "speedup_vs_fp64_per_block_loop": fb1["seconds"] / m["seconds"],
            "speedup_bicgstab_vs_fp64_per_block_loop":
                fb1["seconds"] / methods["bicgstab"]["seconds"] if "seconds" in methods["bicgstab"] else None}


def force_kernels(sap, torch, ctx, V, reps):
    """Time per call of the molecular-dynamics kernels on the 24^3x48 links (the context's
    own): the gauge force (k_gauge_force: F += c Im tr(lambda^a U A) from the staples) and
    the link update (k_update_links: U <- exp(dt P) U by its Taylor series, reunitarised),
    timed as a step forward and back. Algorithmic bytes per call: links read (and written)
    once as 18 FP64 reals, forces and momenta as 8 FP64 reals per link. The context's
    links change by rounding; the caller sets them again."""
    import numpy as np
    F = ctx.new_momenta()
    P = ctx.new_momenta()
    g = torch.Generator(device="cpu").manual_seed(7)
    P.copy_(0.01 * torch.randn(P.numel(), generator=g, dtype=torch.float64))
    links = 4 * V
    res = {}
    for name, fn, nbytes in [
            ("gauge_force", lambda: sap.gauge_force(ctx, F, 1.0, 5.6), links * (18 + 8 + 8) * 8),
            ("update_links", lambda: (sap.sap_update_links(ctx, P, 1e-3), sap.sap_update_links(ctx, P, -1e-3)),
             2 * links * (18 + 8 + 18) * 8)]:
        fn()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(reps):
            fn()
        torch.cuda.synchronize()
        dt = (time.perf_counter() - t0) / reps
        res[name] = {"ms_per_call": round(dt * 1e3, 3), "algorithmic_bytes": nbytes,
                     "GB/s": round(nbytes / dt / 1e9, 1)}
        print(f"[bench] {name}: {dt * 1e3:.3f} ms per call", file=sys.stderr, flush=True)
    # pseudo-fermion force of the block action (FP64 block solve + k_pair_force); the kernel's
    # own time is in the rocprofv3 trace of --only-force
    phi = ctx.new_field(1)
    phi.copy_(torch.randn(phi.numel(), generator=g, dtype=torch.float64))
    opts = sap.solve_opts(tol=1e-10, inner_prec=sap.SAP_F32, inner_tol=1e-5)
    sap.block_pf_force(ctx, F, 1.0, phi, opts)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    n = max(2, reps // 5)
    for _ in range(n):
        sap.block_pf_force(ctx, F, 1.0, phi, opts)
    torch.cuda.synchronize()
    res["block_pf_force_call"] = {"ms_per_call": round((time.perf_counter() - t0) / n * 1e3, 2),
                                  "pair_force_algorithmic_bytes": V * 1472,
                                  "note": "includes the block solves; k_pair_force alone is in the profile"}
    del F, P, phi
    return res


def time_op(sap, torch, fn, steps, warmup):
    """Average time (ms) per launch of fn(k) over `steps` launches after `warmup`."""
    for k in range(warmup):
        fn(k)
    torch.cuda.synchronize()
    stream = torch.cuda.current_stream()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    e0.record(stream)
    for k in range(steps):
        fn(k)
    e1.record(stream)
    torch.cuda.synchronize()
    return e0.elapsed_time(e1) / steps


def roofline(gbs, key):
    return {"bound": "hbm", "achieved": round(gbs, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
            "frac": round(gbs / HBM_PEAK_GBS, 4), "traffic": committed_traffic(key)}


def main():
    args = parse()
    if args.gpus != 1:
        print(json.dumps({"error": "this build runs on one GPU only; --gpus must be 1"}))
        sys.exit(2)
    import numpy as np
    import torch

    import paper_0710_0066_amd as sap
    import synth

    cfg = synth.CONFIGS[WORKLOAD]
    L, k, l0, l0s, nrhs = cfg["L"], cfg["kappa"], cfg["l0"], cfg["l0_sub"], cfg["nrhs"]
    V = int(np.prod(L))
    torch.cuda.set_device(0)
    print(f"[bench] generating {WORKLOAD} inputs", file=sys.stderr, flush=True)
    U = synth.gauge_field(L, cfg["eps"], cfg["seed_gauge"])
    psi = synth.gaussian_spinor(L, cfg["seed_src"], nrhs=nrhs)

    ctx = sap.Context(L, l0, k, l0_sub=l0s, max_rhs=nrhs)
    Ud = torch.from_numpy(U).cuda()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    ctx.set_gauge(Ud)      # pack into the tiled layout and make the FP32 / FP16 link copies
    torch.cuda.synchronize()
    gauge_upload_s = time.perf_counter() - t0
    PREC = {"f64": sap.SAP_F64, "f32": sap.SAP_F32, "f16": sap.SAP_F16}
    # single-rhs operators rotate over ROTATE contexts, each with its own links and fields,
    # so that a launch finds little of its ~0.2-0.4 GB working set in the 256 MB MALL
    rot = [ctx]
    tuned1 = {}               # ctx's single-rhs mappings, used by every rotation context

    def rotation():
        if not tuned1:
            tuned1.update(sap.sap_tune(ctx, 1))
        while len(rot) < ROTATE:
            c = sap.Context(L, l0, k, l0_sub=l0s, max_rhs=1)
            c.set_gauge(Ud)
            for key, us in tuned1.items():
                kind, prec = key.split("_")
                sap.sap_set_hop_map(c, int(kind == "full"), PREC[prec], 1, hop_map_id(sap, min(us, key=us.get)))
            rot.append(c)
        return rot
    fields = {}

    def field(c, prec, n):
        key = (id(c), prec, n)
        if key not in fields:
            fin = c.new_field(n, PREC[prec])
            c.pack_spinor(fin, torch.from_numpy(np.ascontiguousarray(psi[:n])).cuda(), n, PREC[prec])
            fields[key] = (fin, c.new_field(n, PREC[prec]))
        return fields[key]

    def eo(prec, n):
        if n == nrhs:
            fin, fout = field(ctx, prec, n)
            return lambda s: sap.apply_Dslash_eo(ctx, fout, fin, n, s & 1, PREC[prec])
        ops = [(c,) + field(c, prec, n) for c in rotation()]
        return lambda s: sap.apply_Dslash_eo(ops[s % ROTATE][0], ops[s % ROTATE][2], ops[s % ROTATE][1], n,
                                             (s // ROTATE) & 1, PREC[prec])

    def full(prec):
        ops = [(c,) + field(c, prec, 1) for c in rotation()]
        return lambda s: sap.apply_M(ops[s % ROTATE][0], ops[s % ROTATE][2], ops[s % ROTATE][1], 1, PREC[prec])

    if args.only_force:
        force_kernels(sap, torch, ctx, V, args.steps)
        return

    if args.only_solve:        # one batched block solve of both levels, for profiler runs
        meth, p = args.only_solve.split("_")
        o = sap.solve_opts(tol=1e-10, inner_prec=PREC[p], inner_tol={"f64": 0.0, "f32": 1e-5, "f16": 2e-3}[p],
                           method={"cg": sap.SAP_CG, "bicgstab": sap.SAP_BICGSTAB}[meth])
        sap.sap_tune(ctx, nrhs)
        fb = ctx.new_field(nrhs)
        ctx.pack_spinor(fb, torch.from_numpy(psi).cuda(), nrhs)
        fx = ctx.new_field(nrhs)
        for rep in range(2):     # the first pass captures the graphs
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            worst = 0.0
            for level in (1, 2):
                info = sap.solve_blocks(ctx, fx, fb, nrhs, level, sap.SAP_ALL, o)
                worst = max(worst, max(e.true_rel_res for e in info))
            torch.cuda.synchronize()
            print(f"[bench] block solves {args.only_solve} pass {rep}: {time.perf_counter() - t0:.3f} s, "
                  f"max residual {worst:.2e}", file=sys.stderr, flush=True)
        return

    if args.only_dslash:       # one operator only, for profiler runs
        n_op = args.nrhs if args.op == "eo" else 1
        maps = [m for m in args.hop_map.split(",") if m]
        if not maps:
            if args.op == "eo" and args.nrhs == nrhs and args.prec in HEADLINE_MAPS:
                maps = [HEADLINE_MAPS[args.prec]]
            else:     # the tuner's choice, set on every context the launches rotate over
                res = sap.sap_tune(ctx, n_op)
                us = res[("eo" if args.op == "eo" else "full") + "_" + args.prec]
                maps = [min(us, key=us.get)]
                if n_op == 1:
                    tuned1.update(res)
        fn = eo(args.prec, args.nrhs) if args.op == "eo" else full(args.prec)
        for m in maps or [None]:     # the given mappings only (no tuner launches in the profile)
            if m is not None:
                mid = int(m) if m.isdigit() else hop_map_id(sap, m)
                for c in (rot if n_op == 1 else [ctx]):
                    sap.sap_set_hop_map(c, int(args.op == "M"), PREC[args.prec], n_op, mid)
            ms = time_op(sap, torch, fn, args.steps, args.warmup)
            print(f"[bench] {args.op} {args.prec} nrhs={args.nrhs if args.op == 'eo' else 1} map {m}: "
                  f"{ms * 1e3:.1f} us/launch", file=sys.stderr, flush=True)
        if args.copy_calibration:
            copy_calibration(sap, torch)
        return

    print("[bench] tuning the hop mapping", file=sys.stderr, flush=True)
    tuning = {"nrhs_%d" % n: sap.sap_tune(ctx, n) for n in (1, nrhs)}
    tuned1.update(tuning["nrhs_1"])
    # the 12-rhs launches use fixed mappings (HEADLINE_MAPS, the tuner's choices on this
    # workload, whose runner-up mappings are within a few percent), so that the line, its
    # profile and its counters describe one kernel
    for prec, name in HEADLINE_MAPS.items():
        sap.sap_set_hop_map(ctx, 0, PREC[prec], nrhs, hop_map_id(sap, name))
    ms = time_op(sap, torch, eo("f32", nrhs), args.steps, args.warmup)
    gbs = eo_bytes(V, "f32", nrhs) / (ms * 1e-3) / 1e9
    print(f"[bench] D_eo f32 {nrhs} rhs: {ms * 1e3:.1f} us/launch, {gbs:.0f} GB/s", file=sys.stderr, flush=True)
    result = {
        "metric": METRIC, "value": round(gbs, 1), "unit": "GB/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": ms,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32", "data": "synthetic (seeded links exp(i 0.35 H), Gaussian sources)",
        "config": {"workload": WORKLOAD, "lattice": "24^3x48", "op": "D_eo (even-odd hop)",
                   "nrhs": nrhs, "kappa": k, "storage": "f32",
                   "algorithmic_bytes_per_launch": eo_bytes(V, "f32", nrhs)},
        "roofline": roofline(gbs, "eo_f32_12rhs"),
        "gflops": round(FLOP_PER_SITE * (V // 2) * nrhs / (ms * 1e-3) / 1e9, 1),
        "gauge_upload_seconds": round(gauge_upload_s, 4),
    }
    others = {}
    for name, fn, nbytes in [
            ("eo_f64_1rhs", eo("f64", 1), eo_bytes(V, "f64", 1)),
            ("eo_f32_1rhs", eo("f32", 1), eo_bytes(V, "f32", 1)),
            ("eo_f64_12rhs", eo("f64", nrhs), eo_bytes(V, "f64", nrhs)),
            ("eo_f16_1rhs", eo("f16", 1), eo_bytes(V, "f16", 1)),
            ("eo_f16_12rhs", eo("f16", nrhs), eo_bytes(V, "f16", nrhs)),
            ("apply_M_f64_1rhs", full("f64"), apply_M_bytes(V, "f64")),
            ("apply_M_f32_1rhs", full("f32"), apply_M_bytes(V, "f32")),
            ("apply_M_f16_1rhs", full("f16"), apply_M_bytes(V, "f16"))]:
        t = time_op(sap, torch, fn, max(20, args.steps // 2), args.warmup)
        g = nbytes / (t * 1e-3) / 1e9
        others[name] = {"us_per_launch": round(t * 1e3, 2), "algorithmic_bytes": nbytes,
                        "roofline": roofline(g, name)}
        print(f"[bench] {name}: {t * 1e3:.1f} us, {g:.0f} GB/s", file=sys.stderr, flush=True)
    result["other_operators"] = others
    result["single_rhs_rotation"] = (f"single-rhs operators rotate over {ROTATE} contexts (own links and fields), "
                                     "so consecutive launches do not reuse each other's data from the MALL")
    result["force_kernels"] = force_kernels(sap, torch, ctx, V, max(10, args.steps // 10))
    ctx.set_gauge(Ud)
    result["hop_tuning_us"] = {n: {k: {m: round(v, 1) for m, v in d.items()} for k, d in t.items()}
                               for n, t in tuning.items()}
    fields.clear()
    del Ud
    for c in rot[1:]:
        c.close()
    result["hbm_probe"] = hbm_probe(sap, torch)
    if not args.skip_solve:
        result["block_solve"] = block_solve_comparison(sap, torch, ctx, cfg, L)
    if not args.skip_cpu:
        print("[bench] timing the CPU oracle", file=sys.stderr, flush=True)
        result["cpu_baseline"] = cpu_baseline(U, psi, V)
        if args.cpu_extended:
            print("[bench] timing further oracle operations", file=sys.stderr, flush=True)
            result["cpu_extended"] = cpu_extended()
    print(json.dumps(result), flush=True)


def copy_calibration(sap, torch):
    """One copy of 1 GiB by the library's stream probe (k_stream_copy) whose source was
    pushed out of the 256 MB MALL by a second 1 GiB fill: its counters must read 1 GiB
    fetched and 1 GiB written, which fixes the scale of FETCH_SIZE / WRITE_SIZE."""
    n = 1024 * 1024 * 1024
    a = torch.full((n // 4,), 1.0, dtype=torch.float32, device="cuda")
    c = torch.full((n // 4,), 2.0, dtype=torch.float32, device="cuda")
    b = torch.empty_like(a)
    torch.cuda.synchronize()
    sap.sap_stream_probe(b, a, n, 0)
    torch.cuda.synchronize()
    del a, b, c
    print(f"[bench] copy calibration: one stream-probe copy of {n} bytes", file=sys.stderr, flush=True)


if __name__ == "__main__":
    main()
