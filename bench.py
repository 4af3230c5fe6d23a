#!/usr/bin/env python3
"""SP2 density-matrix benchmark on one AMD Instinct MI355X (gfx950).

One step is one call of the whole path through the C ABI (sp2_density): Gershgorin
bounds, input layer, the Alg. 1 layers with the dual-FP16 squaring of Alg. 2, the FP64
refinement layer and the final checks, on the N = 8192 small-gap stress Hamiltonian
(25% occupation, 0.2 eV gap, eigenvalues uniform in [-25, 25] eV) resident in HBM.
The timed steps use the event-instrumented entry point (same kernels, HIP events
recorded between them on the library's stream), so the per-kernel durations below
come from the timed steps themselves.

Reported (one JSON line on stdout; progress on stderr):
  value            whole-call throughput: FLOP executed per call (every squaring layer,
                   3 N^2 (N + 1) for the three half-precision products over the upper
                   triangle, plus the two FP64 refinement products, N^2 (N + 1) each)
                   divided by the time-to-D of the call
  ms_per_step      time-to-D of one full call, H resident on the device
  loop_tflops      squaring layers only (executed FLOP), over the loop time
  paper_convention_tflops  the paper's accounting: 4 N^3 per mixed layer (two dense
                   half-precision products), loop time only, no set-up or refinement
  roofline         the squaring kernel (dominant) against the dense FP16 matrix peak
  fp64             the same computation with FP64 squarings on the GPU (speed comparison)
  accuracy         ||D - D_ref||_F and |Tr D - N_occ| with D_ref the exact projector
  cpu_baseline     the CPU oracle (FP64 NumPy Alg. 1) on a bounded sample of the workload
"""
import argparse
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

PEAK_FP16_TFLOPS = 2500.0     # MI355X dense FP16/BF16 matrix peak
PEAK_FP64_TFLOPS = 78.6       # MI355X FP64 matrix peak
METRIC = "SP2 TFLOP/s + time-to-D at N=8192, mixed vs FP64, at stated ‖D−D_ref‖_F"


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def flop_split_layer(n):
    """Three half-precision products restricted to the upper triangle (with diagonal)."""
    return 3.0 * 2.0 * n * (n * (n + 1) / 2.0)


def flop_plain_layer(n):
    """One FP32/FP64 product restricted to the upper triangle (with diagonal)."""
    return 2.0 * n * (n * (n + 1) / 2.0)


# Persistent-kernel variants (waves, K-slice halves, LDS stages, L2 prefetch distance) per
# tile edge, in the order of the library's kernel option 2..7.
# (waves, K-slice halves, LDS stages, rolling fragment pipeline) per persistent variant
SK_VARIANTS = {256: [(4, 16, 4, 0), (8, 16, 4, 0), (4, 32, 2, 0), (8, 32, 2, 0), (4, 32, 2, 1), (8, 32, 2, 1)],
               128: [(4, 32, 4, 0), (4, 64, 2, 0), (4, 16, 4, 0), (4, 32, 2, 0), (4, 64, 2, 1), (4, 32, 2, 1)]}


def kernel_name(precision, tile, kernel, n, n_padded):
    """Name of the squaring kernel a call used (from sp2_info and the library's size rules)."""
    t16 = {"fp16x2": "_Float16", "bf16x2": "__bf16"}.get(precision)
    if n <= 64 and precision != "fp32":   # with the schedule left open: the whole solve in one launch
        return "k_tiny<%s, %s, true>" % (t16 or "_Float16", "true" if t16 else "false")
    t64 = -(-n // 64)
    ntiles64 = t64 * (t64 + 1) // 2
    if t16:
        if kernel >= 2:
            waves, sk, st, rp = SK_VARIANTS[tile][kernel - 2]
            wn = waves // 2
            mb = tile // 64
            nb = tile // (32 * wn)
            return "k_square_sk<%s, 2, %d, %d, %d, %d, %d, %d>" % (t16, wn, mb, nb, sk, st, rp)
        if kernel == 1 and tile <= 128 and n_padded < 3072:
            return ("k_square_fm1<%s, 4, 4, %d>" if ntiles64 > 512 else "k_square_fm<%s, 4, 2, %d>") % (t16, tile == 128)
        if kernel == 1 and tile in (128, 256):
            return "k_square_dp<%s, 2, %d, %d, 2, 32, 2>" % (t16, 4 if tile == 256 else 2, tile // 64)
        return "k_square_split<%s, %d>" % (t16, tile)
    return "k_square_%s_%s" % ("f64" if precision == "fp64" else "f32", "lead" if ntiles64 < 256 else "mix")


def kernel_sources_digest():
    """SHA-256 over the sources of the squaring kernels: counter records taken with other
    sources no longer describe the kernel."""
    import glob
    import hashlib

    hsh = hashlib.sha256()
    csrc = os.path.join(ROOT, "paper_2101_06385_amd", "csrc")
    for f in sorted(glob.glob(os.path.join(csrc, "k_square*")) + glob.glob(os.path.join(csrc, "k_sk_*")) +
                    [os.path.join(csrc, "sp2_args.h")]):
        hsh.update(os.path.basename(f).encode())
        hsh.update(open(f, "rb").read())
    return hsh.hexdigest()


def recorded_traffic(kname, n):
    """HBM bytes per launch of `kname` at size n from profiles/traffic.json (rocprofv3 FETCH_SIZE
    and WRITE_SIZE, FETCH scaled by the copy-kernel calibration), or None when no record
    matches this kernel, size and source digest."""
    path = os.path.join(ROOT, "profiles", "traffic.json")
    if not os.path.exists(path):
        return None
    try:
        recs = json.load(open(path))
    except ValueError:
        return None
    dig = kernel_sources_digest()
    for r in recs.get("records", []):
        if r.get("kernel") == kname and int(r.get("n", 0)) == n and r.get("sources_sha256") == dig:
            return float(r["hbm_bytes_per_launch"])
    return None


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--n", type=int, default=8192)
    ap.add_argument("--precision", default="fp16x2")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-fp64", action="store_true")
    ap.add_argument("--no-accel", action="store_true", help="skip the accelerated Deep-NN SP2 leg")
    ap.add_argument("--no-autotune", action="store_true", help="skip reporting the autotuner's choice")
    ap.add_argument("--no-bf16", action="store_true", help="skip the BF16X2 comparison leg")
    ap.add_argument("--gen-device", default="cuda", help="where the QR of the workload generator runs")
    ap.add_argument("--cpu-eigh", type=int, default=1, help="time the oracle's diagonalization (numpy eigh + "
                    "V_occ V_occ^T) on the host at the headline size as part of cpu_baseline (0: skip)")
    ap.add_argument("--workload", default="density", choices=["density", "batched", "net", "fermi", "md", "sweep"],
                    help="density: the N=8192 headline (default); batched: 64 Hamiltonians of uneven "
                         "sizes in one graph; net: the 20-layer differentiable network at N=2048; fermi: "
                         "the 11-layer optimized finite-temperature expansion at N (default 8192); md: a "
                         "sequence of slowly changing Hamiltonians with HOMO/LUMO estimates carried forward; "
                         "sweep: the headline measurement at N = 1024 .. 16384")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: the SP2 path runs on one MI355X and is measured on one GPU; "
              "--gpus %d is not supported" % args.gpus, file=sys.stderr)
        sys.exit(2)
    if args.workload == "batched":
        return bench_batched(args)
    if args.workload == "net":
        return bench_net(args)
    if args.workload == "fermi":
        return bench_fermi(args)
    if args.workload == "md":
        return bench_md(args)
    if args.workload == "sweep":
        return bench_sweep(args)

    import numpy as np
    import torch

    from paper_2101_06385_amd import sp2, workloads

    dev = torch.device("cuda:0")
    n = args.n
    t0 = time.perf_counter()
    gen_dev = None if args.gen_device == "cpu" else "cuda:0"
    try:
        w = workloads.config3(n=n, device=gen_dev)
    except Exception as e:  # pragma: no cover - fall back to LAPACK on the host
        log("device QR failed (%s); generating on the host" % e)
        w = workloads.config3(n=n)
    log("workload %s generated in %.1f s" % (w.name, time.perf_counter() - t0))
    h = torch.from_numpy(w.h).to(dev)
    d = torch.empty_like(h)
    opts = sp2.options(args.precision)
    ws = sp2.alloc_workspace(sp2.workspace_size(n, opts), dev)
    torch.cuda.synchronize()

    def step():
        return sp2.density(h, w.n_occ, precision=args.precision, out=d, workspace=ws, timed=True)

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    steps = []
    t_start = time.perf_counter()
    for _ in range(args.steps):
        steps.append(step())
    torch.cuda.synchronize()
    ms_per_step = (time.perf_counter() - t_start) * 1e3 / args.steps
    log("time-to-D %.2f ms per step" % ms_per_step)

    _, info, tm = steps[-1]
    split = args.precision in ("fp16x2", "bf16x2")
    f_layer = flop_split_layer(n) if split else flop_plain_layer(n)
    f_refine = 2 * flop_plain_layer(n)
    k = tm["squarings"]
    flop_call = k * f_layer + f_refine
    value = flop_call / (ms_per_step * 1e-3) / 1e12
    loop_ms = float(np.mean([t["loop_active_ms"] for _, _, t in steps]))
    loop_tflops = k * f_layer / (loop_ms * 1e-3) / 1e12
    sq = [x for _, _, t in steps for x in t["square_ms"][:t["squarings"]]]
    sq_mean = float(np.mean(sq)) if sq else float("nan")
    achieved = f_layer / (sq_mean * 1e-3) / 1e12
    peak = PEAK_FP16_TFLOPS if split else (PEAK_FP64_TFLOPS if args.precision == "fp64" else 157.3)
    kname = kernel_name(args.precision, info["tile"], info["kernel"], n, info["n_padded"])
    traffic = recorded_traffic(kname, n)
    log("layers m=%d squarings=%d loop %.2f ms (%.1f TFLOP/s) square kernel %.3f ms (%.1f TFLOP/s, %s) "
        "refine %.2f ms status %s; whole call %.1f TFLOP/s" % (info["layers"], k, loop_ms, loop_tflops, sq_mean,
                                                              achieved, kname, tm["refine_ms"],
                                                              info["status_name"], value))

    out = {
        "metric": METRIC if n == 8192 else METRIC.replace("N=8192", "N=%d" % n),
        "value": round(value, 3),
        "unit": "TFLOP/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 3),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f16" if args.precision == "fp16x2" else ("bf16" if args.precision == "bf16x2" else
                                                           ("f64" if args.precision == "fp64" else "f32")),
        "data": "synthetic",
        "config": {
            "workload": "small-gap stress Hamiltonian N=%d: H = Q diag(eps) Q^T, Haar Q, 25%% occupation, "
                        "0.2 eV gap, eigenvalues uniform in [-25,25] eV; Gershgorin bounds" % n,
            "n": n, "n_occ": w.n_occ, "precision": args.precision, "accumulate": "f32",
            "layers": info["layers"], "squarings": k, "tile": info["tile"], "n_padded": info["n_padded"],
        },
        "time_to_d_ms": round(ms_per_step, 3),
        "flop_per_call": flop_call,
        "loop_tflops": round(loop_tflops, 3),
        "paper_convention_tflops": round(k * (4.0 if split else 2.0) * n ** 3 / (loop_ms * 1e-3) / 1e12, 3),
        "loop_ms": round(loop_ms, 3),
        "refine_ms": round(float(np.mean([t["refine_ms"] for _, _, t in steps])), 3),
        "prep_ms": round(float(np.mean([t["prep_ms"] for _, _, t in steps])), 3),
        "status": info["status_name"],
        "trace_error": abs(info["trace"] - w.n_occ),
        "idempotency": info["idem"],
        "roofline": {
            "bound": "mfma", "achieved": round(achieved, 3), "peak": peak, "unit": "TFLOP/s",
            "frac": round(achieved / peak, 4), "traffic": traffic,
            "kernel": kname, "flop_per_launch": f_layer, "launch_ms": round(sq_mean, 4),
            "launches_timed": len(sq),
        },
    }

    if not args.no_fp64:
        d64 = torch.empty_like(h)
        o64 = sp2.options("fp64")
        ws64 = sp2.alloc_workspace(sp2.workspace_size(n, o64), dev)
        sp2.density(h, w.n_occ, precision="fp64", out=d64, workspace=ws64)      # warm
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        _, i64 = sp2.density(h, w.n_occ, precision="fp64", out=d64, workspace=ws64)
        torch.cuda.synchronize()
        ttd64 = (time.perf_counter() - t1) * 1e3
        _, i64, tm64 = sp2.density(h, w.n_occ, precision="fp64", out=d64, workspace=ws64, timed=True)
        k64 = tm64["squarings"]
        v64 = k64 * flop_plain_layer(n) / (tm64["loop_active_ms"] * 1e-3) / 1e12
        out["fp64"] = {"time_to_d_ms": round(ttd64, 3), "tflops": round(v64, 3), "layers": i64["layers"],
                       "status": i64["status_name"], "trace_error": abs(i64["trace"] - w.n_occ),
                       "speedup_mixed_vs_fp64": round(ttd64 / ms_per_step, 3),
                       "frac_of_fp64_peak": round(v64 / PEAK_FP64_TFLOPS, 4)}
        log("fp64: time-to-D %.1f ms, %.1f TFLOP/s, layers %d, %s" % (ttd64, v64, i64["layers"], i64["status_name"]))
    else:
        d64 = None

    dbf = None
    if args.precision == "fp16x2" and not args.no_bf16:
        # the same solve with BF16 planes (the other split precision of the method)
        dbf = torch.empty_like(h)
        obf = sp2.options("bf16x2")
        wsbf = sp2.alloc_workspace(sp2.workspace_size(n, obf), dev)
        sp2.density(h, w.n_occ, precision="bf16x2", out=dbf, workspace=wsbf)      # warm
        torch.cuda.synchronize()
        bsteps = []
        t1 = time.perf_counter()
        for _ in range(args.steps):
            bsteps.append(sp2.density(h, w.n_occ, precision="bf16x2", out=dbf, workspace=wsbf, timed=True))
        torch.cuda.synchronize()
        ttdb = (time.perf_counter() - t1) * 1e3 / args.steps
        _, ibf, _ = bsteps[-1]
        sqb = [x for _, _, t in bsteps for x in t["square_ms"][:t["squarings"]]]
        kb = f_layer / (float(np.mean(sqb)) * 1e-3) / 1e12
        out["bf16x2"] = {"time_to_d_ms": round(ttdb, 3), "layers": ibf["layers"], "status": ibf["status_name"],
                         "kernel_tflops": round(kb, 3), "frac": round(kb / PEAK_FP16_TFLOPS, 4),
                         "trace_error": abs(ibf["trace"] - w.n_occ)}
        log("bf16x2: time-to-D %.2f ms, layers %d, square kernel %.1f TFLOP/s" % (ttdb, ibf["layers"], kb))
        del wsbf

    dacc = d64a = None
    if not args.no_accel:
        # Accelerated Deep-NN SP2 on the same H with its HOMO/LUMO values as the prior
        # knowledge the method needs (as from a previous call in a molecular-dynamics run)
        gap = (w.homo, w.lumo)
        dacc = torch.empty_like(h)
        oacc = sp2.options(args.precision, gap=gap)
        wsacc = sp2.alloc_workspace(sp2.workspace_size(n, oacc), dev)
        sp2.density(h, w.n_occ, precision=args.precision, out=dacc, workspace=wsacc, gap=gap)      # warm
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        for _ in range(args.steps):
            _, iacc = sp2.density(h, w.n_occ, precision=args.precision, out=dacc, workspace=wsacc, gap=gap)
        torch.cuda.synchronize()
        ttda = (time.perf_counter() - t1) * 1e3 / args.steps
        acc_out = {"time_to_d_ms": round(ttda, 3), "layers": iacc["layers"], "accelerated_layers": iacc["accelerated"],
                   "status": iacc["status_name"], "trace_error": abs(iacc["trace"] - w.n_occ),
                   "speedup_vs_plain": round(ms_per_step / ttda, 3), "homo_lumo": list(gap)}
        log("accelerated: time-to-D %.2f ms, layers %d (%d accelerated), %s" % (ttda, iacc["layers"],
                                                                             iacc["accelerated"],
                                                                             iacc["status_name"]))
        if not args.no_fp64:
            o64a = sp2.options("fp64", gap=gap)
            ws64a = sp2.alloc_workspace(sp2.workspace_size(n, o64a), dev)
            d64a = torch.empty_like(h)
            sp2.density(h, w.n_occ, precision="fp64", out=d64a, workspace=ws64a, gap=gap)      # warm
            torch.cuda.synchronize()
            t1 = time.perf_counter()
            _, i64a = sp2.density(h, w.n_occ, precision="fp64", out=d64a, workspace=ws64a, gap=gap)
            torch.cuda.synchronize()
            ttd64a = (time.perf_counter() - t1) * 1e3
            acc_out["fp64"] = {"time_to_d_ms": round(ttd64a, 3), "layers": i64a["layers"],
                               "status": i64a["status_name"], "speedup_mixed_vs_fp64": round(ttd64a / ttda, 3)}
            log("accelerated fp64: time-to-D %.1f ms, layers %d" % (ttd64a, i64a["layers"]))
            del ws64a
        out["accelerated"] = acc_out

    if not args.no_cpu_baseline:
        # CPU leg: the oracle (test infrastructure) on a bounded sample, plus the exact
        # projector for the accuracy of the GPU results.
        from oracle import dm as odm
        from oracle import sp2 as osp2

        try:
            from threadpoolctl import threadpool_info
            cores = max([p.get("num_threads", 0) for p in threadpool_info()] + [1])
        except Exception:  # pragma: no cover
            cores = os.cpu_count()
        layers = 10
        tc = time.perf_counter()
        osp2.sp2_alg1(w.h, w.n_occ, max_layers=layers, refine=False)
        tcpu = time.perf_counter() - tc
        cpu_rate = layers * 2.0 * n ** 3 / tcpu / 1e12
        out["cpu_baseline"] = {
            "value": round(cpu_rate, 4), "unit": "TFLOP/s", "cores": int(cores), "kind": "oracle",
            "sample": "first %d FP64 layers of Alg. 1 (oracle.sp2.sp2_alg1, NumPy/OpenBLAS, including its "
                      "Gershgorin bounds and input layer) on the same N=%d Hamiltonian, %.1f s; rate credits "
                      "2N^3 per layer" % (layers, n, tcpu),
            "time_to_d_est_s": round(tcpu / layers * (info["layers"] + 2), 1),
        }
        log("cpu oracle: %.3f TFLOP/s on %d threads (%.1f s)" % (cpu_rate, cores, tcpu))
        d_ref = odm.dm_construct(w.q, w.eps, w.n_occ)
        if args.cpu_eigh:
            # the other host baseline: time-to-D by diagonalization (LAPACK eigh, FP64, all
            # threads) on the same H, and its distance to the constructed projector
            tc = time.perf_counter()
            d_eigh = odm.dm_eigh(w.h, w.n_occ)
            te = time.perf_counter() - tc
            out["cpu_baseline"]["eigh_time_to_d_s"] = round(te, 2)
            out["cpu_baseline"]["eigh_fro_error"] = float(np.linalg.norm(d_eigh - d_ref))
            out["cpu_baseline"]["eigh_speedup_of_gpu_mixed"] = round(te * 1e3 / ms_per_step, 1)
            log("cpu eigh: time-to-D %.1f s (%.0fx the GPU mixed-precision call)" % (te, te * 1e3 / ms_per_step))
            del d_eigh
        acc = {"fro_error": float(np.linalg.norm(d.cpu().numpy() - d_ref)),
               "fro_bound": 1e-3 * math.sqrt(n), "trace_error": abs(info["trace"] - w.n_occ)}
        if d64 is not None:
            acc["fro_error_fp64"] = float(np.linalg.norm(d64.cpu().numpy() - d_ref))
        out["accuracy"] = acc
        if dbf is not None:
            out["bf16x2"]["fro_error"] = float(np.linalg.norm(dbf.cpu().numpy() - d_ref))
        if dacc is not None:
            out["accelerated"]["fro_error"] = float(np.linalg.norm(dacc.cpu().numpy() - d_ref))
            if "fp64" in out["accelerated"]:
                out["accelerated"]["fp64"]["fro_error"] = float(np.linalg.norm(d64a.cpu().numpy() - d_ref))
        log("accuracy: %s" % acc)
    props = torch.cuda.get_device_properties(dev)
    out["env"] = {"device": props.name, "gcn_arch": getattr(props, "gcnArchName", ""),
                  "compute_units": props.multi_processor_count, "hip": torch.version.hip}
    if not args.no_autotune:
        # the autotuner's choice at this size (after every timed leg; its table is reset so
        # that nothing above depended on it)
        tuned = sp2.autotune(n, args.precision)
        sp2.autotune_reset()
        out["autotune"] = {"tile": tuned["tile"], "kernel": tuned["kernel"], "layer_ms": round(tuned["ms"], 4),
                           "headline_schedule": {"tile": info["tile"], "kernel": info["kernel"]}}
        log("autotuner: tile %d kernel %d %.3f ms per layer (headline: tile %d kernel %d)"
            % (tuned["tile"], tuned["kernel"], tuned["ms"], info["tile"], info["kernel"]))
    print(json.dumps(out), flush=True)


def _cores():
    try:
        from threadpoolctl import threadpool_info
        return max([p.get("num_threads", 0) for p in threadpool_info()] + [1])
    except Exception:  # pragma: no cover
        return os.cpu_count()


def bench_batched(args):
    """64 Hamiltonians, N_i = 64 U{4..48}, occupation U[0.2, 0.5], gap U[0.5, 3] eV, solved by
    sp2_density_batched (every step one grouped launch, the sequence one hipGraph); compared
    with the same problems solved one after another by sp2_density."""
    import numpy as np
    import torch

    from paper_2101_06385_amd import sp2, workloads

    dev = torch.device("cuda:0")
    t0 = time.perf_counter()
    ws = workloads.config4(device=None if args.gen_device == "cpu" else "cuda:0")
    log("64 problems generated in %.1f s" % (time.perf_counter() - t0))
    hs = [torch.from_numpy(w.h).to(dev) for w in ws]
    occ = [w.n_occ for w in ws]
    sizes = [w.n for w in ws]
    opts = sp2.options(args.precision)
    wsbuf = sp2.alloc_workspace(sp2.batched_workspace_size(sizes, opts), dev)
    outs = [torch.empty_like(h) for h in hs]

    def step():
        return sp2.density_batched(hs, occ, precision=args.precision, outs=outs, workspace=wsbuf)

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    for _ in range(args.steps):
        _, infos = step()
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t1) * 1e3 / args.steps
    split = args.precision in ("fp16x2", "bf16x2")
    flop = sum((i["layers"] - 1) * (flop_split_layer(n) if split else flop_plain_layer(n)) + 2 * flop_plain_layer(n)
               for i, n in zip(infos, sizes))
    value = flop / (ms * 1e-3) / 1e12
    # the same problems one call at a time (automatic schedule per size)
    single_ws = sp2.alloc_workspace(max(sp2.workspace_size(n, opts) for n in sizes), dev)
    for h, o, d in zip(hs, occ, outs):
        sp2.density(h, o, precision=args.precision, out=d, workspace=single_ws)
    torch.cuda.synchronize()
    t2 = time.perf_counter()
    for h, o, d in zip(hs, occ, outs):
        sp2.density(h, o, precision=args.precision, out=d, workspace=single_ws)
    torch.cuda.synchronize()
    seq_ms = (time.perf_counter() - t2) * 1e3
    _, infos = step()
    torch.cuda.synchronize()
    log("batched: %.2f ms per call (%.1f TFLOP/s); one call per problem: %.2f ms" % (ms, value, seq_ms))
    out = {
        "metric": "batched SP2 TFLOP/s (64 Hamiltonians of uneven sizes, one graph launch)",
        "value": round(value, 3), "unit": "TFLOP/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": round(ms, 3), "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f16" if args.precision == "fp16x2" else args.precision, "data": "synthetic",
        "config": {"workload": "64 Hamiltonians, N_i = 64*U{4..48} (%d..%d, sum %d), occupation U[0.2,0.5], "
                               "gap U[0.5,3] eV; Gershgorin bounds" % (min(sizes), max(sizes), sum(sizes)),
                   "precision": args.precision, "tile": infos[0]["tile"]},
        "flop_per_call": flop,
        "layers": {"min": min(i["layers"] for i in infos), "max": max(i["layers"] for i in infos)},
        "status": sorted(set(i["status_name"] for i in infos)),
        "sequential_ms": round(seq_ms, 3), "speedup_vs_sequential": round(seq_ms / ms, 3),
        "roofline": {"bound": "mfma", "achieved": round(value, 3), "peak": PEAK_FP16_TFLOPS, "unit": "TFLOP/s",
                     "frac": round(value / PEAK_FP16_TFLOPS, 4), "traffic": None,
                     "kernel": "whole batched call (grouped squaring kernels dominate)"},
    }
    if not args.no_accel:
        # the same batch with each problem's HOMO/LUMO values (sp2_density_batched_gap)
        gaps = [(w.homo, w.lumo) for w in ws]
        souts = [torch.empty_like(h) for h in hs]
        sp2.density_batched(hs, occ, precision=args.precision, outs=souts, workspace=wsbuf, gaps=gaps)
        torch.cuda.synchronize()
        t3 = time.perf_counter()
        each = []
        for _ in range(args.steps):
            tc = time.perf_counter()
            _, ainfos = sp2.density_batched(hs, occ, precision=args.precision, outs=souts, workspace=wsbuf, gaps=gaps)
            each.append(round((time.perf_counter() - tc) * 1e3, 2))
        torch.cuda.synchronize()
        ams = (time.perf_counter() - t3) * 1e3 / args.steps
        out["accelerated"] = {"ms_per_call": round(ams, 3), "ms_each_call": each, "speedup_vs_plain": round(ms / ams, 3),
                              "layers": {"min": min(i["layers"] for i in ainfos),
                                         "max": max(i["layers"] for i in ainfos)},
                              "status": sorted(set(i["status_name"] for i in ainfos))}
        log("batched accelerated: %.2f ms per call, layers %d..%d" % (ams, out["accelerated"]["layers"]["min"],
                                                                     out["accelerated"]["layers"]["max"]))
    if not args.no_cpu_baseline:
        from oracle import dm as odm
        from oracle import sp2 as osp2

        w0 = ws[int(np.argmax(sizes))]
        tc = time.perf_counter()
        osp2.sp2_alg1(w0.h, w0.n_occ, max_layers=4, refine=False)
        tcpu = time.perf_counter() - tc
        out["cpu_baseline"] = {"value": round(4 * 2.0 * w0.n ** 3 / tcpu / 1e12, 4), "unit": "TFLOP/s",
                               "cores": int(_cores()), "kind": "oracle",
                               "sample": "first 4 FP64 layers of Alg. 1 (oracle.sp2.sp2_alg1) on the largest "
                                         "problem (N=%d), %.1f s; rate credits 2N^3 per layer" % (w0.n, tcpu)}
        errs = [float(np.linalg.norm(d.cpu().numpy() - odm.dm_construct(w.q, w.eps, w.n_occ))) / np.sqrt(w.n)
                for w, d in zip(ws, outs)]
        out["accuracy"] = {"max_fro_error_over_sqrt_n": max(errs), "bound_over_sqrt_n": 1e-3,
                           "max_trace_error": max(abs(i["trace"] - w.n_occ) for i, w in zip(infos, ws))}
        if "accelerated" in out:
            aerrs = [float(np.linalg.norm(d.cpu().numpy() - odm.dm_construct(w.q, w.eps, w.n_occ))) / np.sqrt(w.n)
                     for w, d in zip(ws, souts)]
            out["accelerated"]["max_fro_error_over_sqrt_n"] = max(aerrs)
            out["accelerated"]["max_trace_error"] = max(abs(i["trace"] - w.n_occ) for i, w in zip(ainfos, ws))
    print(json.dumps(out), flush=True)


def bench_net(args):
    """The 20-layer network X_{k+1} = W_k X_k^2 + B_k X_k + c_k I at N = 2048 (spectrum
    U[-15,15] eV, mu = 0, kT = 0.2 eV target): one step = forward (split squarings) +
    backward (FP32 adjoint, plus checkpoint recomputation where the library keeps only every
    c-th layer) for the loss ||X_20 - T||_F^2."""
    import numpy as np
    import torch

    from paper_2101_06385_amd import sp2, workloads

    dev = torch.device("cuda:0")
    n, K = 2048, 20
    w = workloads.config5(device=None if args.gen_device == "cpu" else "cuda:0")
    # input layer from bounds that enclose the spectrum; alternating SP2 branch coefficients
    # X^2 and 2X - X^2 (both keep the spectrum in [0, 1])
    e1, en = float(w.eps.min()) - 0.5, float(w.eps.max()) + 0.5
    x0 = torch.from_numpy(((en * np.eye(n) - w.h) / (en - e1)).astype(np.float32)).to(dev)
    coef = [(1.0, 0.0, 0.0) if k % 2 == 0 else (-1.0, 2.0, 0.0) for k in range(K)]
    wt = torch.tensor([c[0] for c in coef], dtype=torch.float32, device=dev)
    bt = torch.tensor([c[1] for c in coef], dtype=torch.float32, device=dev)
    ct = torch.tensor([c[2] for c in coef], dtype=torch.float32, device=dev)
    q = torch.from_numpy(w.q).to(dev)
    fd = torch.from_numpy(1.0 / (1.0 + np.exp(w.eps / 0.2))).to(dev)
    target = ((q * fd) @ q.T).float()
    wsb = sp2.alloc_workspace(sp2.net_workspace_size(n, K, args.precision), dev)

    def step():
        xk, _ = sp2.net_forward(x0, wt, bt, ct, precision=args.precision, workspace=wsb)
        gk = 2.0 * (xk - target)
        return sp2.net_backward(gk, wt, bt, ct, wsb, precision=args.precision, want_g0=False), xk

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    e = [torch.cuda.Event(enable_timing=True) for _ in range(3)]
    fwd, bwd = [], []
    t0 = time.perf_counter()
    for _ in range(args.steps):
        e[0].record()
        xk, _ = sp2.net_forward(x0, wt, bt, ct, precision=args.precision, workspace=wsb)
        e[1].record()
        gk = 2.0 * (xk - target)
        sp2.net_backward(gk, wt, bt, ct, wsb, precision=args.precision, want_g0=False)
        e[2].record()
        torch.cuda.synchronize()
        fwd.append(e[0].elapsed_time(e[1]))
        bwd.append(e[1].elapsed_time(e[2]))
    ms = (time.perf_counter() - t0) * 1e3 / args.steps
    # checkpoint spacing of ckpt_every = 0: every layer kept when the workspace equals that of
    # c = 1, else ceil(sqrt(K))
    keep_all = sp2.net_workspace_size(n, K, args.precision, 0) == sp2.net_workspace_size(n, K, args.precision, 1)
    c = 1 if keep_all else int(math.ceil(math.sqrt(K)))
    recompute = K - (K + c - 1) // c
    f_fwd = K * flop_split_layer(n)
    f_bwd = recompute * flop_split_layer(n) + K * 2 * flop_plain_layer(n)
    value = (f_fwd + f_bwd) / (ms * 1e-3) / 1e12
    log("net: step %.2f ms (forward %.2f ms, backward %.2f ms), %.1f TFLOP/s" % (ms, np.mean(fwd), np.mean(bwd), value))
    out = {
        "metric": "differentiable SP2 network TFLOP/s (forward + backward, N=2048, 20 layers)",
        "value": round(value, 3), "unit": "TFLOP/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": round(ms, 3), "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f16 forward / f32 adjoint", "data": "synthetic",
        "config": {"workload": "network N=2048, K=20, spectrum U[-15,15] eV, target Fermi-Dirac kT=0.2 eV, "
                               + ("every layer kept (no recomputation)" if c == 1 else "checkpoints every %d layers" % c),
                   "precision": args.precision},
        "forward_ms": round(float(np.mean(fwd)), 3), "backward_ms": round(float(np.mean(bwd)), 3),
        "forward_tflops": round(f_fwd / (np.mean(fwd) * 1e-3) / 1e12, 3),
        "backward_tflops": round(f_bwd / (np.mean(bwd) * 1e-3) / 1e12, 3),
        "roofline": {"bound": "mfma", "achieved": round(f_fwd / (np.mean(fwd) * 1e-3) / 1e12, 3),
                     "peak": PEAK_FP16_TFLOPS, "unit": "TFLOP/s",
                     "frac": round(f_fwd / (np.mean(fwd) * 1e-3) / 1e12 / PEAK_FP16_TFLOPS, 4), "traffic": None,
                     "kernel": "forward layers (split squaring kernel); the adjoint runs on the FP32 peak 157.3"},
    }
    print(json.dumps(out), flush=True)


def bench_sweep(args):
    """The headline measurement across sizes (the small-gap stress spectrum at each N):
    layers, loop rate, squaring-kernel rate and time-to-D of FP16X2 Alg. 1 and of FP64 SP2."""
    import numpy as np
    import torch

    from paper_2101_06385_amd import sp2, workloads

    dev = torch.device("cuda:0")
    gen = None if args.gen_device == "cpu" else "cuda:0"
    rows = []
    for n in (1024, 2048, 4096, 6144, 8192, 12288, 16384):
        w = workloads.config3(n=n, device=gen)
        h = torch.from_numpy(w.h).to(dev)
        d = torch.empty_like(h)
        ws = sp2.alloc_workspace(sp2.workspace_size(n, sp2.options(args.precision)), dev)
        sp2.density(h, w.n_occ, precision=args.precision, out=d, workspace=ws)
        torch.cuda.synchronize()
        reps = 3
        t0 = time.perf_counter()
        for _ in range(reps):
            _, info, tm = sp2.density(h, w.n_occ, precision=args.precision, out=d, workspace=ws, timed=True)
        torch.cuda.synchronize()
        ms = (time.perf_counter() - t0) * 1e3 / reps
        k = tm["squarings"]
        f_layer = flop_split_layer(n)
        sq = float(np.mean(tm["square_ms"][:k]))
        row = {"n": n, "layers": info["layers"], "tile": info["tile"], "kernel": info["kernel"],
               "time_to_d_ms": round(ms, 3), "loop_tflops": round(k * f_layer / (tm["loop_active_ms"] * 1e-3) / 1e12, 1),
               "kernel_tflops": round(f_layer / (sq * 1e-3) / 1e12, 1),
               "frac": round(f_layer / (sq * 1e-3) / 1e12 / PEAK_FP16_TFLOPS, 4),
               "refine_ms": round(tm["refine_ms"], 3), "status": info["status_name"]}
        if n <= 8192:
            _, i64, t64 = sp2.density(h, w.n_occ, precision="fp64", timed=True)
            row["fp64_time_to_d_ms"] = round(t64["total_ms"], 3)
        rows.append(row)
        log("sweep n=%d: %s" % (n, row))
        del h, d, ws
        torch.cuda.empty_cache()
    big = [r for r in rows if r["n"] == 8192][0]
    out = {"metric": "SP2 squaring-kernel TFLOP/s and time-to-D across N (FP16X2, small-gap stress spectrum)",
           "value": big["kernel_tflops"], "unit": "TFLOP/s", "n_gpus": 1, "steps": 3, "warmup": 1,
           "ms_per_step": big["time_to_d_ms"], "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
           "dtype": "f16" if args.precision == "fp16x2" else args.precision, "data": "synthetic",
           "config": {"workload": "small-gap stress spectrum at N = 1024 .. 16384", "precision": args.precision},
           "rows": rows}
    print(json.dumps(out), flush=True)


def bench_md(args):
    """A molecular-dynamics-like sequence at N (default 8192, the small-gap stress spectrum):
    between calls the eigenvalues move by up to 5 meV and the basis is rotated slightly.  The
    first call runs Alg. 1; every later one runs the accelerated layers with the HOMO/LUMO
    estimate from the previous call's history (sp2_estimate_gap).  Each call is timed."""
    import numpy as np
    import torch

    from paper_2101_06385_amd import sp2, workloads

    dev = torch.device("cuda:0")
    n = args.n
    n_occ = n // 4
    rng = np.random.default_rng(8000 + n)
    eps = workloads.gapped_spectrum(rng, n, n_occ, -25.0, -12.55, -12.35, 25.0)
    gen = None if args.gen_device == "cpu" else "cuda:0"
    q = workloads.haar_orthogonal(rng, n, gen)
    d = torch.empty((n, n), dtype=torch.float64, device=dev)
    ws = sp2.alloc_workspace(sp2.workspace_size(n, sp2.options(args.precision, gap=(-1.0, 1.0))), dev)
    calls = []
    est = None
    for step in range(args.steps + 1):
        h = torch.from_numpy(workloads.symmetric_from_eigen(q, eps, gen)).to(dev)
        if step == 0:   # warm the kernels up once, untimed
            sp2.density(h, n_occ, precision=args.precision, out=d, workspace=ws)
        inside = None if est is None else bool(eps[n_occ - 1] <= est[0] < est[1] <= eps[n_occ])
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        _, info = sp2.density(h, n_occ, precision=args.precision, out=d, workspace=ws, gap=est)
        torch.cuda.synchronize()
        ms = (time.perf_counter() - t0) * 1e3
        calls.append({"ms": round(ms, 3), "layers": info["layers"], "accelerated": info["accelerated"],
                      "status": info["status_name"], "gap_violation": info["gap_violation"],
                      "estimate_inside_gap": inside})
        log("md step %d: %.2f ms, layers %d (%d accelerated), %s" % (step, ms, info["layers"], info["accelerated"],
                                                                   info["status_name"]))
        new = sp2.estimate_gap(info, n, args.precision)
        if new is not None:
            est = new
        if step < args.steps:
            eps = np.sort(eps + rng.uniform(-0.005, 0.005, n))
            g = rng.standard_normal((n, n))
            if gen is None:
                qn, r = np.linalg.qr(q + 1e-3 * g)
                q = qn * np.sign(np.diag(r))[None, :]
            else:
                qt, rt = torch.linalg.qr(torch.from_numpy(q + 1e-3 * g).to(gen))
                q = (qt * torch.sign(torch.diagonal(rt))[None, :]).cpu().numpy()
    acc = [c["ms"] for c in calls[1:]]
    out = {
        "metric": "time-to-D per call of a molecular-dynamics-like sequence at N=%d (first call Alg. 1, "
                  "then accelerated layers from the previous call's HOMO/LUMO estimate)" % n,
        "value": round(float(np.mean(acc)), 3), "unit": "ms", "n_gpus": 1, "steps": args.steps, "warmup": 1,
        "ms_per_step": round(float(np.mean(acc)), 3), "higher_is_better": False, "scaling": "weak",
        "vs_baseline": None, "dtype": "f16" if args.precision == "fp16x2" else args.precision, "data": "synthetic",
        "config": {"workload": "N=%d small-gap stress spectrum, 0.2 eV gap at 25%% occupation; per step eigenvalues "
                               "move by U[-5,5] meV and the basis by QR(Q + 1e-3 G); Gershgorin bounds" % n,
                   "precision": args.precision},
        "plain_ms": calls[0]["ms"], "speedup_vs_plain": round(calls[0]["ms"] / float(np.mean(acc)), 3),
        "calls": calls,
    }
    print(json.dumps(out), flush=True)


def bench_fermi(args):
    """The optimized finite-temperature expansion of the paper's example (11 layers, beta = 40
    and mu = 1/2 in the rescaled energy) fitted on the host and applied to an N x N
    Hamiltonian (spectrum U[-15,15] eV, Gershgorin bounds): one step = sp2_fermi_apply."""
    import numpy as np
    import torch

    from paper_2101_06385_amd import sp2, workloads

    dev = torch.device("cuda:0")
    n, L = args.n, 11
    rng = np.random.default_rng(7000 + n)
    eps = np.sort(rng.uniform(-15.0, 15.0, n))
    gen = None if args.gen_device == "cpu" else "cuda:0"
    q = workloads.haar_orthogonal(rng, n, gen)
    h = torch.from_numpy(workloads.symmetric_from_eigen(q, eps, gen)).to(dev)
    bounds = sp2.spectral_bounds(h)
    span = bounds[1] - bounds[0]
    t0 = time.perf_counter()
    theta, c, loss = sp2.fermi_fit(L, bounds[0] + 0.5 * span, span / 40.0, bounds)
    fit_ms = (time.perf_counter() - t0) * 1e3
    out_d = torch.empty_like(h)
    ws = sp2.alloc_workspace(sp2.fermi_workspace_size(n, bounds, args.precision), dev)
    for _ in range(args.warmup):
        sp2.fermi_apply(h, theta, c, bounds, precision=args.precision, out=out_d, workspace=ws, observables=False)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    for _ in range(args.steps):
        sp2.fermi_apply(h, theta, c, bounds, precision=args.precision, out=out_d, workspace=ws, observables=False)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t1) * 1e3 / args.steps
    split = args.precision in ("fp16x2", "bf16x2")
    flop = L * (flop_split_layer(n) if split else flop_plain_layer(n))
    value = flop / (ms * 1e-3) / 1e12
    _, obs = sp2.fermi_apply(h, theta, c, bounds, precision=args.precision, out=out_d, workspace=ws)
    log("fermi: %d layers at N=%d, %.2f ms per call, %.1f TFLOP/s; fit %.0f ms on the host, loss %.2e"
        % (L, n, ms, value, fit_ms, loss))
    out = {
        "metric": "optimized finite-temperature SP2 expansion TFLOP/s (N=%d, 11 layers, beta=40)" % n,
        "value": round(value, 3), "unit": "TFLOP/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": round(ms, 3), "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f16" if args.precision == "fp16x2" else args.precision, "data": "synthetic",
        "config": {"workload": "Fermi operator N=%d, spectrum U[-15,15] eV, Gershgorin bounds, 11 layers fitted "
                               "for beta=40, mu=1/2 in the rescaled energy" % n, "precision": args.precision},
        "fit_ms_host": round(fit_ms, 1), "fit_loss": loss, "trace": obs[0],
    }
    if not args.no_cpu_baseline:
        from oracle import fermi as ofermi

        x = (eps - bounds[0]) / span
        vals = ofermi.model_scalar(x, theta, c)
        rows = [0, n // 2, n - 1]
        ref = (q[rows] * vals[None, :]) @ q.T
        d_rows = out_d[rows].cpu().numpy()
        fd = ofermi.fermi(x, 40.0, 0.5)
        exact = (q[rows] * fd[None, :]) @ q.T
        out["accuracy"] = {"max_err_vs_network_rows": float(np.abs(d_rows - ref).max()),
                           "max_err_vs_fermi_rows": float(np.abs(d_rows - exact).max()),
                           "trace_vs_network": float(obs[0] - vals.sum()),
                           "fit_max_err_on_spectrum": float(np.abs(vals - fd).max())}
        log("fermi accuracy: %s" % out["accuracy"])
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
