"""Benchmark: unknowns solved per second of the Q^4 SEM fast-diagonalisation
solve of -Lap u + alpha u = f at n = 999 per axis (250^3 elements, alpha = 1,
homogeneous Dirichlet on [-1, 1]^3, ~1e9 unknowns), on one MI355X.

Variants (each timed over K steps; one step = one complete solve of a right-hand
side already resident in HBM):
  f64     sem_solve: six FP64 mode products with the fused eigenvalue divide;
  f32 / bf16 / bf16x3 refined
          sem_solve_refined: low-precision mode products + FP64 residual and
          update, iterated until the update or the remaining error predicted from
          the contraction of the updates is <= 1e-10 ||u|| (every iteration,
          residual and norm read-back inside the timed region).
Each refined result is checked against the FP64 solve (relative max error); the
headline value is the fastest variant within 1e-10.

    python bench.py [--steps K] [--warmup W] [--gpus 1] [--no-cpu-baseline] [--variants f64,bf16,...]

Prints one JSON line.  Besides the headline value it reports the dominant
kernel's roofline fraction (per-launch duration measured with HIP events on the
stream the kernels run on) and the CPU oracle timed on this host.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "unknowns solved/s, FP64 vs refined FP32/BF16 at 1e-10 rel err, Q^4 n=999"
PEAK_FP64_TFLOPS = 78.6
PEAK_FP32_TFLOPS = 157.3
PEAK_BF16_TFLOPS = 2516.6
PEAK_HBM_GBS = 8000.0


def log(msg: str) -> None:
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


def host_info() -> dict:
    """Host cores for the CPU baseline: nproc, the CPUs this process may run on, the
    CPU model, and the threads the BLAS behind numpy's matmul actually uses."""
    model = "unknown"
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    try:
        affinity = len(os.sched_getaffinity(0))
    except AttributeError:  # pragma: no cover
        affinity = os.cpu_count()
    threads = None
    try:
        from threadpoolctl import threadpool_info
        threads = max((i.get("num_threads", 1) for i in threadpool_info() if i.get("user_api") == "blas"),
                      default=None)
    except Exception:  # pragma: no cover
        pass
    return {"nproc": os.cpu_count(), "affinity_cpus": affinity, "cpu_model": model,
            "blas_threads": int(threads or affinity)}


def bench_batch(args, P, torch, dev, log):
    """Batched workload: args.batch problems, k in {2..8}, 8..64 elements per axis,
    alpha ~ U[0, 10], N(0,1) right-hand sides (seed 2311); FP64 refinement to
    ||delta|| <= tol ||u||.  Two batch precisions are timed: FP32 mode products for
    every problem (one persistent launch per pass), and SEM_BF16X3, where the
    problems with every dimension >= 96 run split-BF16 passes; the faster one is
    reported."""
    from concurrent.futures import ThreadPoolExecutor

    from workloads import batch_draws, batch_rhs
    specs = batch_draws(args.batch, 2311)
    box = (-1.0, 1.0, -1.0, 1.0, -1.0, 1.0)
    t0 = time.perf_counter()
    plans = [P.Plan(s["k"], s["ne"], box, s["alpha"], "dirichlet") for s in specs]
    batch = P.Batch(plans)
    plan_s = time.perf_counter() - t0
    total = sum(p.numel for p in plans)
    log(f"batch: {len(plans)} plans, {total} unknowns, created + tuned in {plan_s:.1f}s, "
        f"tile rows per bucket {batch.tile_rows()}")
    with ThreadPoolExecutor(16) as ex:
        hosts = list(ex.map(lambda ip: batch_rhs(ip[1].shape, 2311, ip[0]), enumerate(plans)))
    fs = [torch.from_numpy(h).to(dev) for h in hosts]
    stream = torch.cuda.current_stream(dev)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    reps = max(1, min(args.steps, 3))
    per_prec, outs = {}, {}
    for prec in ("f32", "bf16x3"):
        us = [torch.empty_like(f) for f in fs]
        torch.cuda.synchronize()
        its, st = batch.solve(fs, us, prec=prec, tol=args.tol, max_iter=40, raise_on_error=False)  # warm-up
        torch.cuda.synchronize()
        e0.record(stream)
        for _ in range(reps):
            its, st = batch.solve(fs, us, prec=prec, tol=args.tol, max_iter=40, raise_on_error=False)
        e1.record(stream)
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1) / reps
        log(f"batch solve {prec}: {ms:.1f} ms, {total / (ms * 1e-3):.3e} unknowns/s, "
            f"iterations {min(its)}..{max(its)}, status {st}")
        # algorithmic mode-product flop: 4 N (n_x + n_y + n_z) per FD application,
        # one application per refinement iteration of each problem
        flop = sum(4.0 * pl.numel * sum(pl.shape) * it for pl, it in zip(plans, its))
        per_prec[prec] = {"ms_per_batch": ms, "unknowns_per_s": total / (ms * 1e-3),
                          "iterations": [min(its), max(its)], "status": st,
                          "mode_product_tflops": flop / (ms * 1e-3) / 1e12}
        outs[prec] = us
    best = min((p for p in per_prec if per_prec[p]["status"] == 0), key=lambda p: per_prec[p]["ms_per_batch"],
               default="f32")
    nsplit = sum(1 for p in plans if min(p.shape) >= 96)
    res = {"workload": f"{len(plans)} independent Q^k Helmholtz solves, k in 2..8, 8..64 elements per axis, "
                       f"alpha in [0,10], Dirichlet [-1,1]^3, N(0,1) rhs (seed 2311)",
           "unknowns": total, "precision": best, **per_prec[best], "by_precision": per_prec,
           "tile_rows": batch.tile_rows(), "setup_seconds": plan_s,
           "dtype": ("f32 mode products" if best == "f32" else
                     f"split-bf16 mode products for the {nsplit} problems with every dimension >= 96, "
                     f"f32 for the rest") + ", f64 residual/update"}
    # mode products: FP32 MFMA in the FP32 batch (the split problems of the
    # SEM_BF16X3 batch issue four BF16 MFMAs per product)
    mp = per_prec["f32"]["mode_product_tflops"]
    res["roofline"] = {"bound": "mfma", "kernel": "FP32 batch, all passes (4 N (nx+ny+nz) flop per iteration)",
                       "achieved": mp, "peak": PEAK_FP32_TFLOPS, "unit": "TFLOP/s", "frac": mp / PEAK_FP32_TFLOPS}
    if not args.no_cpu_baseline:
        import oracle as O
        # the four largest problems, the two smallest and (split BF16) the two
        # smallest split ones, each against a full oracle solve; the oracle's time
        # on them is the batch's CPU baseline
        order = sorted(range(len(plans)), key=lambda i: plans[i].numel)
        check = order[-4:] + order[:2]
        if best == "bf16x3":
            check += [i for i in order if min(plans[i].shape) >= 96][:2]
        errs, cpu_s, cpu_n = [], 0.0, 0
        for i in check:
            s = specs[i]
            prob = O.Problem(s["k"], s["ne"], box, s["alpha"], "dirichlet")
            t0 = time.perf_counter()
            ref = O.fd_solve(prob, hosts[i])
            cpu_s += time.perf_counter() - t0
            cpu_n += plans[i].numel
            errs.append(O.rel_max_err(outs[best][i].cpu().numpy(), ref))
            del ref
        res["rel_max_err_vs_oracle_checked"] = max(errs)
        res["oracle_checked_problems"] = len(check)
        host = host_info()
        res["cpu_baseline"] = {"value": cpu_n / cpu_s, "unit": "unknowns/s", "cores": host["blas_threads"],
                               "kind": "oracle", "sample": f"oracle FP64 solves of the {len(check)} checked problems "
                                                           f"({cpu_n} unknowns, {cpu_s:.1f} s)",
                               "cpu_model": host["cpu_model"]}
        log(f"batch: rel err vs oracle {max(errs):.2e} ({len(check)} problems, the 4 largest among them); "
            f"oracle {cpu_n / cpu_s:.3e} unknowns/s")
    del fs, outs, batch, plans
    torch.cuda.empty_cache()
    return res


def bench_schrodinger(args, P, torch, dev, log):
    """Variable coefficients (the paper's Schrodinger-equation section): alpha u -
    Lap u + V u = f on [-16, 16]^3, periodic as in the paper, Q^5 with
    args.schrodinger_ne^3 elements (200 -> n = 1000, the 1000^3 DoFs of Table tab5),
    alpha = 1, V from eq. (beta)
    with beta = 1, f from the exact solution cos(pi x/16) cos(pi y/16) cos(pi z/16);
    PCG with the FD solve of ((alpha + beta/2) I - Lap) as preconditioner, in FP64
    and in split BF16, to ||r||_M <= 1e-12 ||f||_M."""
    from workloads import SCHRODINGER_BOX, schrodinger_data
    ne, alpha, beta = args.schrodinger_ne, 1.0, 1.0
    t0 = time.perf_counter()
    plan = P.Plan(5, (ne, ne, ne), SCHRODINGER_BOX, alpha, "periodic")
    plan_s = time.perf_counter() - t0
    v, ue, f = schrodinger_data(*(plan.nodes(a) for a in range(3)), alpha, beta)
    vd, fd, ued = (torch.from_numpy(a).to(dev) for a in (v, f, ue))
    del v, f, ue
    n = plan.numel
    stream = torch.cuda.current_stream(dev)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    res = {"workload": f"alpha u - Lap u + V u = f, V = beta sin^2(pi x/4) sin^2(pi y/4) sin^2(pi z/4), "
                       f"beta = {beta:g}, alpha = {alpha:g}, [-16,16]^3 periodic, Q^5, {ne}^3 elements "
                       f"(n={plan.shape[0]}), PCG with the FD preconditioner (shift alpha + beta/2), "
                       f"tol 1e-12",
           "unknowns": n, "plan_seconds": plan_s,
           "paper_context": "Table tab5: 20.4 s on one A100 (MATLAB, FP64, periodic Q^5, 1000^3 DoFs, 10 iterations)",
           "by_preconditioner": {}}
    u = torch.empty_like(fd)
    for prec in ("f64", "bf16x3"):
        plan.pcg_solve(vd, fd, u, prec=prec, tol=1e-12)  # warm-up; default shift alpha + max(V)/2
        torch.cuda.synchronize()
        e0.record(stream)
        _, it, rel, st = plan.pcg_solve(vd, fd, u, prec=prec, tol=1e-12, raise_on_error=False)
        e1.record(stream)
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1)
        err = float((u - ued).abs().max())
        log(f"schrodinger {prec} preconditioner: {ms:.1f} ms per solve, {it} iterations, "
            f"rel residual {rel:.1e}, max error vs exact {err:.2e}, {n / (ms * 1e-3):.3e} unknowns/s")
        res["by_preconditioner"][prec] = {"ms_per_solve": ms, "iterations": it, "rel_residual": rel,
                                          "max_err_vs_exact": err, "unknowns_per_s": n / (ms * 1e-3),
                                          "status": st}
    ok = [p for p, r in res["by_preconditioner"].items() if r["status"] == 0]
    best = min(ok, key=lambda p: res["by_preconditioner"][p]["ms_per_solve"], default="f64")
    res.update({"preconditioner": best, **res["by_preconditioner"][best]})
    # the preconditioner's mode products dominate: their flop, 4 N (nx + ny + nz)
    # per application (the products as defined; the reflection-split products
    # execute half of it), over the whole solve time
    nx, ny, nz = plan.shape
    it_b = res["by_preconditioner"][best]["iterations"]
    fd_flop = 4.0 * n * (nx + ny + nz) * (it_b + 1)
    ach = fd_flop / (res["by_preconditioner"][best]["ms_per_solve"] * 1e-3) / 1e12
    peak = {"f64": PEAK_FP64_TFLOPS, "f32": PEAK_FP32_TFLOPS}.get(best, PEAK_BF16_TFLOPS)
    res["roofline"] = {"bound": "mfma", "kernel": "whole PCG solve, preconditioner mode products counted",
                       "achieved": ach, "peak": peak, "unit": "TFLOP/s", "frac": ach / peak,
                       "executed_frac": ach / peak / 2.0}
    res["tuned_shapes"] = plan.tuning(best) if best != "f64" else None
    del u, vd, fd, ued, plan
    torch.cuda.empty_cache()
    if not args.no_cpu_baseline:
        import oracle as O
        # a reduced mesh of the same problem against the oracle's PCG
        ne_s = 40
        prob = O.Problem(5, (ne_s,) * 3, SCHRODINGER_BOX, alpha, "periodic")
        v, ue, f = schrodinger_data(*(o.x for o in prob.axes), alpha, beta)
        t0 = time.perf_counter()
        ref, it_ref, _ = O.pcg_schrodinger(prob, v, f, alpha + beta / 2, tol=1e-12)
        cpu_s = time.perf_counter() - t0
        plan = P.Plan(5, (ne_s,) * 3, SCHRODINGER_BOX, alpha, "periodic")
        vd, fd = torch.from_numpy(v).to(dev), torch.from_numpy(f).to(dev)
        u, it, rel, st = plan.pcg_solve(vd, fd, prec=best, tol=1e-12, raise_on_error=False)
        err = O.rel_max_err(u.cpu().numpy(), ref)
        host = host_info()
        log(f"schrodinger n={prob.shape[0]}^3 vs oracle PCG: {it} iterations (oracle {it_ref}), rel err {err:.2e}; "
            f"oracle {cpu_s:.1f} s")
        res["oracle_check"] = {"n": prob.shape[0], "iterations": it, "oracle_iterations": it_ref,
                               "rel_max_err_vs_oracle": err, "preconditioner": best}
        res["cpu_baseline"] = {"value": prob.shape[0] ** 3 / cpu_s, "unit": "unknowns/s",
                               "cores": host["blas_threads"], "kind": "oracle",
                               "sample": f"oracle PCG at n={prob.shape[0]}^3 ({it_ref} iterations, {cpu_s:.1f} s)",
                               "cpu_model": host["cpu_model"]}
        del u, vd, fd, plan
        torch.cuda.empty_cache()
    return res


# HBM bytes per launch from rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE runs of the
# current kernels at n = 999, scaled by a device copy of known size (FETCH x 2.000,
# WRITE x 1.000); recorded here because counters cannot be read inside the timed
# run.  Variants without such runs report null.
PROFILED_TRAFFIC = {
    # one dense FP64 y-axis mode product (mode_nn_f64, sem_mode_product)
    "f64": {"fetch_bytes": 20.70e9, "write_bytes": 8.17e9, "algorithmic_bytes": 15.97e9,
            "mfma_flops_counted": 2.112e12, "mfma_busy": 0.836, "source": "profiles/mode_f64_n999.md"},
    # one split-BF16 FD application (conversion, six passes, unfold)
    "bf16x3": {"fetch_bytes": 43.5e9, "write_bytes": 36.7e9, "source": "profiles/split_bf16_refined_n999.md"},
}

# The kernel whose launch the headline roofline times, per low-precision variant.
KERNEL_NAME = {
    "bf16x3": "mode_rot_dma<BF16X3, bf16, STORE, COL_FOLD> (z forward, y fold)",
    "bf16": "mode_rot_dma<BF16, bf16, STORE, COL_FOLD> (z forward, y fold)",
    "f32": "mode_rot_f32<f32, f32, STORE> (z forward)",
}
# rocprofv3 counters of that kernel at n = 999 (per launch; HBM bytes scaled as
# above; MFMA ops = SQ_INSTS_VALU_MFMA_MOPS_BF16 x 512; busy = SQ_VALU_MFMA_BUSY_CYCLES
# / (GRBM_GUI_ACTIVE per XCD x 1024 SIMDs)).  Variants without such runs: null.
PROFILED_KERNEL = {
    "bf16x3": {"fetch_bytes": 5.22e9, "write_bytes": 4.09e9, "algorithmic_bytes": 7.98e9,
               "mfma_flops_counted": 4.291e12, "mfma_busy": 0.557, "clock_ghz": 1.92,
               "source": "profiles/split_bf16_refined_n999.md"},
}


def _traffic(name):
    t = PROFILED_TRAFFIC.get(name)
    return None if t is None else t["fetch_bytes"] + t["write_bytes"]


def bench_ch(args, P, torch, dev, log):
    """Cahn-Hilliard IMEX stepping on [0, 2pi]^3, Neumann, Q^4, 64^3 elements
    (n = 257), eps = 0.05, m = 0.02, dt = 1e-4, phi_0 ~ U[-0.05, 0.05] (seed 2312);
    FP32 solve + 1 FP64 refinement sweep per step (2e-12 of the oracle's step),
    each step a HIP graph replay."""
    import math

    import numpy as np

    from workloads import ch_initial
    box = (0.0, 2 * math.pi, 0.0, 2 * math.pi, 0.0, 2 * math.pi)
    ch = P.CahnHilliard(4, (64, 64, 64), box, 0.05, 0.02, 1e-4, prec="f32", refine_sweeps=1)
    phi0 = ch_initial(ch.shape, 2312, 0.05)
    a = torch.from_numpy(phi0).to(dev)
    b = a.clone()
    ch.step(a, b, 3)  # capture + warm-up
    a.copy_(torch.from_numpy(phi0))
    b.copy_(a)
    stream = torch.cuda.current_stream(dev)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    e0.record(stream)
    ch.step(a, b, args.ch_steps)
    e1.record(stream)
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1)
    n = ch.numel
    phi = a.cpu().numpy()
    ax = [P.axis_host(4, 64, 0.0, 2 * math.pi, "neumann")["mass"]] * 3
    m3 = np.einsum("i,j,k->ijk", *ax)
    drift = abs(float(np.sum(m3 * phi)) - float(np.sum(m3 * phi0))) / float(np.sum(m3 * np.abs(phi0)))
    log(f"cahn-hilliard: {args.ch_steps} steps in {ms:.0f} ms ({ms / args.ch_steps:.3f} ms/step, "
        f"{n * args.ch_steps / (ms * 1e-3):.3e} unknown-steps/s), relative mass drift {drift:.1e}")
    # per step: one FP32 FD application (six mode products, 4 N (n_x + n_y + n_z) flop)
    # and the FP64 banded passes of the right-hand side and of the sweep
    nx, ny, nz = ch.shape
    fd_flop = 4.0 * n * (nx + ny + nz)
    ach = fd_flop / (ms / args.ch_steps * 1e-3) / 1e12
    res = {"workload": "Cahn-Hilliard IMEX (BDF2), [0,2pi]^3 Neumann, Q^4 64^3 elements, n=257, eps=0.05, "
                       "m=0.02, dt=1e-4, phi0 ~ U[-0.05,0.05] (seed 2312)",
           "steps": args.ch_steps, "ms_per_step": ms / args.ch_steps,
           "unknown_steps_per_s": n * args.ch_steps / (ms * 1e-3), "unknowns": n,
           "dtype": "f32 solve + 1 f64 refinement sweep", "graph": True, "relative_mass_drift": drift,
           "max_abs_phi": float(np.max(np.abs(phi))),
           "roofline": {"bound": "mfma", "kernel": "whole step (FD application counted: 4 N (nx+ny+nz) flop)",
                        "achieved": ach, "peak": PEAK_FP32_TFLOPS, "unit": "TFLOP/s", "frac": ach / PEAK_FP32_TFLOPS},
           "tuned_shapes": None}  # FP32 strips: no shape to tune
    if args.ch_oracle_steps > 0 and not args.no_cpu_baseline:
        import oracle as O
        # the same start, args.ch_oracle_steps steps on the GPU and in the oracle
        a.copy_(torch.from_numpy(phi0))
        b.copy_(a)
        ch.step(a, b, args.ch_oracle_steps)
        phi_gpu = a.cpu().numpy()
        prob = O.Problem(4, (64, 64, 64), box, 0.0, "neumann")
        cur, prev = phi0, phi0
        t0 = time.perf_counter()
        for _ in range(args.ch_oracle_steps):
            cur, prev = O.ch_step(prob, cur, prev, 0.05, 0.02, 1e-4), cur
        cpu_s = time.perf_counter() - t0
        err = O.rel_max_err(phi_gpu, cur)
        host = host_info()
        log(f"cahn-hilliard: after {args.ch_oracle_steps} steps rel max err vs oracle {err:.2e}; oracle "
            f"{cpu_s / args.ch_oracle_steps:.2f} s/step on {host['blas_threads']} threads")
        res["rel_err_vs_oracle"] = err
        res["rel_err_vs_oracle_after_steps"] = args.ch_oracle_steps
        res["cpu_baseline"] = {"value": n * args.ch_oracle_steps / cpu_s, "unit": "unknown-steps/s",
                               "cores": host["blas_threads"], "kind": "oracle",
                               "sample": f"{args.ch_oracle_steps} oracle steps of the same workload from the same "
                                         f"phi0, {cpu_s:.1f} s", "cpu_model": host["cpu_model"]}
    return res


def main() -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--ne", type=int, default=250, help="elements per axis (250 -> n = 999)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--kernel-reps", type=int, default=5)
    ap.add_argument("--variants", default="f64,f32,bf16,bf16x3")
    ap.add_argument("--tol", type=float, default=1e-10,
                    help="refinement stop: ||delta|| <= tol ||u|| or predicted remaining error <= tol")
    ap.add_argument("--batch", type=int, default=256,
                    help="problems in the batched leg (k in 2..8, 8..64 elements per axis); 0 skips it")
    ap.add_argument("--ch-steps", type=int, default=1000,
                    help="Cahn-Hilliard steps at n = 257 (64^3 Q^4 elements); 0 skips the leg")
    ap.add_argument("--ch-oracle-steps", type=int, default=20,
                    help="Cahn-Hilliard steps compared with (and timed in) the oracle; 0 skips")
    ap.add_argument("--schrodinger-ne", type=int, default=200,
                    help="elements per axis of the variable-coefficient PCG leg (0 = skip)")
    ap.add_argument("--calib-copy", action="store_true",
                    help="also run one plain elementwise copy of f (N*8 bytes read + written) so that HBM "
                         "counters of the kernels can be scaled against a kernel of known traffic")
    args = ap.parse_args()
    if args.gpus != 1:
        print(json.dumps({"error": "this build runs on one GPU only; multi-GPU sharding is design-only",
                          "n_gpus": args.gpus}))
        return 2

    import numpy as np
    import torch

    import paper_2310_00226_amd as P
    from workloads import helmholtz_rhs

    k, ne, alpha = 4, (args.ne,) * 3, 1.0
    box = (-1.0, 1.0, -1.0, 1.0, -1.0, 1.0)
    dev = torch.device("cuda", 0)
    torch.cuda.set_device(dev)

    t0 = time.perf_counter()
    plan = P.Plan(k, ne, box, alpha, "dirichlet")
    plan_s = time.perf_counter() - t0
    nx, ny, nz = plan.shape
    N = plan.numel
    log(f"plan {plan.shape} built in {plan_s:.2f}s")

    t0 = time.perf_counter()
    f_host = helmholtz_rhs(plan.nodes(0), plan.nodes(1), plan.nodes(2), alpha)
    log(f"inputs generated in {time.perf_counter() - t0:.1f}s")
    f = torch.from_numpy(f_host).to(dev)
    u = torch.empty_like(f)
    torch.cuda.synchronize()

    for _ in range(args.warmup):
        plan.solve(f, u)
    torch.cuda.synchronize()
    stream = torch.cuda.current_stream(dev)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    e0.record(stream)
    for _ in range(args.steps):
        plan.solve(f, u)
    e1.record(stream)
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / args.steps
    value = N / (ms * 1e-3)
    log(f"FP64 solve: {ms:.2f} ms/step, {value:.3e} unknowns/s")

    variants = {"f64": {"ms_per_solve": ms, "unknowns_per_s": value, "iterations": 1, "rel_err_vs_f64": 0.0}}
    outputs = {"f64": u}  # every variant's solution stays on the device for the oracle comparison
    want = [v for v in args.variants.split(",") if v and v != "f64"]
    if want:
        scale = float(u.abs().max())
        for prec in want:
            ur = torch.empty_like(f)
            outputs[f"{prec}_refined"] = ur
            _, it, rel, st = plan.solve_refined(f, ur, prec=prec, tol=args.tol, max_iter=40, raise_on_error=False)
            torch.cuda.synchronize()
            for _ in range(max(0, args.warmup - 1)):
                plan.solve_refined(f, ur, prec=prec, tol=args.tol, max_iter=40, raise_on_error=False)
            torch.cuda.synchronize()
            e0.record(stream)
            for _ in range(args.steps):
                _, it, rel, st = plan.solve_refined(f, ur, prec=prec, tol=args.tol, max_iter=40,
                                                    raise_on_error=False)
            e1.record(stream)
            torch.cuda.synchronize()
            vms = e0.elapsed_time(e1) / args.steps
            err = float((ur - u).abs().max()) / scale
            variants[f"{prec}_refined"] = {"ms_per_solve": vms, "unknowns_per_s": N / (vms * 1e-3),
                                           "iterations": it, "last_update_rel": rel, "status": st,
                                           "rel_err_vs_f64": err,
                                           # launch shapes the first solve tuned, per pass in order
                                           # (BF16 tile-order group; FP32 strips have none)
                                           "tuned_shapes": plan.tuning(prec)}
            log(f"{prec} refined: {vms:.2f} ms/solve, {N / (vms * 1e-3):.3e} unknowns/s, {it} iterations, "
                f"rel err vs FP64 {err:.2e}, status {st}")
    ok = {k: v for k, v in variants.items() if v["rel_err_vs_f64"] <= 1e-10 and v.get("status", 0) == 0}
    best = max(ok, key=lambda k: ok[k]["unknowns_per_s"])
    fd_flops = 4.0 * N * (nx + ny + nz)  # six dense mode products, 2 n_a N flop each
    nrep = [P.axis_fold_host(k, ne[a], box[2 * a], box[2 * a + 1], "dirichlet")["nrep"] for a in range(3)]
    folded_flops = 4.0 * N * sum(nrep)  # the reflection-split passes: half-length blocks

    # dominant kernel group of a refined variant: one low-precision FD application
    # (its six mode-product launches, the right-hand side conversion included),
    # timed alone with HIP events on the stream the kernels run on
    lowp_roof = None
    for name, v in variants.items():
        if name == "f64":
            continue
        # one low-precision FD application of this variant (right-hand-side
        # conversion and six mode-product launches), timed alone with HIP events on
        # the stream the kernels run on
        prec = name.split("_")[0]
        ul = torch.empty_like(f)
        plan.solve_lowp(f, ul, prec=prec)
        torch.cuda.synchronize()
        e0.record(stream)
        for _ in range(args.kernel_reps):
            plan.solve_lowp(f, ul, prec=prec)
        e1.record(stream)
        torch.cuda.synchronize()
        fd_ms = e0.elapsed_time(e1) / args.kernel_reps
        del ul
        peak = PEAK_FP32_TFLOPS if prec == "f32" else PEAK_BF16_TFLOPS
        # achieved counts the six mode products as defined, 4 N sum_a n_a flop per
        # application; all run the reflection-split transforms, whose products contract
        # half-length blocks and execute 4 N sum_a nrep_a (nrep_a = orbit
        # representatives of axis a, ~n_a / 2)
        executed = folded_flops
        ach = fd_flops / (fd_ms * 1e-3) / 1e12
        roof = {"bound": "mfma", "kernel": f"{prec} FD application: " +
                ("fold + six reflection-split mode_rot_dma passes + unfold" if prec != "f32" else
                 "five launches of reflection-split strips"),
                "achieved": ach, "peak": peak, "unit": "TFLOP/s", "frac": ach / peak,
                "traffic": _traffic(prec), "traffic_detail": PROFILED_TRAFFIC.get(prec),
                "launch_ms": fd_ms, "flops_per_launch": fd_flops, "executed_flops_per_launch": executed,
                "executed_frac": executed / (fd_ms * 1e-3) / 1e12 / peak,
                "mfma_products_per_flop": 4 if prec == "bf16x3" else 1}
        v["fd_application"] = roof
        log(f"{prec} FD application alone: {fd_ms:.2f} ms, {ach:.1f} TFLOP/s of the dense products "
            f"({ach / peak:.3f} of {peak} TFLOP/s), executed {executed / (fd_ms * 1e-3) / 1e12:.1f}")
        if name == best:
            lowp_roof = roof

    # dominant kernel of the winning low-precision variant: the pass that takes the
    # largest share of its solve, z forward with the y fold in its store (pass 1 of
    # the reflection-split sequence; for FP32 the z-forward mode_rot_f32),
    # launched alone through sem_lowp_pass and timed with HIP events on the plan's
    # stream (torch's current stream).  achieved counts 2 n flop per unknown, the
    # mode product as defined (the per-unit work of the measurement plan); the
    # reflection-split kernel executes 2 nrep of them, reported beside it.
    kernel_roof = None
    bprec = best.split("_")[0]
    if best != "f64":
        plan.lowp_pass(bprec, 0, 1)
        torch.cuda.synchronize()
        e0.record(stream)
        plan.lowp_pass(bprec, 0, args.kernel_reps)
        e1.record(stream)
        torch.cuda.synchronize()
        pass_ms = e0.elapsed_time(e1) / args.kernel_reps
        alg = 2.0 * N * nz
        executed = 2.0 * N * nrep[2] if bprec != "f32" else alg
        peak = PEAK_FP32_TFLOPS if bprec == "f32" else PEAK_BF16_TFLOPS
        ach = alg / (pass_ms * 1e-3) / 1e12
        prof = PROFILED_KERNEL.get(bprec)
        kernel_roof = {
            "bound": "mfma", "kernel": KERNEL_NAME[bprec], "achieved": ach, "peak": peak, "unit": "TFLOP/s",
            "frac": ach / peak, "traffic": None if prof is None else prof["fetch_bytes"] + prof["write_bytes"],
            "launch_ms": pass_ms, "flops_per_launch": alg, "executed_flops_per_launch": executed,
            "executed_frac": executed / (pass_ms * 1e-3) / 1e12 / peak,
            "counters": prof}
        log(f"{bprec} pass 1 alone ({KERNEL_NAME[bprec]}): {pass_ms:.3f} ms, {ach:.1f} TFLOP/s of the dense "
            f"product ({ach / peak:.3f} of {peak}), executed {executed / (pass_ms * 1e-3) / 1e12:.1f} TFLOP/s")

    # the batched NN mode product (y axis) of the FP64 solve, timed alone per launch
    tmp = torch.empty_like(f)
    plan.mode_product(1, False, f, tmp)
    torch.cuda.synchronize()
    e0.record(stream)
    for _ in range(args.kernel_reps):
        plan.mode_product(1, False, f, tmp)
    e1.record(stream)
    torch.cuda.synchronize()
    launch_ms = e0.elapsed_time(e1) / args.kernel_reps
    flops_launch = 2.0 * N * ny
    achieved = flops_launch / (launch_ms * 1e-3) / 1e12
    solve_tflops = fd_flops / (ms * 1e-3) / 1e12  # six mode products
    log(f"mode product (y, NN): {launch_ms:.3f} ms/launch, {achieved:.1f} TFLOP/s; solve {solve_tflops:.1f} TFLOP/s")
    # other spectral multipliers on the same FP64 transforms (only the third
    # forward product's epilogue differs from the solve)
    spectral = {}
    for kind, param in (("exp", 1e-3), ("power", 0.5)):
        plan.apply_spectral(kind, alpha, param, f, tmp)
        torch.cuda.synchronize()
        e0.record(stream)
        for _ in range(args.kernel_reps):
            plan.apply_spectral(kind, alpha, param, f, tmp)
        e1.record(stream)
        torch.cuda.synchronize()
        spectral[f"{kind}_ms"] = e0.elapsed_time(e1) / args.kernel_reps
    log(f"spectral multipliers (FP64): exp(-1e-3 (L + alpha)) {spectral['exp_ms']:.1f} ms, "
        f"(L + alpha)^-0.5 {spectral['power_ms']:.1f} ms per application")
    if args.calib_copy:
        tmp.copy_(f)           # device-to-device copy: reads and writes N * 8 bytes
        torch.neg(f, out=tmp)  # elementwise kernel with the same traffic
        torch.cuda.synchronize()
    del tmp

    out = {
        "metric": METRIC,
        "value": variants[best]["unknowns_per_s"],
        "unit": "unknowns/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": variants[best]["ms_per_solve"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64" if best == "f64" else best.split("_")[0] + " mode products, f64 residual/update",
        "best_variant": best,
        "variants": variants,
        "data": "synthetic: f = (3 pi^2 + 1) sin(pi x) sin(pi y) sin(pi z) + 1e-3 N(0,1), seed 2310",
        "config": {"workload": f"Q^4 SEM Helmholtz alpha=1, Dirichlet [-1,1]^3, {ne[0]}^3 elements, "
                               f"n={nx} per axis ({N} unknowns), fast-diagonalisation solve to 1e-10 relative "
                               f"error: {best.split('_')[0]} mode products with FP64 refinement"
                               if best != "f64" else
                               f"Q^4 SEM Helmholtz alpha=1, Dirichlet [-1,1]^3, {ne[0]}^3 elements, "
                               f"n={nx} per axis ({N} unknowns), FP64 fast-diagonalisation solve",
                   "k": k, "elements_per_axis": ne[0], "n": nx, "unknowns": N, "alpha": alpha},
        "solve_tflops": solve_tflops,
        "spectral_multipliers": {"workload": "u = g(H_3 + alpha) f at the same n, FP64: exp(-1e-3 x) and x^-0.5",
                                 **spectral},
        "plan_seconds": plan_s,
        "roofline_f64": {"bound": "mfma", "kernel": "mode_nn_f64 (y-axis mode product)",
                         "achieved": achieved, "peak": PEAK_FP64_TFLOPS, "unit": "TFLOP/s",
                         "frac": achieved / PEAK_FP64_TFLOPS, "traffic": _traffic("f64"),
                         "traffic_detail": PROFILED_TRAFFIC["f64"],
                         "launch_ms": launch_ms, "flops_per_launch": flops_launch},
    }
    out["roofline"] = kernel_roof if kernel_roof is not None else out["roofline_f64"]
    out["roofline_fd_application"] = lowp_roof

    if args.batch > 0:
        out["batched"] = bench_batch(args, P, torch, dev, log)
    if args.ch_steps > 0:
        out["cahn_hilliard"] = bench_ch(args, P, torch, dev, log)
    if args.schrodinger_ne > 0:
        out["schrodinger_pcg"] = bench_schrodinger(args, P, torch, dev, log)

    if not args.no_cpu_baseline:
        import oracle as O
        host = host_info()
        del f
        torch.cuda.empty_cache()
        log("oracle: plan (untimed) ...")
        prob = O.Problem(k, ne, box, alpha, "dirichlet")
        log("oracle: full FP64 solve on the host ...")
        t0 = time.perf_counter()
        u_ref = O.fd_solve(prob, f_host)
        cpu_s = time.perf_counter() - t0
        uref_d = torch.from_numpy(u_ref).to(dev)
        ref_scale = float(uref_d.abs().max())
        for name, out_d in outputs.items():
            e_or = float((out_d - uref_d).abs().max()) / ref_scale
            variants[name]["rel_err_vs_oracle"] = e_or
            log(f"{name}: rel max err vs oracle {e_or:.3e}")
        err = variants["f64"]["rel_err_vs_oracle"]
        del uref_d, outputs, u
        torch.cuda.empty_cache()
        log(f"oracle solve {cpu_s:.1f}s; GPU FP64 rel max err vs oracle {err:.3e}")
        out["cpu_baseline"] = {"value": N / cpu_s, "unit": "unknowns/s", "cores": host["blas_threads"],
                               "kind": "oracle",
                               "sample": f"one full oracle FP64 solve of the same n={nx} workload "
                                         f"(numpy/OpenBLAS matmuls), {cpu_s:.1f} s",
                               "nproc": host["nproc"], "affinity_cpus": host["affinity_cpus"],
                               "cpu_model": host["cpu_model"], "threads_used": host["blas_threads"]}
        out["rel_max_err_vs_oracle"] = err
    print(json.dumps(out), flush=True)
    return 0


if __name__ == "__main__":
    sys.exit(main())
