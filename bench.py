#!/usr/bin/env python
"""Benchmark: P2/P3 Poisson time-to-1e-8 residual with the auxiliary-space
preconditioned CG on one MI355X.

A step is one complete solve (CG from u = 0 to ||r|| <= 1e-8 ||f||, every
preconditioner application included) of the default workload: P2 elements
on the unit cube cut into 48^3 cubes x 6 tets, interior vertices jittered by
+-0.2h (seed 0), kappa = 1, f from u = sin(pi x) sin(pi y) sin(pi z)
(857,375 unknowns).  The headline value is the FP32-preconditioner form
(FP64 CG); the all-FP64 form is measured beside it at the same tolerance.

Other modes: `--krylov fgmres` times the paper's own protocol (flexible
GMRES(30) from a random initial guess on a zero right-hand side, to 1e-6);
`--workload p2_n64_32rhs` the 32-source lock-step solve; `--workload
p2_n40_adjoint` one forward and backward pass of a least-squares loss through
the adjoint solve.

Prints one JSON line.  Inputs are resident in HBM before the timed region.
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "P2/P3 Poisson time-to-1e-8 residual, DOF/s, precond HBM GB/s; mixed vs FP64"
HBM_PEAK_GBS = 8000.0


_T0 = time.time()


def progress(msg):
    """One line per finished stage on stderr (the JSON line stays alone on stdout)."""
    print(f"[bench {time.time() - _T0:7.1f} s] {msg}", file=sys.stderr, flush=True)

WORKLOADS = {
    "p2_n48_jitter": dict(k=2, n=48, jitter=0.2, seed=0, kappa=None),
    "p2_n8": dict(k=2, n=8, jitter=0.0, seed=0, kappa=None),
    "p3_n32_grf": dict(k=3, n=32, jitter=0.0, seed=0, kappa=1),
    # P4 (35 nodes per tet) at the same 857,375 unknowns, kappa = 1
    "p4_n24": dict(k=4, n=24, jitter=0.0, seed=0, kappa=None),
    # the same with kappa = exp(GRF seed 1): P^1 against the intermediate P^2 auxiliary space
    "p4_n24_grf": dict(k=4, n=24, jitter=0.0, seed=0, kappa=1),
    # 32 right-hand sides solved in lock-step (sources fourier_f(0..31))
    "p2_n64_32rhs": dict(k=2, n=64, jitter=0.0, seed=0, kappa=None, nrhs=32),
    # gradient of L = |u - u_t|^2 / 2 with respect to f and log kappa: forward
    # solve, adjoint solve and the per-tet gradient (kappa and the target
    # coefficient from GRF seeds 1 and 2)
    "p2_n40_adjoint": dict(k=2, n=40, jitter=0.0, seed=0, kappa=1, kappa_target=2, adjoint=True),
}


TRAFFIC_TABLE = os.path.join(ROOT, "profiles", "hbm_traffic_sell_sweep.md")
KERNEL_SOURCE = os.path.join(ROOT, "paper_1204_2586_amd", "csrc", "hip", "kernels.hip")


def measured_traffic(workload, operator, category, precision):
    """HBM bytes per launch of a kernel category as measured by the
    FETCH_SIZE and WRITE_SIZE counters (scaled by a plain copy of known
    size), from the committed summary table; None when the table has no
    row for this case or the kernel source changed since the counters were
    taken (its sha1 differs)."""
    import hashlib
    import re
    if not os.path.exists(TRAFFIC_TABLE):
        return None
    with open(KERNEL_SOURCE, "rb") as fh:
        sha = hashlib.sha1(fh.read()).hexdigest()
    for line in open(TRAFFIC_TABLE):
        cells = [c.strip() for c in line.strip().strip("|").split("|")]
        if len(cells) >= 6 and cells[:4] == [workload, operator, category, precision]:
            if cells[4] != sha or not re.fullmatch(r"\d+", cells[5]):
                return None
            return int(cells[5])
    return None


def cycle_lanes(info):
    """Storage the setup chose for the V-cycle's operators: "ell<L>" row-split
    sliced ELL with L lanes per row, "csr<L>" CSR with L lanes per row,
    "fixed" (I_P) fixed-width column-major slots."""
    def name(v):
        return f"ell{v}" if v > 0 else (f"csr{-v}" if v < 0 else "-")
    levels = max(int(info.levels) - 1, 0)
    return {"restrict": name(info.lanes_restrict),
            "prolong": name(info.lanes_prolong) if info.lanes_prolong else "fixed",
            "down": [name(info.lanes_down[l]) for l in range(levels)],
            "up": [name(info.lanes_up[l]) for l in range(levels)]}


def index_bytes_per_entry(info):
    """Column-stream bytes per entry of the device A_h layout (16-bit offsets
    in some slices, 32-bit columns in the others), and the per-slice
    metadata bytes (one 16-byte word: offsets, groups, width)."""
    return info.sell_index_bytes / max(info.stored_A, 1), 16 * info.sell_slices


def algorithmic_bytes(cat, n, nnz, s, fmt):
    """Bytes a kernel must move at least once per launch (matrix values and
    column stream over the nnz entries, each vector array once).  s = bytes
    of the floating-point type, fmt = index_bytes_per_entry(info)."""
    idx, meta = fmt
    mat = (s + idx) * nnz + meta
    if cat == "pk_sweep":      # z_in (gather), rhs, dinv, z_out
        return mat + 4 * s * n
    if cat == "pk_last":       # z_in, rhs (FP64), dinv, z_out (FP64)
        return mat + 2 * s * n + 16 * n
    if cat == "pk_first":      # first sweep from zero, z = D^-1 r: r (FP64), dinv, z, (FP32 copy of r)
        return 8 * n + 2 * s * n + (s * n if s == 4 else 0)
    if cat == "pk_resid":      # rhs, z (gather), res
        return mat + 3 * s * n
    if cat == "cg_spmv":       # FP64 operator, x (gather), y
        return (8 + idx) * nnz + meta + 16 * n
    return None


def matfree_bytes(cat, n, nt, nloc, s):
    """Bytes that one matrix-free product pass cannot do without: a 4 B word
    per tet node (nodes padded to a multiple of four), six weights per tet and
    each dof value once, plus the vectors of the fused update (as in
    algorithmic_bytes).  The patches' dof lists and the partial sums of shared
    dofs depend on the mesh and are not counted."""
    op = nt * 16 * -(-nloc // 4) + nt * 6 * s + n * s
    if cat == "pk_sweep":
        return op + 3 * s * n
    if cat == "pk_last":
        return op + s * n + 16 * n
    if cat == "pk_resid":
        return op + 2 * s * n
    if cat == "cg_spmv":       # FP64: p gathered (in op), q written
        return matfree_bytes("pk_resid", n, nt, nloc, 8) - 8 * n
    return None


def restrict_bytes(info, s):
    """The fused restricted residual r_H = [I_R, -I_R A_h] [r; z]: CSR
    operator, both gathered vectors, the P^1 result."""
    n, nH = info.n_h, info.n_H
    return (s + 4) * info.nnz_restrict + 4 * (nH + 1) + 2 * s * n + s * nH


def apply_bytes(info, s, nu, first=True):
    """Algorithmic bytes of one preconditioner application z = B r with the
    assembled operator, summed over its kernels (each matrix, index and
    vector byte counted once per kernel that needs it).  s = bytes of the
    preconditioner's floating-point type."""
    n, N, nH, NP = info.n_h, info.nnz_A, info.n_H, info.nnz_IP
    fmt = index_bytes_per_entry(info)
    fused = info.nnz_restrict > 0
    # inside CG the first sweep from zero is fused into the CG update (first=False)
    total = algorithmic_bytes("pk_first", n, N, s, fmt) if first else 0
    total += 2 * (nu - 1) * algorithmic_bytes("pk_sweep", n, N, s, fmt)
    total += algorithmic_bytes("pk_last", n, N, s, fmt)
    if fused:
        total += restrict_bytes(info, s)                             # r_H = [I_R, -I_R A_h][r; z]
    else:
        total += algorithmic_bytes("pk_resid", n, N, s, fmt)
        total += (s + 4) * NP + 4 * (nH + 1) + s * n + s * nH      # r_H = I_R res
    total += (s + 4) * NP + 4 * (n + 1) + s * nH + 2 * s * n      # z += I_P e_H
    L = info.levels
    for l in range(L):
        nl, Nl = info.level_rows[l], info.level_nnz[l]
        if l + 1 == L:                                               # dense coarse inverse
            total += s * nl * nl + 2 * s * nl
            continue
        nc, Pl = info.level_rows[l + 1], info.level_nnz_P[l]
        if fused:
            total += (s + 4) * info.level_nnz_down[l] + 4 * (nc + 1) + s * nl + s * nc   # b' = down b
            total += (s + 4) * info.level_nnz_up[l] + 4 * (nl + 1) + 2 * s * nl + s * nc  # y = up [b; e]
            continue
        mat = (s + 4) * Nl + 4 * (nl + 1)
        total += mat + 4 * s * nl                                    # x = D^-1 b, r = b - A x
        total += (s + 4) * Pl + 4 * (nc + 1) + s * nl + s * nc       # b_{l+1} = P^T r
        total += (s + 4) * Pl + 4 * (nl + 1) + s * nc + 2 * s * nl   # x += P e
        total += mat + 4 * s * nl                                    # post-sweep
    return total


def kernel_table(prof, args, s, wl, nt):
    """Per-category launches, average duration and algorithmic GB/s of a
    profiled mixed-precision solve."""
    n, nnz = s.n, int(s.info.nnz_A)
    kernels = {}
    nloc = (wl["k"] + 1) * (wl["k"] + 2) * (wl["k"] + 3) // 6
    for cat, (cnt, tot) in prof.items():
        if args.operator == "matfree" and cat in ("pk_sweep", "pk_last", "cg_spmv"):
            ab = matfree_bytes(cat, n, nt, nloc, 8 if cat == "cg_spmv" else 4)
        else:
            ab = algorithmic_bytes(cat, n, nnz, 4, index_bytes_per_entry(s.info))
        if cat == "pk_resid" and s.info.nnz_restrict > 0:
            ab = restrict_bytes(s.info, 4)
        if cnt and ab:
            avg_ms = tot / cnt
            kernels[cat] = dict(launches=cnt, total_ms=tot, avg_us=avg_ms * 1e3, bytes=ab,
                                gbs=ab / (avg_ms * 1e-3) / 1e9)
    return kernels


def host_cpu():
    """Model name of the host CPU and the number of logical CPUs this process
    may run on."""
    model = "unknown"
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                model = line.split(":", 1)[1].strip()
                break
    except OSError:
        pass
    return model, len(os.sched_getaffinity(0))


def timed_solves(s, f, u, args, mode):
    """K unprofiled solves (each CG iteration replayed as a HIP graph; the
    throughput figures come from these), then the same K solves with HIP
    events around every launch for the per-kernel durations."""
    import torch
    s.set_precision(mode)
    for _ in range(args.warmup):
        s.solve(f, tol=args.tol, out=u)
    torch.cuda.synchronize()
    t = time.perf_counter()
    its = []
    for _ in range(args.steps):
        _, info = s.solve(f, tol=args.tol, out=u)
        its.append(info.iterations)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t) * 1e3 / args.steps
    sol = u.clone()
    true_res = float(torch.linalg.norm(f - s.matvec(sol)) / torch.linalg.norm(f))
    s.profile(True)
    torch.cuda.synchronize()
    t = time.perf_counter()
    for _ in range(args.steps):
        s.solve(f, tol=args.tol, out=u)
    torch.cuda.synchronize()
    ms_prof = (time.perf_counter() - t) * 1e3 / args.steps
    prof = s.profile_read()
    # whole preconditioner applications only: no event records between an
    # application's own launches
    s.profile("apply")
    for _ in range(args.steps):
        s.solve(f, tol=args.tol, out=u)
    torch.cuda.synchronize()
    prof_apply = s.profile_read()["apply"]
    progress(f"{mode} solves: {ms:.3f} ms each, {its[-1]} iterations")
    s.profile(False)
    return dict(ms=ms, ms_profiled=ms_prof, iterations=its, true_rel_residual=true_res, prof=prof, u=sol,
                prof_apply=prof_apply)


def measure_single(s, f, args, wl, nt, operator):
    """Mixed and FP64 timed solves of one system with one operator, the
    dominant kernel's roofline and the whole preconditioner's bandwidth."""
    import torch
    s.set_operator(operator)
    u = torch.zeros_like(f)
    mixed = timed_solves(s, f, u, args, "mixed")
    fp64 = timed_solves(s, f, u, args, "fp64")
    ka = argparse.Namespace(operator=operator)
    kernels = kernel_table(mixed["prof"], ka, s, wl, nt)
    dom = max(kernels, key=lambda c: kernels[c]["total_ms"])
    kd = kernels[dom]
    precond = {}
    for name, res, sz in (("mixed", mixed, 4), ("fp64", fp64, 8)):
        cnt, tot = res["prof_apply"]
        us = tot / max(cnt, 1) * 1e3
        c1, t1 = res["prof"]["apply"]
        entry = {"us": us, "us_with_launch_events": t1 / max(c1, 1) * 1e3}
        if operator == "assembled" and int(s.info.aux_space) == 1:
            ab = apply_bytes(s.info, sz, args.nu, first=res["prof"].get("pk_first", (0, 0))[0] > 0)
            entry.update(bytes=ab, gbs=ab / (us * 1e-6) / 1e9, frac=ab / (us * 1e-6) / 1e9 / HBM_PEAK_GBS)
        precond[name] = entry
    return dict(mixed=mixed, fp64=fp64, kernels=kernels, dom=dom, kd=kd, precond=precond)


def roofline_entry(workload, operator, m):
    kd = m["kd"]
    return {"bound": "hbm", "kernel": m["dom"], "achieved": kd["gbs"], "peak": HBM_PEAK_GBS, "unit": "GB/s",
            "frac": kd["gbs"] / HBM_PEAK_GBS, "traffic": measured_traffic(workload, operator, m["dom"], "mixed"),
            "bytes_per_launch": kd["bytes"], "avg_us": kd["avg_us"]}


def rel_err(u_gpu, x_ref):
    import numpy as np
    x = np.asarray(x_ref)
    return float(np.linalg.norm(u_gpu.cpu().numpy() - x) / np.linalg.norm(x))


def oracle_reference(xyz, tets, wl, kappa, args, reps):
    """The CPU oracle (single-threaded FP64 C) on the same system, with its
    own load vector of the manufactured source: `reps` timed CG solves to the
    benchmark's tolerance from u = 0 on one core (median reported; its setup
    is not timed), and one untimed solve to 1e-13, the discrete solution
    within rounding.  Returns the timing entry and both oracle solutions."""
    import statistics

    import oracle
    import workloads as W
    t0 = time.time()
    P = oracle.Problem(xyz, tets, wl["k"], kappa).setup_amg(nu=args.nu)
    b = P.load(W.manufactured_f)
    setup = time.time() - t0
    progress(f"oracle setup ({P.n} unknowns): {setup:.1f} s")
    model, ncpu = host_cpu()
    keep = os.sched_getaffinity(0)
    one = {min(keep)}
    times = []
    os.sched_setaffinity(0, one)             # the oracle is single-threaded: one core
    try:
        for _ in range(reps):
            t0 = time.perf_counter()
            x, it, rr, st = P.pcg(b, tol=args.tol)
            times.append(time.perf_counter() - t0)
            progress(f"oracle timed solve {len(times)}/{reps}: {times[-1]:.1f} s")
        x_tight, it_tight, _, _ = P.pcg(b, tol=1e-13)
        progress(f"oracle 1e-13 reference solve: {it_tight} iterations")
    finally:
        os.sched_setaffinity(0, keep)
    dt = statistics.median(times)
    entry = {"value": P.n / dt, "unit": "DOF/s", "cores": 1, "kind": "oracle",
             "cpu_model": model, "host_cpus": ncpu, "repeats": reps,
             "seconds": [round(v, 2) for v in times], "iterations": it,
             "sample": f"median of {reps} FP64 CG solves of the full {args.workload_name} system (n_h={P.n}) "
                       f"to {args.tol:g}, {it} iterations, {dt:.1f} s each, pinned to one core; oracle setup "
                       f"{setup:.1f} s and a 1e-13 reference solve ({it_tight} iterations) not timed"}
    return entry, x, x_tight


def oracle_errors(res, x, x_tight):
    """Each GPU result against the FP64 oracle: its solution at the same
    tolerance and its 1e-13 solution (the discrete solution)."""
    return {"mixed_vs_oracle_rel_err": rel_err(res["mixed"]["u"], x),
            "fp64_vs_oracle_rel_err": rel_err(res["fp64"]["u"], x),
            "mixed_vs_discrete_solution_rel_err": rel_err(res["mixed"]["u"], x_tight),
            "fp64_vs_discrete_solution_rel_err": rel_err(res["fp64"]["u"], x_tight)}


def single_summary(name, operator, n, m, errs=None):
    mixed, fp64 = m["mixed"], m["fp64"]
    d = {"operator": operator, "n_h": n,
         "mixed": {"ms": round(mixed["ms"], 3), "dof_per_s": n / (mixed["ms"] * 1e-3),
                   "iterations": mixed["iterations"][-1], "true_rel_residual": mixed["true_rel_residual"]},
         "fp64": {"ms": round(fp64["ms"], 3), "dof_per_s": n / (fp64["ms"] * 1e-3),
                  "iterations": fp64["iterations"][-1], "true_rel_residual": fp64["true_rel_residual"]},
         "roofline": roofline_entry(name, operator, m),
         "precond_apply": m["precond"],
         "kernels_mixed": {c: {k: (round(v, 3) if isinstance(v, float) else v) for k, v in dd.items()}
                           for c, dd in m["kernels"].items()}}
    if errs:
        d.update(errs)
    return d


def run_extra_p3(args):
    """P3 on 32^3 cubes with kappa = exp(GRF seed 1): assembled and
    matrix-free, each mixed and FP64, against one oracle solve."""
    import numpy as np
    import torch

    import paper_1204_2586_amd as aux
    import workloads as W
    name = "p3_n32_grf"
    wl = WORKLOADS[name]
    xyz, tets = W.kuhn_mesh(wl["n"], jitter=wl["jitter"], seed=wl["seed"])
    kappa = np.exp(W.grf_log_kappa(xyz, tets, seed=wl["kappa"]))
    dev = torch.device("cuda:0")
    t0 = time.time()
    s = aux.Solver(xyz, tets, wl["k"], kappa, nu=args.nu, precision="mixed", device=dev)
    setup_s = time.time() - t0
    progress(f"GPU setup: {setup_s:.2f} s")
    b = s.load(W.manufactured_f)
    f = torch.tensor(b, dtype=torch.float64, device=dev)
    out = {"order": wl["k"], "cubes_per_side": wl["n"], "kappa": "exp(GRF seed 1)", "n_h": s.n,
           "nnz_A": int(s.info.nnz_A), "setup_s": round(setup_s, 2)}
    ms = {op: measure_single(s, f, args, wl, len(tets), op) for op in ("assembled", "matfree")}
    s.set_operator("assembled")
    ref = None
    if not args.no_cpu_baseline:
        a = argparse.Namespace(**vars(args))
        a.workload_name = name
        ref = oracle_reference(xyz, tets, wl, kappa, a, reps=1)
        out["cpu_baseline"] = ref[0]
    for op, m in ms.items():
        out[op] = single_summary(name, op, s.n, m, oracle_errors(m, ref[1], ref[2]) if ref else None)
    return out


def run_extra_nested(args):
    """P4 on 24^3 cubes with kappa = exp(GRF seed 1): the P^1 auxiliary
    space against the intermediate P^2 space (Remark 6.2), each with the
    assembled and the matrix-free P^4 operator, mixed and FP64;
    one step is one solve to 1e-8.  Parity with the oracle's nested
    preconditioner is tested at small sizes; here the two spaces' solutions
    are compared with each other."""
    import numpy as np
    import torch

    import paper_1204_2586_amd as aux
    import workloads as W
    name = "p4_n24_grf"
    wl = WORKLOADS[name]
    xyz, tets = W.kuhn_mesh(wl["n"], jitter=wl["jitter"], seed=wl["seed"])
    kappa = np.exp(W.grf_log_kappa(xyz, tets, seed=wl["kappa"]))
    dev = torch.device("cuda:0")
    out = {"order": 4, "cubes_per_side": wl["n"], "kappa": "exp(GRF seed 1)"}
    sol = {}
    for space in (1, 2):
        t0 = time.time()
        s = aux.Solver(xyz, tets, 4, kappa, nu=args.nu, precision="mixed", device=dev, aux_space=space)
        setup_s = time.time() - t0
        progress(f"GPU setup (aux_space {space}): {setup_s:.2f} s")
        f = torch.tensor(s.load(W.manufactured_f), dtype=torch.float64, device=dev)
        u = torch.zeros_like(f)
        e = {"setup_s": round(setup_s, 2), "n_h": s.n}
        for op in ("assembled", "matfree"):
            s.set_operator(op)
            e[op] = {}
            for mode in ("mixed", "fp64"):
                r = timed_solves(s, f, u, args, mode)
                cnt, tot = r["prof_apply"]
                e[op][mode] = {"ms": round(r["ms"], 3), "dof_per_s": s.n / (r["ms"] * 1e-3),
                               "iterations": r["iterations"][-1], "true_rel_residual": r["true_rel_residual"],
                               "precond_apply_us": round(tot / max(cnt, 1) * 1e3, 2)}
                if mode == "mixed" and op == "assembled":
                    sol[space] = r["u"]
        out["p1_space" if space == 1 else "p2_space"] = e
        del s
        torch.cuda.empty_cache()
    out["p2_vs_p1_solution_rel_diff"] = float(torch.linalg.norm(sol[2] - sol[1]) / torch.linalg.norm(sol[1]))
    out["speedup_p2_space_mixed"] = {op: out["p1_space"][op]["mixed"]["ms"] / out["p2_space"][op]["mixed"]["ms"]
                                     for op in ("assembled", "matfree")}
    return out


def run_kappa_update(args):
    """P2 on 48^3 jittered cubes: new per-tet coefficients (exp of GRF seeds
    2..4) through aux_set_kappa -- device assembly, then the AMG hierarchy,
    composite level operators and dense cycle built on the device (the
    default) or on the host -- each followed by a mixed solve of the new
    system.  The first update (mesh-only maps, untimed) uses GRF seed 1."""
    import numpy as np
    import torch

    import paper_1204_2586_amd as aux
    import workloads as W
    xyz, tets = W.kuhn_mesh(48, jitter=0.2, seed=0)
    kappas = [np.exp(W.grf_log_kappa(xyz, tets, seed=sd)) for sd in (1, 2, 3, 4)]
    dev = torch.device("cuda:0")
    out = {"workload": "p2_n48_jitter, kappa = exp(GRF seeds 2-4)", "n_h": None}
    for mode in ("device", "host"):
        s = aux.Solver(xyz, tets, 2, kappas[0], nu=args.nu, precision="mixed", device=dev, amg_setup=mode)
        out["n_h"] = s.n
        f = torch.tensor(s.load(W.manufactured_f), dtype=torch.float64, device=dev)
        s.set_kappa(kappas[0])
        ms, amg, its = [], [], []
        for kap in kappas[1:]:
            torch.cuda.synchronize()
            t = time.perf_counter()
            s.set_kappa(kap)
            torch.cuda.synchronize()
            ms.append((time.perf_counter() - t) * 1e3)
            amg.append(s.info.amg_setup_seconds * 1e3)
            _, info = s.solve(f, tol=args.tol)
            its.append(info.iterations)
        out[f"amg_on_{mode}"] = {"ms_per_update": [round(v, 1) for v in ms],
                                 "amg_build_ms": [round(v, 1) for v in amg], "iterations_after": its}
        progress(f"coefficient updates (AMG on the {mode}): {min(ms):.1f} ms")
        del s
        torch.cuda.empty_cache()
    out["speedup_device_amg"] = min(out["amg_on_host"]["ms_per_update"]) / min(out["amg_on_device"]["ms_per_update"])
    return out


def run_stokes(args, k=2, n=48, n_oracle=16):
    """Stokes, Hood-Taylor P^k-P^{k-1} (Sec. 5) on a jittered mesh of n^3
    cubes: FGMRES(30) with the block triangular preconditioner Q_t to 1e-8
    from zero, body force of a smooth manufactured solution; one step is one
    solve.  The oracle solves the n_oracle^3 system of the same family (the
    CPU sample, and the GPU's error against it at that size)."""
    import numpy as np
    import torch

    import oracle
    import paper_1204_2586_amd as aux
    import workloads as W
    dev = torch.device("cuda:0")

    def system(m):
        xyz, tets = W.kuhn_mesh(m, jitter=0.2, seed=0)
        t0 = time.time()
        s = aux.Solver(xyz, tets, k, nu=args.nu, precision="mixed", device=dev)
        npr = s.stokes_setup()
        setup_s = time.time() - t0
        progress(f"GPU setup: {setup_s:.2f} s")
        b = np.concatenate([s.load(W.stokes_f(c)) for c in range(3)] + [np.zeros(npr)])
        return xyz, tets, s, b, setup_s

    xyz, tets, s, b, setup_s = system(n)
    bt = torch.tensor(b, dtype=torch.float64, device=dev)
    N = 3 * s.n + s.n_p
    reps = max(1, min(args.steps, 5))
    res = {}
    for mode in ("mixed", "fp64"):
        s.set_precision(mode)
        s.stokes_fgmres(bt, tol=1e-8, restart=30)
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(reps):
            x, info, _ = s.stokes_fgmres(bt, tol=1e-8, restart=30)
        torch.cuda.synchronize()
        ms = (time.perf_counter() - t) * 1e3 / reps
        true_res = float(torch.linalg.norm(bt - s.stokes_operator(x)) / torch.linalg.norm(bt))
        res[mode] = dict(ms=ms, iterations=info.iterations, true_rel_residual=true_res)
        progress(f"Stokes P{k}-P{k - 1} {mode}: {ms:.1f} ms per solve, {info.iterations} steps")
    s.set_precision("mixed")
    r = torch.zeros(N, dtype=torch.float64, device=dev)
    r[3 * s.n:] = torch.tensor(np.random.default_rng(3).standard_normal(s.n_p), dtype=torch.float64, device=dev)
    _, mass_steps = s.stokes_qt(r)
    pair = f"p{k}p{k - 1}"
    out = {"metric": f"Stokes (Hood-Taylor P{k}-P{k - 1}) FGMRES(30) + Q_t solve throughput to 1e-8",
           "unit": "unknowns/s", "value": N / (res["mixed"]["ms"] * 1e-3),
           "ms_per_solve": round(res["mixed"]["ms"], 3),
           "dtype": "f64 FGMRES / f32 velocity preconditioner / f64 pressure mass CG",
           "config": {"workload": f"stokes_{pair}_n{n}_jitter", "cubes_per_side": n, "jitter": 0.2,
                      "n_velocity": 3 * s.n, "n_pressure": s.n_p, "unknowns": N,
                      "iterations": res["mixed"]["iterations"],
                      "true_rel_residual": res["mixed"]["true_rel_residual"],
                      "us_per_fgmres_step": round(res["mixed"]["ms"] * 1e3 / max(res["mixed"]["iterations"], 1), 1),
                      "mass_cg_steps_per_qt": mass_steps, "setup_s": round(setup_s, 2)},
           "fp64": {"value": N / (res["fp64"]["ms"] * 1e-3), "ms_per_solve": round(res["fp64"]["ms"], 3),
                    "iterations": res["fp64"]["iterations"], "true_rel_residual": res["fp64"]["true_rel_residual"]}}
    del s, bt
    torch.cuda.empty_cache()
    if not args.no_cpu_baseline:
        xyz, tets, s, b, _ = system(n_oracle)
        x, info, _ = s.stokes_fgmres(torch.tensor(b, dtype=torch.float64, device=dev), tol=1e-8, restart=30)
        x = x.cpu().numpy()
        P = oracle.Problem(xyz, tets, k).setup_amg(nu=args.nu).stokes_setup()
        t0 = time.perf_counter()
        xo, it, rr, st, _ = P.stokes_fgmres(b, tol=1e-8, restart=30, fp32=True)
        dt = time.perf_counter() - t0
        progress(f"oracle Stokes solve ({len(b)} unknowns): {dt:.1f} s, {it} steps")
        m = s.n
        pm = lambda v: v[3 * m:] - v[3 * m:].mean()
        out["cpu_baseline"] = {"value": len(b) / dt, "unit": "unknowns/s", "cores": 1, "kind": "oracle",
                               "sample": f"one FGMRES(30) + Q_t solve (FP32 velocity preconditioner) of the "
                                         f"jittered P{k}-P{k - 1} {n_oracle}^3 system ({len(b)} unknowns) to "
                                         f"1e-8, {it} steps, {dt:.1f} s"}
        out[f"oracle_error_{n_oracle}"] = {"gpu_steps": info.iterations, "oracle_steps": it,
                                           "velocity_rel_diff": float(np.linalg.norm(x[:3 * m] - xo[:3 * m])
                                                                      / np.linalg.norm(xo[:3 * m])),
                                           "pressure_rel_diff_mod_const": float(np.linalg.norm(pm(x) - pm(xo))
                                                                                / np.linalg.norm(pm(xo)))}
        del s
        torch.cuda.empty_cache()
    return out


def run_stokes_pairs(args):
    """P2-P1 on 48^3 cubes and P3-P2 on 32^3 cubes (2.69M and 2.85M unknowns)."""
    out = run_stokes(args, k=2, n=48, n_oracle=16)
    out["p3p2_n32_jitter"] = run_stokes(args, k=3, n=32, n_oracle=8)
    return out


def run(args):
    import numpy as np
    import torch

    import paper_1204_2586_amd as aux
    import workloads as W

    wl = WORKLOADS[args.workload]
    xyz, tets = W.kuhn_mesh(wl["n"], jitter=wl["jitter"], seed=wl["seed"])
    kappa = None
    if wl["kappa"] is not None:
        kappa = np.exp(W.grf_log_kappa(xyz, tets, seed=wl["kappa"]))
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    t0 = time.time()
    s = aux.Solver(xyz, tets, wl["k"], kappa, nu=args.nu, precision="mixed", device=dev, operator=args.operator,
                   aux_space=args.aux_space)
    setup_s = time.time() - t0
    progress(f"GPU setup: {setup_s:.2f} s")
    b = s.load(W.manufactured_f)
    f = torch.tensor(b, dtype=torch.float64, device=dev)
    n, nnz = s.n, int(s.info.nnz_A)

    m = measure_single(s, f, args, wl, len(tets), args.operator)
    mixed, fp64, kd = m["mixed"], m["fp64"], m["kd"]
    diff = float(torch.linalg.norm(mixed["u"] - fp64["u"]) / torch.linalg.norm(fp64["u"]))

    out = {
        "metric": METRIC,
        "value": n / (mixed["ms"] * 1e-3),
        "unit": "DOF/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": mixed["ms"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64 CG / f32 preconditioner",
        "data": "synthetic",
        "config": {"workload": args.workload, "operator": args.operator, "nu": args.nu, "order": wl["k"],
                   "aux_space": args.aux_space,
                   "cubes_per_side": wl["n"],
                   "jitter": wl["jitter"], "n_h": n, "nnz_A": nnz, "tol": args.tol,
                   "iterations": mixed["iterations"][-1], "true_rel_residual": mixed["true_rel_residual"],
                   "amg_levels": int(s.info.levels), "op_complexity": round(float(s.info.op_complexity), 4),
                   "setup_s": round(setup_s, 2), "sell_window": int(s.info.sell_window),
                   "sell_16bit_slices": f"{int(s.info.sell_narrow_slices)}/{int(s.info.sell_slices)}",
                   "sell_tune_ms": [round(v, 4) for v in s.info.sell_tune_ms],
                   "cycle_lanes": cycle_lanes(s.info), "sell_split": int(s.info.sell_split),
                   "ms_per_step_profiled": round(mixed["ms_profiled"], 3)},
        "fp64": {"value": n / (fp64["ms"] * 1e-3), "ms_per_step": fp64["ms"],
                 "iterations": fp64["iterations"][-1], "true_rel_residual": fp64["true_rel_residual"],
                 "mixed_vs_fp64_rel_diff": diff,
                 "speedup_mixed_over_fp64": fp64["ms"] / mixed["ms"]},
        "roofline": roofline_entry(args.workload, args.operator, m),
        "kernels_mixed": {c: {k: (round(v, 3) if isinstance(v, float) else v) for k, v in d.items()}
                          for c, d in m["kernels"].items()},
        "precond_apply": m["precond"],
    }
    # achievable HBM bandwidth on this device: plain 1 GiB device copies;
    # the dominant kernel's rate against it beside the fraction of the peak
    out["hbm_copy_gbs"] = round(calibrate_copy(reps=5)["copy_gbs"], 1)
    out["roofline"]["frac_of_copy"] = out["roofline"]["achieved"] / out["hbm_copy_gbs"]
    if not args.no_cpu_baseline:
        a = argparse.Namespace(**vars(args))
        a.workload_name = args.workload
        entry, x, x_tight = oracle_reference(xyz, tets, wl, kappa, a, reps=3)
        out["cpu_baseline"] = entry
        out["oracle_error"] = oracle_errors(m, x, x_tight)
    if args.extras:
        # the metric's P3 case and the lock-step batch (the clean HBM case),
        # each with its own roofline and oracle comparison
        del s, m, mixed, fp64
        torch.cuda.empty_cache()
        out["workloads"] = {"p3_n32_grf": run_extra_p3(args)}
        torch.cuda.empty_cache()
        a = argparse.Namespace(**vars(args))
        a.workload = "p2_n64_32rhs"
        out["workloads"]["p2_n64_32rhs"] = summarize_batched(run_batched(a))
        torch.cuda.empty_cache()
        out["workloads"]["stokes_p2p1_n48_jitter"] = run_stokes(args)
        torch.cuda.empty_cache()
        out["workloads"]["stokes_p3p2_n32_jitter"] = run_stokes(args, k=3, n=32, n_oracle=8)
        torch.cuda.empty_cache()
        out["workloads"]["p4_n24_grf_aux_spaces"] = run_extra_nested(args)
        torch.cuda.empty_cache()
        out["workloads"]["p2_n48_coefficient_update"] = run_kappa_update(args)
    return out


def summarize_batched(r):
    """The batched record as an entry of the default line."""
    keys = ("value", "ms_per_step", "config", "fp64", "block_cg", "single_rhs_sequential", "roofline", "kernels_mixed",
            "precond_apply_us", "cpu_baseline", "oracle_error")
    return {k: r[k] for k in keys if k in r}


def batched_bytes(cat, n, nnz, s, nr, fmt):
    """Algorithmic bytes of one launch of a block kernel over nr columns
    (block vectors [n][nr]; matrix, index and vector bytes counted once)."""
    idx, meta = fmt
    mat = (s + idx) * nnz + meta
    if cat == "pk_sweep":      # Z_in (gather), RHS, Z_out; dinv
        return mat + 3 * s * n * nr + s * n
    if cat == "pk_last":       # Z_in, RHS (FP64), Z_out (FP64); dinv
        return mat + s * n * nr + 16 * n * nr + s * n
    if cat == "pk_first":      # R (FP64), dinv, Z, (FP32 copy of R)
        return 8 * n * nr + s * n + s * n * nr + (s * n * nr if s == 4 else 0)
    if cat == "pk_resid":      # RHS, Z (gather), RES
        return mat + 3 * s * n * nr
    if cat == "cg_spmv":       # FP64 operator, P (gather), Q
        return (8 + idx) * nnz + meta + 16 * n * nr
    return None


def run_batched(args):
    import numpy as np
    import torch

    import paper_1204_2586_amd as aux
    import workloads as W

    wl = WORKLOADS[args.workload]
    nrhs = wl["nrhs"]
    xyz, tets = W.kuhn_mesh(wl["n"], jitter=wl["jitter"], seed=wl["seed"])
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    t0 = time.time()
    s = aux.Solver(xyz, tets, wl["k"], None, nu=args.nu, precision="mixed", device=dev,
                   batch_order=getattr(args, "batch_order", 0))
    setup_s = time.time() - t0
    progress(f"GPU setup: {setup_s:.2f} s")
    t0 = time.time()
    B = s.load_many(W.fourier_fields(range(nrhs)), nrhs, threads=args.threads)
    load_s = time.time() - t0
    F = torch.tensor(B, dtype=torch.float64, device=dev)
    n, nnz = s.n, int(s.info.nnz_A)

    def timed(mode):
        s.set_precision(mode)
        for _ in range(args.warmup):
            s.solve_batched(F, tol=args.tol)
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(args.steps):
            U, infos = s.solve_batched(F, tol=args.tol)
        torch.cuda.synchronize()
        ms = (time.perf_counter() - t) * 1e3 / args.steps
        res = torch.stack([torch.linalg.norm(F[:, c] - s.matvec(U[:, c].contiguous())) / torch.linalg.norm(F[:, c])
                           for c in range(nrhs)])
        s.profile(True)
        s.solve_batched(F, tol=args.tol)
        prof = s.profile_read()
        s.profile(False)
        return dict(ms=ms, its=[i.iterations for i in infos], true_res=float(res.max()), prof=prof, U=U)

    mixed = timed("mixed")
    progress(f"batched mixed: {mixed['ms']:.2f} ms per batch")
    fp64 = timed("fp64")
    progress(f"batched fp64: {fp64['ms']:.2f} ms per batch")
    # the same sources one at a time (mixed), for the lock-step gain
    s.set_precision("mixed")
    u = torch.zeros(n, dtype=torch.float64, device=dev)
    cols = [F[:, c].contiguous() for c in range(nrhs)]
    s.solve(cols[0], tol=args.tol, out=u)
    torch.cuda.synchronize()
    t = time.perf_counter()
    single_its = []
    for c in range(nrhs):
        _, info = s.solve(cols[c], tol=args.tol, out=u)
        single_its.append(info.iterations)
    torch.cuda.synchronize()
    single_ms = (time.perf_counter() - t) * 1e3
    progress(f"sequential single-source solves: {single_ms:.1f} ms")
    diff = float(torch.linalg.norm(mixed["U"] - fp64["U"]) / torch.linalg.norm(fp64["U"]))
    # O'Leary's block CG on the same sources (FP32 preconditioner)
    s.set_precision("mixed")
    for _ in range(args.warmup):
        s.solve_block(F, tol=args.tol)
    torch.cuda.synchronize()
    t = time.perf_counter()
    for _ in range(args.steps):
        Ub, binfos = s.solve_block(F, tol=args.tol)
    torch.cuda.synchronize()
    block_ms = (time.perf_counter() - t) * 1e3 / args.steps
    progress(f"block CG: {block_ms:.2f} ms per batch")
    block_res = max(float(torch.linalg.norm(F[:, c] - s.matvec(Ub[:, c].contiguous())) / torch.linalg.norm(F[:, c]))
                    for c in range(nrhs))
    block_diff = float(torch.linalg.norm(Ub - fp64["U"]) / torch.linalg.norm(fp64["U"]))

    nr = 8
    while nr < nrhs:
        nr *= 2
    kernels = {}
    for cat, (cnt, tot) in mixed["prof"].items():
        ab = batched_bytes(cat, n, nnz, 4, nr, index_bytes_per_entry(s.info))
        if cat == "pk_resid" and s.info.nnz_restrict > 0:    # fused restricted residual, block vectors
            ab = (4 + 4) * s.info.nnz_restrict + 8 * s.info.n_H + (2 * n + s.info.n_H) * 4 * nr
        if cnt and ab:
            avg_ms = tot / cnt
            kernels[cat] = dict(launches=cnt, total_ms=round(tot, 3), avg_us=round(avg_ms * 1e3, 2), bytes=ab,
                                gbs=round(ab / (avg_ms * 1e-3) / 1e9, 1))
    dom = max(kernels, key=lambda c: kernels[c]["total_ms"])
    kd = kernels[dom]
    cnt, tot = mixed["prof"]["apply"]
    out = {
        "metric": METRIC,
        "value": nrhs * n / (mixed["ms"] * 1e-3),
        "unit": "DOF/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": mixed["ms"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64 CG / f32 preconditioner",
        "data": "synthetic",
        "config": {"workload": args.workload, "order": wl["k"], "cubes_per_side": wl["n"], "nrhs": nrhs,
                   "n_h": n, "nnz_A": nnz, "tol": args.tol, "iterations_max": max(mixed["its"]),
                   "iterations_min": min(mixed["its"]), "true_rel_residual_max": mixed["true_res"],
                   "setup_s": round(setup_s, 2), "load_s": round(load_s, 1), "sell_window": int(s.info.sell_window),
                   "batch_tile_rows": {"fp32": int(s.info.batch_tile_rows[0]), "fp64": int(s.info.batch_tile_rows[1])},
                   "batch_order": getattr(args, "batch_order", 0),
                   "sell_16bit_slices": f"{int(s.info.sell_narrow_slices)}/{int(s.info.sell_slices)}"},
        "fp64": {"value": nrhs * n / (fp64["ms"] * 1e-3), "ms_per_step": fp64["ms"],
                 "iterations_max": max(fp64["its"]), "true_rel_residual_max": fp64["true_res"],
                 "mixed_vs_fp64_rel_diff": diff, "speedup_mixed_over_fp64": fp64["ms"] / mixed["ms"]},
        "block_cg": {"ms_per_step": block_ms, "value": nrhs * n / (block_ms * 1e-3),
                     "iterations": binfos[0].iterations, "true_rel_residual_max": block_res,
                     "block_vs_lockstep_fp64_rel_diff": block_diff,
                     "speedup_over_lockstep": mixed["ms"] / block_ms},
        "single_rhs_sequential": {"ms_for_all": single_ms, "value": nrhs * n / (single_ms * 1e-3),
                                  "iterations_max": max(single_its),
                                  "speedup_batched_over_sequential": single_ms / mixed["ms"]},
        "roofline": {"bound": "hbm", "kernel": dom, "achieved": kd["gbs"], "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": kd["gbs"] / HBM_PEAK_GBS, "traffic": None,
                     "bytes_per_launch": kd["bytes"], "avg_us": kd["avg_us"]},
        "kernels_mixed": kernels,
        "precond_apply_us": {"mixed": tot / max(cnt, 1) * 1e3},
    }
    if not args.no_cpu_baseline:
        entry, x = cpu_baseline_single(xyz, tets, wl, args)
        out["cpu_baseline"] = entry
        out["oracle_error"] = {"column": 0, "mixed_vs_oracle_rel_err": rel_err(mixed["U"][:, 0], x),
                               "fp64_vs_oracle_rel_err": rel_err(fp64["U"][:, 0], x)}
    return out


def calibrate_copy(nbytes=1 << 30, reps=3):
    """Plain device copies of a known size: what a hardware byte counter
    reads for them scales the counters of the solver's kernels."""
    import torch
    src = torch.ones(nbytes // 8, dtype=torch.float64, device="cuda:0")
    dst = torch.empty_like(src)
    dst.copy_(src)
    torch.cuda.synchronize()
    t = time.perf_counter()
    for _ in range(reps):
        dst.copy_(src)
    torch.cuda.synchronize()
    dt = (time.perf_counter() - t) / reps
    return {"copy_bytes_read": nbytes, "copy_bytes_written": nbytes, "reps": reps,
            "copy_gbs": 2 * nbytes / dt / 1e9}


def cpu_baseline_single(xyz, tets, wl, args):
    """The CPU oracle on one of the batched sources (column 0): one FP64 CG
    solve at full size on one core; the oracle's own setup and load vector
    are not timed.  Returns the timing entry and the oracle's solution."""
    import numpy as np

    import oracle
    import workloads as W
    P = oracle.Problem(xyz, tets, wl["k"], None).setup_amg(nu=args.nu)
    src = W.fourier_fields([0])

    def f(p):                                # evaluated in slices to bound memory
        out = np.empty(p.shape[0])
        for i in range(0, p.shape[0], 1 << 22):
            out[i:i + (1 << 22)] = src(p[i:i + (1 << 22)])[0]
        return out

    b = P.load(f)
    progress(f"oracle setup and load vector ({P.n} unknowns) done")
    model, ncpu = host_cpu()
    keep = os.sched_getaffinity(0)
    os.sched_setaffinity(0, {min(keep)})
    try:
        t0 = time.perf_counter()
        x, it, rr, st = P.pcg(b, tol=args.tol)
        dt = time.perf_counter() - t0
        progress(f"oracle solve: {dt:.1f} s, {it} iterations")
    finally:
        os.sched_setaffinity(0, keep)
    entry = {"value": P.n / dt, "unit": "DOF/s", "cores": 1, "kind": "oracle", "cpu_model": model,
             "host_cpus": ncpu, "repeats": 1, "seconds": [round(dt, 2)], "iterations": it,
             "sample": f"one FP64 CG solve of source 0 of {args.workload} (n_h={P.n}) to {args.tol:g} on one "
                       f"core, {it} iterations, {dt:.1f} s; the 32-source batch would take {32 * dt:.0f} s"}
    return entry, x


def run_fgmres(args):
    """The paper's protocol (Sec. 6.1): flexible GMRES(restart) from a random
    initial guess on a zero right-hand side, stopped at a 1e-6 relative
    residual; one step is one solve."""
    import numpy as np
    import torch

    import paper_1204_2586_amd as aux
    import workloads as W

    wl = WORKLOADS[args.workload]
    xyz, tets = W.kuhn_mesh(wl["n"], jitter=wl["jitter"], seed=wl["seed"])
    kappa = None
    if wl["kappa"] is not None:
        kappa = np.exp(W.grf_log_kappa(xyz, tets, seed=wl["kappa"]))
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    t0 = time.time()
    s = aux.Solver(xyz, tets, wl["k"], kappa, nu=args.nu, precision="mixed", device=dev, operator=args.operator,
                   aux_space=args.aux_space)
    setup_s = time.time() - t0
    progress(f"GPU setup: {setup_s:.2f} s")
    n = s.n
    x0 = torch.tensor(np.random.default_rng(7).uniform(-1.0, 1.0, n), dtype=torch.float64, device=dev)
    zero = torch.zeros_like(x0)
    r0 = float(torch.linalg.norm(s.matvec(x0)))

    def timed(mode):
        s.set_precision(mode)
        for _ in range(args.warmup):
            s.fgmres(zero, tol=args.tol, x0=x0, restart=args.restart)
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(args.steps):
            x, info, hist = s.fgmres(zero, tol=args.tol, x0=x0, restart=args.restart)
        torch.cuda.synchronize()
        ms = (time.perf_counter() - t) * 1e3 / args.steps
        true_res = float(torch.linalg.norm(s.matvec(x))) / r0
        s.profile(True)
        for _ in range(args.steps):
            s.fgmres(zero, tol=args.tol, x0=x0, restart=args.restart)
        torch.cuda.synchronize()
        prof = s.profile_read()
        s.profile(False)
        return dict(ms=ms, iterations=info.iterations, true_rel_residual=true_res, prof=prof)

    mixed = timed("mixed")
    progress(f"FGMRES mixed: {mixed['ms']:.2f} ms per solve")
    fp64 = timed("fp64")
    progress(f"FGMRES fp64: {fp64['ms']:.2f} ms per solve")
    kernels = kernel_table(mixed["prof"], args, s, wl, len(tets))
    dom = max(kernels, key=lambda c: kernels[c]["total_ms"])
    kd = kernels[dom]
    apply_us = mixed["prof"]["apply"][1] / max(mixed["prof"]["apply"][0], 1) * 1e3
    out = {
        "metric": "FGMRES solve throughput, paper protocol (zero right-hand side, random initial guess)",
        "value": n / (mixed["ms"] * 1e-3),
        "unit": "DOF/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": mixed["ms"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64 FGMRES / f32 preconditioner",
        "data": "synthetic",
        "config": {"workload": args.workload, "krylov": f"fgmres({args.restart})", "operator": args.operator,
                   "nu": args.nu,
                   "order": wl["k"], "cubes_per_side": wl["n"], "jitter": wl["jitter"], "n_h": n,
                   "tol": args.tol, "iterations": mixed["iterations"],
                   "true_rel_residual": mixed["true_rel_residual"], "setup_s": round(setup_s, 2),
                   "apply_us_per_step": round(apply_us, 1),
                   "us_per_arnoldi_step": round(mixed["ms"] * 1e3 / max(mixed["iterations"], 1), 1)},
        "fp64": {"value": n / (fp64["ms"] * 1e-3), "ms_per_step": fp64["ms"], "iterations": fp64["iterations"],
                 "true_rel_residual": fp64["true_rel_residual"]},
        "roofline": {"bound": "hbm", "kernel": dom, "achieved": kd["gbs"], "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": kd["gbs"] / HBM_PEAK_GBS,
                     "traffic": measured_traffic(args.workload, args.operator, dom, "mixed"),
                     "bytes_per_launch": kd["bytes"], "avg_us": kd["avg_us"]},
    }
    if not args.no_cpu_baseline:
        import statistics

        import oracle
        P = oracle.Problem(xyz, tets, wl["k"], kappa).setup_amg(nu=args.nu)
        x0h = x0.cpu().numpy()
        model, ncpu = host_cpu()
        times = []
        for _ in range(3):
            t0 = time.perf_counter()
            xo, it, rr, st, _ = P.fgmres(np.zeros(P.n), tol=args.tol, restart=args.restart, x0=x0h)
            times.append(time.perf_counter() - t0)
            progress(f"oracle timed solve {len(times)}/{reps}: {times[-1]:.1f} s")
        dt = statistics.median(times)
        out["cpu_baseline"] = {"value": P.n / dt, "unit": "DOF/s", "cores": 1, "kind": "oracle",
                               "cpu_model": model, "host_cpus": ncpu, "repeats": 3,
                               "sample": f"median of 3 FP64 FGMRES({args.restart}) solves of the full {args.workload} "
                                         f"system (n_h={P.n}) by the paper's protocol to {args.tol:g}, {it} "
                                         f"steps, {dt:.1f} s each"}
        # both sides from the same random initial guess: the iterates after the
        # same number of steps are the same up to rounding
        s.set_precision("fp64")
        x64, i64, _ = s.fgmres(zero, tol=args.tol, x0=x0, restart=args.restart)
        s.set_precision("mixed")
        xm, im, _ = s.fgmres(zero, tol=args.tol, x0=x0, restart=args.restart)
        out["oracle_error"] = {"oracle_steps": it, "fp64_steps": i64.iterations, "mixed_steps": im.iterations,
                               "fp64_iterate_vs_oracle_rel_diff": rel_err(x64, xo),
                               "mixed_iterate_vs_oracle_rel_diff": rel_err(xm, xo),
                               "note": "zero right-hand side: the iterate is the remaining error after the "
                                       "steps, compared at the step counts shown"}
    return out


def run_adjoint(args):
    """One step = one forward and one backward pass of L = |u - u_t|^2 / 2
    through the autograd function: the forward CG solve u = A(kappa)^-1 f,
    the adjoint CG solve lam = A^-1 (u - u_t) and the per-tet gradient
    dL/dlog kappa_t = -lam_t^T K_t u_t (dL/df = lam).  The coefficient does
    not change between steps, so the host setup runs once, before timing."""
    import numpy as np
    import torch

    import paper_1204_2586_amd as aux
    import workloads as W

    wl = WORKLOADS[args.workload]
    xyz, tets = W.kuhn_mesh(wl["n"], jitter=wl["jitter"], seed=wl["seed"])
    logk = W.grf_log_kappa(xyz, tets, seed=wl["kappa"])
    logk_t = W.grf_log_kappa(xyz, tets, seed=wl["kappa_target"])
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    f = torch.tensor(aux.Solver(xyz, tets, wl["k"], host_only=True).load(W.manufactured_f), device=dev)
    lk0 = torch.tensor(logk, device=dev)
    res = {}
    for prec in ("mixed", "fp64"):
        prob = aux.KappaSolve(xyz, tets, wl["k"], tol=args.tol, device=dev, precision=prec, nu=args.nu)
        with torch.no_grad():
            ut = aux.AuxSolveFn.apply(f, torch.tensor(logk_t, device=dev), prob)

        def step():
            fv = f.clone().requires_grad_(True)
            lk = lk0.clone().requires_grad_(True)
            u = aux.AuxSolveFn.apply(fv, lk, prob)
            loss = 0.5 * torch.sum((u - ut) ** 2)
            loss.backward()
            return u, lk.grad, fv.grad

        t0 = time.time()
        step()                                    # the host setup for this kappa
        setup_s = time.time() - t0
        progress(f"GPU setup: {setup_s:.2f} s")
        for _ in range(args.warmup):
            step()
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(args.steps):
            u, gk, gf = step()
        torch.cuda.synchronize()
        ms = (time.perf_counter() - t) * 1e3 / args.steps
        s = prob._solver
        _, fi = s.solve(f, tol=args.tol)
        lam, ai = s.solve((u - ut).contiguous(), tol=args.tol)
        # the gradient kernel alone, HIP events on the stream it runs on
        ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        g = s.kappa_grad(u, lam)
        ev0.record()
        for _ in range(20):
            s.kappa_grad(u, lam, out=g)
        ev1.record()
        torch.cuda.synchronize()
        kg_us = ev0.elapsed_time(ev1) * 1e3 / 20
        prof = None
        if prec == "mixed":
            s.profile(True)
            for _ in range(args.steps):
                s.solve(f, tol=args.tol)
            torch.cuda.synchronize()
            prof = s.profile_read()
            s.profile(False)
        res[prec] = dict(ms=ms, setup_s=setup_s, it_forward=fi.iterations, it_adjoint=ai.iterations, kg_us=kg_us,
                         prof=prof, solver=s, gk=gk.clone())
    s = res["mixed"]["solver"]
    n, nt = s.n, len(tets)
    nloc = (wl["k"] + 1) * (wl["k"] + 2) * (wl["k"] + 3) // 6
    # per tet: nloc dof indices, the 4x4 metric, kappa and g; u and lam once
    kg_bytes = nt * (4 * nloc + 16 * 8 + 8 + 8) + 2 * 8 * n
    kernels = kernel_table(res["mixed"]["prof"], args, s, wl, nt)
    dom = max(kernels, key=lambda c: kernels[c]["total_ms"])
    kd = kernels[dom]
    gdiff = float(torch.linalg.norm(res["mixed"]["gk"] - res["fp64"]["gk"]) / torch.linalg.norm(res["fp64"]["gk"]))
    out = {
        "metric": "adjoint gradient throughput: forward solve + adjoint solve + per-tet log-coefficient gradient",
        "value": n / (res["mixed"]["ms"] * 1e-3),
        "unit": "DOF/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": res["mixed"]["ms"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64 CG / f32 preconditioner, f64 gradient",
        "data": "synthetic",
        "config": {"workload": args.workload, "order": wl["k"], "cubes_per_side": wl["n"], "n_h": n, "n_tets": nt,
                   "tol": args.tol, "nu": args.nu, "iterations_forward": res["mixed"]["it_forward"],
                   "iterations_adjoint": res["mixed"]["it_adjoint"], "setup_s": round(res["mixed"]["setup_s"], 2),
                   "kappa_grad_us": round(res["mixed"]["kg_us"], 2), "kappa_grad_bytes": kg_bytes,
                   "kappa_grad_gbs": round(kg_bytes / (res["mixed"]["kg_us"] * 1e-6) / 1e9, 1),
                   "grad_mixed_vs_fp64_rel_diff": gdiff},
        "fp64": {"value": n / (res["fp64"]["ms"] * 1e-3), "ms_per_step": res["fp64"]["ms"],
                 "iterations_forward": res["fp64"]["it_forward"], "iterations_adjoint": res["fp64"]["it_adjoint"]},
        "roofline": {"bound": "hbm", "kernel": dom, "achieved": kd["gbs"], "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": kd["gbs"] / HBM_PEAK_GBS, "traffic": None,
                     "bytes_per_launch": kd["bytes"], "avg_us": kd["avg_us"]},
    }
    if not args.no_cpu_baseline:
        import oracle
        P = oracle.Problem(xyz, tets, wl["k"], np.exp(logk)).setup_amg(nu=args.nu)
        Pt = oracle.Problem(xyz, tets, wl["k"], np.exp(logk_t)).setup_amg(nu=args.nu)
        b = f.cpu().numpy()
        u_t, _, _, _ = Pt.pcg(b, tol=args.tol)
        import statistics
        model, ncpu = host_cpu()
        times = []
        for _ in range(3):
            t0 = time.perf_counter()
            uo, it1, _, _ = P.pcg(b, tol=args.tol)
            lo, it2, _, _ = P.pcg(uo - u_t, tol=args.tol)
            go = P.kappa_grad(uo, lo)
            times.append(time.perf_counter() - t0)
            progress(f"oracle timed solve {len(times)}/{reps}: {times[-1]:.1f} s")
        dt = statistics.median(times)
        out["cpu_baseline"] = {"value": P.n / dt, "unit": "DOF/s", "cores": 1, "kind": "oracle",
                               "cpu_model": model, "host_cpus": ncpu, "repeats": 3,
                               "sample": f"median of 3: one FP64 forward solve ({it1} iterations), adjoint solve "
                                         f"({it2}) and per-tet gradient of the full {args.workload} system "
                                         f"(n_h={P.n}), {dt:.1f} s each"}
        out["oracle_error"] = {"mixed_grad_vs_oracle_rel_err": rel_err(res["mixed"]["gk"], go),
                               "fp64_grad_vs_oracle_rel_err": rel_err(res["fp64"]["gk"], go),
                               "note": "oracle gradient from its own FP64 solves to the same tolerance"}
    return out


def main():
    ap = argparse.ArgumentParser(description=__doc__)
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--workload", default="p2_n48_jitter", choices=sorted(WORKLOADS))
    ap.add_argument("--tol", type=float, default=None,
                    help="relative residual (default 1e-8 for CG, 1e-6 for FGMRES, the paper's)")
    ap.add_argument("--krylov", default="cg", choices=["cg", "fgmres", "stokes"],
                    help="cg: time to 1e-8 from zero; fgmres: the paper's protocol (zero right-hand side, "
                         "random initial guess); stokes: the P2-P1 Stokes solve with Q_t on the 48^3 mesh")
    ap.add_argument("--restart", type=int, default=30, help="FGMRES restart length")
    ap.add_argument("--nu", type=int, default=2,
                    help="l1-Jacobi sweeps before and after the coarse correction (the workloads are defined with 2)")
    ap.add_argument("--operator", default="assembled", choices=["assembled", "matfree"],
                    help="P^k products inside the preconditioner: sliced-ELL A_h or the MFMA element operator")
    ap.add_argument("--aux-space", type=int, default=1, choices=[1, 2],
                    help="auxiliary space of a single-vector workload: 1 P^1 (the paper's), 2 the intermediate "
                         "P^2 space of Remark 6.2 (orders 3 and 4)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-extras", action="store_true",
                    help="with the default workload, skip the P3 32^3 and 32-source P2 64^3 entries of the line")
    ap.add_argument("--threads", type=int, default=16, help="host threads for the load vectors of the batch")
    ap.add_argument("--batch-order", type=int, default=0, choices=[0, 1],
                    help="dof order of the batched solve: 0 the single-vector order, 1 Morton curve with die ranges")
    ap.add_argument("--coefficient-update", action="store_true",
                    help="only time new coefficients through aux_set_kappa at P2 48^3 (AMG built on the device "
                         "and on the host)")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="only run plain 1 GiB device-to-device copies (reference for HBM byte counters)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(json.dumps({"error": "this benchmark runs on one GPU only; --gpus must be 1 "
                                   "(the multi-GPU decomposition is described, not built)"}))
        sys.exit(2)
    if args.calibrate_copy:
        print(json.dumps(calibrate_copy()), flush=True)
        return
    if args.coefficient_update:
        if args.tol is None:
            args.tol = 1e-8
        print(json.dumps(run_kappa_update(args)), flush=True)
        return
    if args.tol is None:
        args.tol = 1e-6 if args.krylov == "fgmres" else 1e-8
    args.extras = (not args.no_extras and args.workload == "p2_n48_jitter" and args.krylov == "cg"
                   and args.operator == "assembled" and args.aux_space == 1)
    if args.krylov == "fgmres" and ("nrhs" in WORKLOADS[args.workload] or WORKLOADS[args.workload].get("adjoint")):
        print(json.dumps({"error": "FGMRES runs the single-vector solve workloads only"}))
        sys.exit(2)
    wl = WORKLOADS[args.workload]
    if args.krylov == "stokes":
        fn = run_stokes_pairs
    elif "nrhs" in wl:
        fn = run_batched
    elif wl.get("adjoint"):
        fn = run_adjoint
    else:
        fn = run_fgmres if args.krylov == "fgmres" else run
    print(json.dumps(fn(args)), flush=True)


if __name__ == "__main__":
    main()
