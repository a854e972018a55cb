"""Throughput of the factorized on-the-fly apply_H on one MI355X.

A step is one apply_H (diagonal + pp + nn + pn, every jump applied) in the
chosen arithmetic mode on the 20-m-state space with 5 protons and 5 neutrons
at M = 0 (dim 18,600,516), inputs resident in HBM. The library records HIP
events between its kernels on the launch stream during the timed steps, which
gives the duration of the dominant kernel (pn) for the roofline object. After
the timed steps the script runs the Lanczos comparison the metric asks for
(float32-vector path against the plain float64 path, lowest 10 of 200
iterations; the tiled float64 path beside them), thick-restart Lanczos in
float32 and float64, the block apply_H (blocks of 2, 4, 8) and block Lanczos,
the one-body densities, the adjoint (dx and every label density), a J-coupled
interaction with good-J checks, and times the CPU oracle on a bounded sample
of rows (each leg can be switched off with its --no-* flag). One JSON line is
printed.

Usage: python bench.py [--gpus 1] [--steps K] [--warmup W]
"""
import argparse
import hashlib
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "apply_H/s + HBM GB/s; FP32-MFMA vs FP64 Lanczos at 1e-5 rel eigen err"
HBM_PEAK_GBS = 8000.0
MFMA_PEAK_TFLOPS = {"f32": 157.3, "f64": 78.6}   # dense matrix-core peaks of one MI355X
MFMA_FLOPS_PER_INSTR = 2 * 16 * 16 * 4           # 16x16x4 instruction


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def kernel_source_hash():
    """Hash of the sources that shape the tiled kernels and their tables (kernel
    code, table builder, shared layout constants): stored PMC traffic is used
    only for exactly these sources."""
    h = hashlib.sha256()
    for f in ("kernels_tiled.hip", "kernels_pn_cores.hip", "tiled_common.h", "host_ham.cpp", "host_cores.cpp",
              "fotci_internal.h"):
        h.update(open(os.path.join(ROOT, "paper_1801_08432_amd", "csrc", f), "rb").read())
    return h.hexdigest()[:16]


def stored_traffic(mode):
    """HBM bytes per k_pn launch from the committed PMC summary, or None.

    The summary (profiles/pn_traffic_pf_5p5n.txt) holds lines
    'source_hash <h>' and '<mode> bytes_per_launch <B>'; values are used only
    when the hash matches the current kernel source."""
    path = os.path.join(ROOT, "profiles", "pn_traffic_pf_5p5n.txt")
    if not os.path.exists(path):
        return None
    h, val = None, None
    for line in open(path):
        f = line.split()
        if len(f) >= 2 and f[0] == "source_hash":
            h = f[1]
        if len(f) >= 3 and f[0] == mode and f[1] == "bytes_per_launch":
            val = float(f[2])
    return val if h == kernel_source_hash() else None


def cpu_baseline(w, x, seconds):
    """Time the CPU oracle's matvec on a bounded window of rows, scaled to apply_H/s."""
    from oracle import basis as ob
    from oracle import fast as of
    o = ob.build_basis(w["two_j"], w["Z"], w["N"], w["two_M"])
    prep = of.Prepared(o)
    rows = 20000
    t0 = time.perf_counter()
    of.apply_h(prep, w, x, rows=(0, rows))
    t = time.perf_counter() - t0
    # grow the window to about `seconds` of work
    rows = int(min(o.dim, max(rows, rows * seconds / max(t, 1e-3))))
    r0 = (o.dim - rows) // 2
    t0 = time.perf_counter()
    of.apply_h(prep, w, x, rows=(r0, r0 + rows))
    t = time.perf_counter() - t0
    cores = len(os.sched_getaffinity(0)) if hasattr(os, "sched_getaffinity") else os.cpu_count()
    omp = os.environ.get("OMP_NUM_THREADS")
    if omp:
        cores = min(cores, int(omp))
    return dict(value=(rows / o.dim) / t, unit="apply_H/s", cores=cores, kind="oracle",
                sample="rows %d..%d of %d (%.1f%%), %.2f s; value scaled by dim/rows" %
                       (r0, r0 + rows, o.dim, 100.0 * rows / o.dim, t),
                cpu_model=host_cpu_model(), host_ram_gb=host_ram_gb(), host_logical_cpus=os.cpu_count())


def host_cpu_model():
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return None


def host_ram_gb():
    try:
        for line in open("/proc/meminfo"):
            if line.startswith("MemTotal:"):
                return round(int(line.split()[1]) / 1024 ** 2, 1)
    except OSError:
        pass
    return None


# The paper's own timing for the same shape of problem (Ch. 3, Table
# timetable): the 48Cr pf-shell run, dimension about 2 million with about
# 1.5e9 operations per matrix-vector product (the shape of the 4p4n 20-state
# workload), took about 15 minutes for 150 Lanczos iterations on one serial
# CPU whose model the paper does not name, with single-precision vectors.
PAPER_CONTEXT = dict(
    source="Ch. 3, Table timetable",
    workload="48Cr, pf shell (20 m-states per species, 4p4n), dim ~2.0e6, ~1.5e9 operations per apply",
    time="~15 min for 150 Lanczos iterations (apply + reorthogonalisation)",
    hardware="one serial CPU run; machine not named in the paper",
    derived_lanczos_iter_per_s=round(150 / (15 * 60), 3),
    derived_ops_per_s=1.5e9 * 150 / (15 * 60),
    note="context only: a different machine, interaction and workload size from this run")


def jcoupled_leg(w, mode):
    """Rotational invariance at full size: a random J-coupled interaction on
    the same space and particle numbers, decoupled by the library; lowest 5
    converged by thick-restart Lanczos in the bench mode, then <J^2> of each
    Ritz vector with J^2 itself decoupled from J-coupled form and applied in
    float64."""
    import torch
    from paper_1801_08432_amd import fotci, inputs, observables
    dev = "cuda:0"
    space = w["two_j"]
    ep, en, pp, nn, pn = inputs.random_jcoupled(space, 1805)
    t0 = time.perf_counter()
    dec = fotci.decouple_tbme(space, pp, nn, pn)
    t_dec = time.perf_counter() - t0
    h = fotci.Hamiltonian.build(space, w["Z"], w["N"], w["two_M"], dict(eps_p=ep, eps_n=en, **dec), device=dev)
    eps, jp, jn, jpn = observables.j_squared(space)
    hj = fotci.Hamiltonian.build(space, w["Z"], w["N"], w["two_M"],
                                 dict(eps_p=eps, eps_n=eps.copy(), **fotci.decouple_tbme(space, jp, jn, jpn)),
                                 device=dev)
    piv = torch.from_numpy(inputs.random_vector(h.dim, 1806)).to(dev)
    t0 = time.perf_counter()
    tol = 1e-9 if mode.startswith("f64") else 1e-6
    r = h.lanczos_thick_restart(piv, 5, 20, 60, max_restarts=100, mode=mode, tol=tol, want_vectors=True)
    t_tr = time.perf_counter() - t0
    js, dev_max = [], 0.0
    for k in range(5):
        v = r["evecs"][k].contiguous()
        j2 = float(torch.dot(v, hj.apply(v, mode="f64")))
        J = int(round((-1 + np.sqrt(1 + 4 * max(j2, 0.0))) / 2))
        js.append(J)
        dev_max = max(dev_max, abs(j2 - J * (J + 1)))
    del h, hj
    torch.cuda.empty_cache()
    return dict(decouple_ms=round(1e3 * t_dec, 2), n_elements=len(pp) + len(nn) + len(pn), evals=r["evals"].tolist(),
                J=js, max_abs_J2_deviation=dev_max, max_resid=float(r["resid"].max()),
                thick_restart=dict(seconds=round(t_tr, 2), restarts=r["restarts"], applies=r["applies"],
                                   tol=tol, converged=r["converged"]))


def vjp_leg(h, reps=2):
    """Time the adjoint of apply_H (float64): dx = H g and every label density
    dL/dV (Ch. 5 "Two-body densities"), with per-part HIP events; the pn
    densities do one multiply-add per pn operation."""
    import torch
    from paper_1801_08432_amd import inputs
    dev = "cuda:0"
    g = torch.from_numpy(inputs.random_vector(h.dim, 1805)).to(dev)
    x = torch.from_numpy(inputs.random_vector(h.dim, 1806)).to(dev)
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(3)]
    res = {}
    for want_dx in (True, False):
        h.vjp(x, g, want_dx=want_dx)
        torch.cuda.synchronize()
        ev[0].record()
        for _ in range(reps):
            h.vjp(x, g, want_dx=want_dx)
        ev[1].record()
        torch.cuda.synchronize()
        res["with_dx" if want_dx else "densities_only"] = round(ev[0].elapsed_time(ev[1]) / reps, 3)
    pn_ops = h.op_counts()["pn"]
    return dict(ms=res["with_dx"], densities_ms=res["densities_only"], pn_ops=pn_ops,
                pn_gops=round(pn_ops / (res["densities_only"] * 1e-3) / 1e9, 2))


def density_leg(h, w, reps=5):
    """Time the one-body transition densities of two float64 vectors; the
    streamed bytes are the g and x rows (proton side) and columns (neutron
    side) read once per jump of the class that keeps m and parity."""
    import torch
    from paper_1801_08432_amd import fotci, inputs
    dev = "cuda:0"
    g = torch.from_numpy(inputs.random_vector(h.dim, 1803)).to(dev)
    x = torch.from_numpy(inputs.random_vector(h.dim, 1804)).to(dev)
    h.one_body_density(g, x)
    torch.cuda.synchronize()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(reps):
        h.one_body_density(g, x)
    e1.record()
    torch.cuda.synchronize()
    t = e0.elapsed_time(e1) / 1e3 / reps
    two_m = np.concatenate([np.arange(-tj, tj + 1, 2) for tj in w["two_j"]])
    ns = len(two_m)
    sec = h.basis.export()["sectors"]
    nbytes = 0
    for kind, first_col, count_col, size_col, n_sd in ((fotci.JUMP_P1, 2, 3, 5, h.basis.n_psd),
                                                       (fotci.JUMP_N1, 4, 5, 3, h.basis.n_nsd)):
        sd_sec = np.full(n_sd, -1)
        for si, row in enumerate(sec):
            sd_sec[row[first_col]:row[first_col] + row[count_col]] = si
        jj = h.jumps.export(kind)
        keep = (two_m[jj[:, 3] // ns] == two_m[jj[:, 3] % ns]) & (sd_sec[jj[:, 1]] >= 0)
        nbytes += int(np.sum(2 * 8 * sec[sd_sec[jj[keep, 1]], size_col]))
    return dict(ms=round(1e3 * t, 4), streamed_bytes=nbytes, achieved_gbs=round(nbytes / t / 1e9, 1))


def block_leg(h, mode, steps, one_vector_ms, nbs=(2, 4, 8)):
    """Block apply_H (blocks of n_b vectors stored row-wise): mean time per
    block apply and per kernel from HIP events, apply_H/s counted per vector,
    and the speed-up per vector over the one-vector apply."""
    import torch
    dt = torch.float64 if mode.startswith("f64") else torch.float32
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(1803)
    res = {}
    for nb in nbs:
        X = torch.randn(h.dim, nb, dtype=dt, device="cuda:0", generator=gen)
        Y = torch.empty_like(X)
        for _ in range(2):
            h.apply_block(X, Y, mode=mode)
        torch.cuda.synchronize()
        h.profile_start(steps)
        t0 = time.perf_counter()
        for _ in range(steps):
            h.apply_block(X, Y, mode=mode)
        torch.cuda.synchronize()
        t = (time.perf_counter() - t0) / steps
        kms, _ = h.profile_stop()
        res[str(nb)] = dict(ms_per_block_apply=round(1e3 * t, 4), apply_H_per_s=round(nb / t, 2),
                            speedup_per_vector=round(one_vector_ms / (1e3 * t / nb), 3),
                            kernels_ms={k: round(v, 4) for k, v in kms.items()})
        log("[bench] block apply n_b=%d: %s" % (nb, res[str(nb)]))
        del X, Y
    return dict(mode=mode, layout="row-wise (vector index fastest)", by_n_block=res)


def block_lanczos_leg(h, mode, n_block, n_iter, ref=None):
    """Block Lanczos from a seeded block: time per block iteration and per
    Krylov vector, residuals, and the lowest eigenvalues against a reference
    run when given."""
    import torch
    piv = torch.from_numpy(np.random.default_rng(1804).standard_normal((h.dim, n_block))).to("cuda:0")
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    r = h.lanczos_block(piv, 10, n_iter, mode=mode)
    t = time.perf_counter() - t0
    out = dict(mode=mode, n_block=n_block, n_iter=n_iter, blocks_done=r["n_done"], seconds=round(t, 3),
               s_per_block_iter=round(t / max(r["n_done"], 1), 5),
               s_per_vector=round(t / max(r["n_done"] * n_block, 1), 6),
               resid=[float("%.3g" % v) for v in r["resid"]], workspace_gb=round(r["workspace_bytes"] / 1e9, 2))
    if ref is not None:
        out["rel_diff_vs_standard_f64_plain"] = [float("%.3g" % v) for v in np.abs(r["evals"] - ref) / np.abs(ref)]
    log("[bench] block lanczos: %s" % out)
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--workload", default="pf_5p5n")
    ap.add_argument("--mode", default="f32")
    ap.add_argument("--lanczos-iters", type=int, default=200)
    ap.add_argument("--no-lanczos", action="store_true")
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--no-density", action="store_true")
    ap.add_argument("--no-trlan", action="store_true")
    ap.add_argument("--no-jcoupled", action="store_true")
    ap.add_argument("--no-block", action="store_true")
    ap.add_argument("--no-vjp", action="store_true")
    ap.add_argument("--block-iters", type=int, default=100)
    ap.add_argument("--cpu-seconds", type=float, default=15.0)
    ap.add_argument("--copy-calibration", action="store_true",
                    help="also copy 1 GiB (float32) once, a known-size kernel for HBM counter calibration")
    a = ap.parse_args()
    if a.gpus != 1:
        print("bench.py runs on exactly one GPU: the path is built and measured on one "
              "MI355X only (multi-GPU sharding is described in the design notes and not implemented)", file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_1801_08432_amd import fotci, inputs

    dev = "cuda:0"
    w = inputs.workload(a.workload)
    t0 = time.perf_counter()
    h = fotci.Hamiltonian.build(w["two_j"], w["Z"], w["N"], w["two_M"], w, device=dev)
    torch.cuda.synchronize()
    t_setup = time.perf_counter() - t0
    ops = h.op_counts()
    n_ops = sum(ops.values())
    log("[bench] setup %.2f s, dim %d, ops/apply %.4g" % (t_setup, h.dim, n_ops))

    mode = a.mode
    f64 = mode.startswith("f64")
    es = 8 if f64 else 4
    xs = inputs.random_vector(h.dim, 1801)
    x = torch.from_numpy(xs).to(dev)
    if not f64:
        x = x.float()
    y = torch.empty_like(x)
    for _ in range(a.warmup):
        h.apply(x, y, mode=mode)
    torch.cuda.synchronize()
    ev0 = torch.cuda.Event(enable_timing=True)
    ev1 = torch.cuda.Event(enable_timing=True)
    h.profile_start(a.steps)
    t0 = time.perf_counter()
    ev0.record()
    for _ in range(a.steps):
        h.apply(x, y, mode=mode)
    ev1.record()
    torch.cuda.synchronize()
    t_wall = time.perf_counter() - t0
    kernels_ms, n_prof = h.profile_stop()
    t_events = ev0.elapsed_time(ev1) / 1e3 / a.steps
    ms_per_step = 1e3 * t_wall / a.steps
    log("[bench] %s: %.3f ms/apply wall, %.3f ms/apply (events); kernels %s" %
        (mode, ms_per_step, 1e3 * t_events, {k: round(v, 4) for k, v in kernels_ms.items()}))

    # Roofline of the dominant kernel (k_pn). Its binding roof is the matrix
    # cores: the algorithmic work is 2 flops per pn operation, while x, y and
    # the tables read once (the compulsory bytes) would take a few hundredths
    # of a millisecond at HBM peak. achieved = useful flops per launch / the
    # launch's event-measured duration, against the dense matrix-core peak of
    # the mode's precision. The measured HBM traffic (PMC counters) and the
    # per-operation streamed-bytes model are reported beside it as labelled
    # fields, not as the roofline fraction.
    dom = "k_pn" if "k_pn" in kernels_ms else max(kernels_ms, key=kernels_ms.get)
    t_dom = kernels_ms[dom] / 1e3
    n_p1 = h.jumps.count(fotci.JUMP_P1)
    n_n1 = h.jumps.count(fotci.JUMP_N1)
    dom_ops = ops["pn"] if dom == "k_pn" else n_ops
    useful_tflops = 2 * dom_ops / t_dom / 1e12
    peak = MFMA_PEAK_TFLOPS["f64" if f64 else "f32"]
    traffic = stored_traffic(mode)
    tables = n_p1 * 12 + n_n1 * 4 + h.basis.n_psd * 64 * 4
    y_bytes = 2 * h.dim * es
    streamed = dom_ops * es + y_bytes + tables
    compulsory = h.dim * es + y_bytes + tables
    roof = dict(bound="mfma", achieved=round(useful_tflops, 3), peak=peak, unit="TFLOP/s",
                frac=round(useful_tflops / peak, 4), traffic=traffic,
                kernel=dom, kernel_ms=round(1e3 * t_dom, 4),
                work="2 flops x %d pn operations per launch" % dom_ops,
                hbm=dict(measured_bytes_per_launch=traffic,
                         measured_gbs=None if traffic is None else round(traffic / t_dom / 1e9, 1),
                         measured_frac=None if traffic is None else round(traffic / t_dom / 1e9 / HBM_PEAK_GBS, 4),
                         compulsory_bytes=compulsory,
                         compulsory_frac=round(compulsory / t_dom / 1e9 / HBM_PEAK_GBS, 5),
                         peak_gbs=HBM_PEAK_GBS),
                streamed_model=dict(bytes_per_launch=streamed,
                                    effective_gbs=round(streamed / t_dom / 1e9, 1),
                                    note="one x element per pn operation + y + tables; not HBM traffic "
                                         "(x is reused from LDS and matrix-core operands), so its GB/s can "
                                         "exceed the HBM peak"))
    # the counts of the jump kernels' lists; the core kernels' matrix-core
    # instructions are in profiles/pn_counters_pf_5p5n.txt
    cores = fotci.lib().fotci_apply_work_bytes(h._h, fotci.MODES[mode], 1) > 0
    roof["pn_kernel"] = "k_pn_core" if cores else ("k_pn" if f64 else "k_pn2")
    if dom == "k_pn" and not cores:
        pw = h.pn_work(mode)
        mf = pw["mfma_instr"] * MFMA_FLOPS_PER_INSTR / t_dom / 1e12
        roof["mfma"] = dict(instr_per_launch=pw["mfma_instr"], executed_tflops=round(mf, 2),
                            executed_frac=round(mf / peak, 4),
                            useful_over_executed=round(2 * dom_ops / (pw["mfma_instr"] * MFMA_FLOPS_PER_INSTR), 4),
                            tile_visits=pw["tile_visits"], gather_slots=pw["gather_slots"])

    out = {"metric": METRIC, "value": round(1.0 / (t_wall / a.steps), 3), "unit": "apply_H/s", "n_gpus": 1,
           "steps": a.steps, "warmup": a.warmup, "ms_per_step": round(ms_per_step, 4), "higher_is_better": True,
           "scaling": "weak", "vs_baseline": None, "dtype": "f64" if f64 else "f32", "data": "synthetic",
           "config": {"workload": "%s (2j=%s, %dp%dn, 2M=%d, dim %d)" % (a.workload, list(w["two_j"]), w["Z"],
                                                                      w["N"], w["two_M"], h.dim),
                      "mode": mode, "ops_per_apply": n_ops, "setup_s": round(t_setup, 2)},
           "kernels_ms": {k: round(v, 4) for k, v in kernels_ms.items()},
           "roofline": roof}

    # The same apply in the float64 modes (tiled, and the plain gather path),
    # for the precision path's speed-up against both.
    by_mode = {mode: round(ms_per_step, 4)}
    for m2, reps in (("f64", 10), ("f64_plain", 3)):
        if m2 == mode:
            continue
        x2 = torch.from_numpy(xs).to(dev)
        y2 = torch.empty_like(x2)
        h.apply(x2, y2, mode=m2)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(reps):
            h.apply(x2, y2, mode=m2)
        torch.cuda.synchronize()
        by_mode[m2] = round(1e3 * (time.perf_counter() - t0) / reps, 4)
        del x2, y2
    out["apply_ms_by_mode"] = by_mode
    if not f64:
        out["apply_speedup"] = dict(vs_f64_tiled=round(by_mode["f64"] / by_mode[mode], 3),
                                    vs_f64_plain=round(by_mode["f64_plain"] / by_mode[mode], 3))
    log("[bench] apply ms by mode %s" % by_mode)

    if a.copy_calibration:
        src = torch.empty(1 << 28, dtype=torch.float32, device=dev).fill_(1.0)
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst
    if not a.no_lanczos:
        piv = torch.from_numpy(inputs.random_vector(h.dim, 1802)).to(dev)
        res = {}
        for m, ro in ((mode, "cgs2"), ("f64", "cgs2"), ("f64_plain", "cgs2"), (mode, "dgks")):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            r = h.lanczos_lowest(piv, 10, a.lanczos_iters, mode=m, reorth=ro)
            t = time.perf_counter() - t0
            key = m if ro == "cgs2" else m + "_dgks"
            res[key] = (r, t)
            log("[bench] lanczos %s: %.2f s, evals %s" % (key, t, np.array2string(r["evals"][:3])))
        e32, e64 = res[mode][0]["evals"], res["f64_plain"][0]["evals"]
        rel = np.abs(e32 - e64) / np.abs(e64)
        out["lanczos"] = dict(n_iter=a.lanczos_iters, n_keep=10,
                              s_per_iter={m: round(res[m][1] / a.lanczos_iters, 5) for m in res},
                              max_rel_eig_err=float(rel.max()),
                              max_resid={m: float(res[m][0]["resid"].max()) for m in res},
                              resid_f64_plain=[float("%.3g" % v) for v in res["f64_plain"][0]["resid"]],
                              speedup_vs_f64_plain=round(res["f64_plain"][1] / res[mode][1], 3),
                              speedup_vs_f64_tiled=round(res["f64"][1] / res[mode][1], 3),
                              f64_tiled_rel_err_vs_plain=float(np.max(np.abs(res["f64"][0]["evals"] - e64) /
                                                                       np.abs(e64))),
                              dgks_rel_err_vs_f64_plain=float(np.max(np.abs(res[mode + "_dgks"][0]["evals"] - e64) /
                                                                     np.abs(e64))),
                              reorth="classical Gram-Schmidt twice (the *_dgks run: second pass only when "
                                     "the first shrinks w below 1/sqrt(2))")
    if not a.no_trlan:
        piv = torch.from_numpy(inputs.random_vector(h.dim, 1802)).to(dev)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        # float32 storage floors the true residual near 1e-7 ||H||: ask it for
        # what it can reach; float64 for 1e-8
        tol = 1e-8 if f64 else 1e-6
        r = h.lanczos_thick_restart(piv, 10, 30, 80, max_restarts=60, mode=mode, tol=tol)
        t = time.perf_counter() - t0
        tr = dict(mode=mode, n_keep=10, n_thick=30, n_basis=80, tol=tol, seconds=round(t, 2),
                  restarts=r["restarts"], applies=r["applies"], converged=r["converged"],
                  max_resid=float(r["resid"].max()), workspace_gb=round(r["workspace_bytes"] / 1e9, 2),
                  standard_workspace_gb=round(h.lanczos_workspace_bytes(10, a.lanczos_iters, mode) / 1e9, 2))
        if "lanczos" in out:
            ref = res["f64_plain"][0]["evals"]
            tr["lowest5_rel_diff_vs_standard_f64_plain"] = float(np.max(np.abs(r["evals"][:5] - ref[:5]) /
                                                                       np.abs(ref[:5])))
        # the same run in float64: all ten states converged on both sides
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        r64 = h.lanczos_thick_restart(piv, 10, 30, 80, max_restarts=60, mode="f64", tol=1e-8)
        tr["f64_seconds"] = round(time.perf_counter() - t0, 2)
        tr["f64_converged"] = r64["converged"]
        tr["f64_tol"] = 1e-8
        tr["f64_max_resid"] = float(r64["resid"].max())
        tr["max_rel_eig_err_vs_f64"] = float(np.max(np.abs(r["evals"] - r64["evals"]) / np.abs(r64["evals"])))
        out["thick_restart"] = tr
        log("[bench] thick restart: %s" % tr)
    if not a.no_block:
        out["block"] = block_leg(h, mode, a.steps, 1e3 * t_wall / a.steps)
        ref = res["f64_plain"][0]["evals"] if "lanczos" in out else None
        out["block"]["lanczos"] = block_lanczos_leg(h, mode, 4, a.block_iters, ref)
    if not a.no_density:
        out["one_body_density"] = density_leg(h, w)
    if not a.no_vjp:
        out["vjp"] = vjp_leg(h)
        log("[bench] vjp: %s" % out["vjp"])
    if not a.no_jcoupled:
        out["jcoupled"] = jcoupled_leg(w, mode)
    if not a.no_cpu:
        out["cpu_baseline"] = cpu_baseline(w, xs, a.cpu_seconds)
    out["paper_context"] = PAPER_CONTEXT
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
