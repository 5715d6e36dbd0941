"""Benchmark of the RPA chi0 hot path on one MI355X.

Default (--mode cycle): the 48^3 workload (64 Gaussian wells on a jittered lattice, N_s = 64,
N_r = 256, 8 Gauss-Legendre frequencies, COCG tol 1e-8), RPA_MIXED (FP64 real-form solves
with an exact residual check on this grid).  A step is one pass of the hot path at one frequency: one subspace
iteration (u = nu^{1/2} V, chi0 u by the projector and 16384 batched Sternheimer solves,
Delta rho, R = nu^{1/2} chi0 u, the projected matrix and its Rayleigh-Ritz energy, Cholesky-QR)
through rpa_subspace_iter; step k works on frequency k mod 8, every frequency keeping its own
block (the independent-frequency schedule, frequency by frequency).  `value` is chi0
block-applies per second over the timed steps.  After them, time-to-E_c is measured with
rpa_energy at a fixed number of subspace iterations per frequency, in the mixed path and in
the FP64 path on the same inputs ("compare": the metric's FP32-refined vs FP64).

--mode energy: a step is rpa_energy over all frequencies plus rpa_energy_backward (the
24^3 workload's form; relative energy test, optional preconditioned or block COCG).

Inputs are synthetic, seeded and resident in HBM before the timed region.  Printed: one JSON
line with the metric, the roofline of the dominant kernel (batched COCG) measured with HIP
events on its own stream, and the CPU oracle timed on a bounded sample.
"""
import argparse
import ctypes
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
# algorithmic bytes per grid point per COCG iteration: read and write x, r, p
ALG_BYTES = {"fp64": 96.0, "mixed": 48.0}

KERNELS = {None: "cocg_wg", "streaming": "rcocg_wg", "resident-ring": "ring_wg", "resident": "full_wg"}


def real_form_kernel(precision, shape, min_omega, nsys=1 << 20):
    """(kind, ring): the real-form kernel that the library launches for nsys systems on a grid of this
    shape, and the basis vectors that it keeps; (None, 0) where the complex kernels solve (a complex64
    recurrence at every frequency, a plane without a shape, a forced launch shape)."""
    from paper_2504_01816_amd import lib as L
    if precision == "mixed" and min_omega <= 0.0:
        return None, 0
    ring = ctypes.c_int32(0)
    # mixed: complex solutions, for the exact residual
    kind = L.load().rpa_internal_real_form((ctypes.c_int32 * 3)(*shape), min(nsys, 1 << 20),
                                           int(precision == "mixed"), ctypes.byref(ring))
    return (None, "streaming", "resident-ring", "resident")[kind], ring.value


def alg_bytes(precision, shape, min_omega, nsys=1 << 20):
    """Bytes per point and iteration that the kernel that runs moves by design.  Complex kernels: x, r,
    p read and written.  Real form: a sweep reads w and v_k and writes v_{k+1} and w (32), a ring vector
    is read once more (8), complex p and x are read and written once per ring; with v, w and V_loc in
    registers a ring vector is written and read once (16) and the halves of the ring take turns; with p
    and x there too nothing (b once in and x once out, whatever the iterations)."""
    kind, ring = real_form_kernel(precision, shape, min_omega, nsys)
    if kind is None:
        return ALG_BYTES[precision]
    px = 64.0 if precision == "mixed" else 48.0
    return {"streaming": 40.0 + px / max(ring, 1), "resident-ring": 16.0 + 2 * px / max(ring, 1),
            "resident": 0.0}[kind]


def kernel_name(precision, shape, min_omega, nsys=1 << 20):
    kind, _ = real_form_kernel(precision, shape, min_omega, nsys)
    if kind:
        return ("%s (batched COCG in its real Lanczos form, one workgroup per system)" % KERNELS[kind])
    return ("cocg_wg<%s> (batched COCG, one workgroup per system)" %
            ("float, float2" if precision == "mixed" else "double, double"))


def cells_alg_bytes(precision, wl, min_omega):
    """alg_bytes over the cells of a workload, weighted with their points times systems (the
    statistics do not say which cell an iteration belongs to)."""
    w = [c.nd * c.n_occ * nr for c, nr in zip(wl.cells, wl.n_r)]
    b = [alg_bytes(precision, c.shape, min_omega) for c in wl.cells]
    return sum(x * y for x, y in zip(w, b)) / sum(w)


def solve_dtype(precision, shapes, min_omega):
    """The compute dtype of the Sternheimer solves: complex64 recurrences run only in the mixed path
    and where the real-form FP64 kernels do not take their place."""
    c64 = precision == "mixed" and any(real_form_kernel(precision, s, min_omega)[0] is None for s in shapes)
    return "c64+f64" if c64 else "c128"


def host_driven_bytes(precond, block, shape, fused_axis=32):
    """Algorithmic HBM bytes per point and system-iteration of the host-driven solvers: the
    step (q = A p; with the x and r updates for single systems: 128 B) and its direction update
    (r^T z and p: 64 B), or the block kernels (q = A p 32 B, alpha step 128 B, beta step 80 B);
    the preconditioner adds 32 B per pass: 3 fused passes where every axis has at most fused_axis
    points (64 in the library), else the 7 of the general products."""
    b = 240.0 if block >= 2 else 192.0
    if precond:
        b += 32.0 * (3 if max(shape) <= fused_axis else 7)
    return b


def subspace_converged(iters, ec_tol, cap):
    """Per cell and frequency: whether the relative energy test held before the cap of `cap`
    subspace iterations; None for a fixed count (ec_tol <= 0), which has no test."""
    if ec_tol <= 0.0:
        return None
    return [[bool(k < cap) for k in row] for row in iters]


def ec_label(iters, ec_tol, cap):
    """What time_to_ec_s measures: a fixed subspace count, or the energy test, held at every
    frequency or not."""
    if ec_tol <= 0.0:
        return "fixed count of %d subspace iterations per frequency" % cap
    cv = subspace_converged(iters, ec_tol, cap)
    n_cap = sum(1 for row in cv for c in row if not c)
    if n_cap == 0:
        return "energy test (ec_tol %g) held at every frequency" % ec_tol
    return ("not converged: %d of %d frequencies stopped at the cap of %d subspace iterations "
            "before the energy test (ec_tol %g) held" % (n_cap, sum(len(row) for row in cv),
                                                         cap, ec_tol))


def cycle_kernel_class(omega, precision, min_omega):
    """The COCG kernel a cycle step at frequency omega runs: the precision's own, or FP64 for
    a mixed step below mixed_min_omega."""
    return precision if omega >= min_omega else "fp64"


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--mode", default="cycle", choices=["cycle", "energy"],
                    help="cycle: a step is one subspace iteration at one frequency, frequencies "
                         "in turn; energy: a step is rpa_energy (+ backward)")
    ap.add_argument("--config", type=int, default=None,
                    help="workload index (0..4); default 2 (48^3) in cycle mode, 1 (24^3) in "
                         "energy mode")
    ap.add_argument("--precision", default=None, choices=["fp64", "mixed"],
                    help="default mixed in cycle mode, fp64 in energy mode")
    ap.add_argument("--refine-tol", type=float, default=0.0,
                    help="mixed: relative residual drop between reliable updates (0: library "
                         "default)")
    ap.add_argument("--mixed-min-omega", type=float, default=-1.0,
                    help="mixed: frequencies below this (Ha) solve in FP64 (negative: library "
                         "default)")
    ap.add_argument("--ec-iters", type=int, default=1,
                    help="cycle mode: fixed subspace iterations per frequency of the "
                         "time-to-E_c runs")
    ap.add_argument("--freq-mode", default="independent", choices=["warm", "independent"],
                    help="warm: frequencies in sequence, each started from the previous one's "
                         "subspace (Algorithm 1); independent: every frequency from V0, all "
                         "frequencies batched into one chi0 launch per subspace iteration")
    ap.add_argument("--sq-order", type=int, default=0,
                    help="energy by Gauss spectral quadrature of this order (0: Rayleigh-Ritz)")
    ap.add_argument("--no-backward", action="store_true")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--ec-tol", type=float, default=1e-8)
    ap.add_argument("--precond", action="store_true",
                    help="Sternheimer solves by COCG with the Kronecker shifted-Laplacian "
                         "preconditioner (FP64)")
    ap.add_argument("--block", type=int, default=0,
                    help="block COCG width (2..8; 0: single systems), with --precond "
                         "preconditioned (FP64)")
    ap.add_argument("--max-systems", type=int, default=0,
                    help="cap on COCG systems per launch (0: the library's memory budget)")
    ap.add_argument("--max-subspace", type=int, default=50)
    ap.add_argument("--cells-sequential", action="store_true",
                    help="energy mode, several cells: one rpa_energy call per cell, one after "
                         "another, instead of one call running the cells concurrently")
    ap.add_argument("--compare", default="other", choices=["none", "other"],
                    help="other: also time the same path in the other precision")
    args = ap.parse_args()
    if args.config is None:
        args.config = 2 if args.mode == "cycle" else 1
    if args.precision is None:
        args.precision = "mixed" if args.mode == "cycle" else "fp64"
    return args


def cocg_traffic(workload, precision, point_iters_per_launch):
    """HBM bytes per COCG launch from the committed FETCH_SIZE / WRITE_SIZE measurement
    (bytes per point-iteration, copy-kernel scaled) times this run's point-iterations per
    launch; None when the kernel sources changed since the counters were taken."""
    from paper_2504_01816_amd import profiling

    path = os.path.join(ROOT, "profiles", "cocg_wg_traffic.json")
    if not os.path.exists(path):
        return None, None
    sha = profiling.kernel_source_hash()
    for e in json.load(open(path))["entries"]:
        if e["precision"] == precision and e["workload"] == workload and e["kernel_source_sha256"] == sha:
            return e["bytes_per_point_iter"] * point_iters_per_launch, e["bytes_per_point_iter"]
    return None, None


def cpu_baseline(wl):
    """Oracle (as written, single BLAS thread) on two trial vectors at every frequency."""
    from threadpoolctl import threadpool_limits

    from oracle import chi0 as ochi0
    from oracle import coulomb as ocoul

    c = wl.cells[0]
    nr = wl.n_r[0]
    pick = list(range(len(wl.omegas)))
    nv = 2
    V = wl.V0[0][:nv].T.copy()
    times = []
    with threadpool_limits(1):
        for m in pick:
            t0 = time.perf_counter()
            U = ocoul.nu_apply(V, c.shape, c.h, 1)
            D, _, _ = ochi0.chi0_apply(U, c.vloc, c.psi.T, c.eps, float(wl.omegas[m]), c.shape, c.h,
                                       wl.cocg_tol, 5000)
            ocoul.nu_apply(D, c.shape, c.h, 1)
            times.append((time.perf_counter() - t0) / nv)
    per_apply = nr * float(np.mean(times))
    return {"value": 1.0 / per_apply, "unit": "chi0 block-applies/s", "cores": 1,
            "kind": "oracle",
            "sample": "%d of %d trial vectors (%d of %d Sternheimer systems, nu^1/2 both sides) "
                      "at each of the %d frequencies; block-apply time = %d x mean per-vector "
                      "time %.2f s" % (nv, nr, nv * c.n_occ, c.n_occ * nr, len(pick), nr,
                                       float(np.mean(times)))}


def _oracle_orbitals(job):
    """Worker: the oracle's Sternheimer solves (its right-hand sides, its COCG, its stencil) for
    some orbitals of one trial vector; returns their iteration counts."""
    os.environ["OMP_NUM_THREADS"] = "1"
    from oracle import chi0 as ochi0
    from oracle import cocg as ococg
    from oracle import fd as ofd

    u, vloc, psi, eps, om, shape, h, tol, orbs = job
    bp, _ = ochi0.build_rhs(u[:, None], psi, h ** 3)
    shifts = np.asarray(eps)[orbs] + 1j * om
    _, it, _ = ococg.cocg_batched(lambda v: ofd.hamiltonian_apply(v, vloc, shape, h), shifts,
                                  -bp[:, orbs], tol, 5000)
    return int(it.sum())


def cpu_baseline_parallel(wl, U0, sys_iters_per_apply, omegas_idx=(0, 1)):
    """The oracle's Sternheimer solves for one trial vector (all N_s orbitals, dealt to worker
    processes round-robin) at the highest frequencies, timed on every usable host core (at most
    16); its rate in system-iterations per second, divided into the COCG system-iterations of
    one chi0 block-apply that the FP64 GPU path measured on the same workload, gives the
    oracle's (extrapolated) block-applies per second."""
    import multiprocessing as mp
    from concurrent.futures import ProcessPoolExecutor

    c = wl.cells[0]
    ns = c.n_occ
    cores = max(1, min(16, len(os.sched_getaffinity(0))))
    psi = np.ascontiguousarray(c.psi.T)
    groups = [list(range(w, ns, cores)) for w in range(min(cores, ns))]
    total_it, wall = 0, 0.0
    with ProcessPoolExecutor(max_workers=len(groups), mp_context=mp.get_context("spawn")) as ex:
        list(ex.map(abs, range(len(groups))))          # workers started before the clock
        for m in omegas_idx:
            jobs = [(U0, c.vloc, psi, c.eps, float(wl.omegas[m]), c.shape, c.h, wl.cocg_tol, g)
                    for g in groups]
            t0 = time.perf_counter()
            total_it += sum(ex.map(_oracle_orbitals, jobs))
            wall += time.perf_counter() - t0
    rate = total_it / wall
    return {"value": rate / sys_iters_per_apply, "unit": "chi0 block-applies/s", "cores": len(groups),
            "kind": "oracle",
            "sample": "trial vector 0 (all %d Sternheimer systems, one worker process per core, "
                      "orbitals dealt round-robin) at omega = %s: %d COCG system-iterations in "
                      "%.1f s = %.1f per s; extrapolated to a block-apply by the FP64 GPU path's "
                      "mean of %.4g system-iterations per block-apply over the 8 frequencies "
                      "(projector and nu^1/2 not included)" % (
                          ns, ", ".join("%.4g" % wl.omegas[m] for m in omegas_idx), total_it,
                          wall, rate, sys_iters_per_apply)}


def run_cycle(args):
    import torch

    from paper_2504_01816_amd import api, synth
    from paper_2504_01816_amd import lib as L

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    dev = "cuda:0"
    t0 = time.perf_counter()
    wl = synth.workload(args.config, device=dev)      # ground state on the GPU (untimed)
    c = wl.cells[0]
    dc = api.device_cell(c, dev)
    nr, nf = wl.n_r[0], len(wl.omegas)
    print("[bench] workload %s generated in %.1f s" % (wl.name, time.perf_counter() - t0),
          file=sys.stderr, flush=True)
    # input preparation (untimed): the orthonormal start block, one copy per frequency
    Q, _ = torch.linalg.qr(torch.tensor(wl.V0[0], device=dev).T)
    Vs = [Q.T.contiguous() for _ in range(nf)]
    del Q
    prec = {"fp64": L.RPA_FP64, "mixed": L.RPA_MIXED}

    def opts(p):
        o = dict(precision=prec[p], cocg_tol=wl.cocg_tol, subspace_iters=1, ec_tol=0.0)
        if args.refine_tol > 0:
            o["refine_tol"] = args.refine_tol
        if args.mixed_min_omega >= 0:
            o["mixed_min_omega"] = args.mixed_min_omega
        return o

    def step(k):
        m = k % nf
        torch.cuda.synchronize()
        a = time.perf_counter()
        r = api.rpa_subspace_iter(dc, float(wl.omegas[m]), float(wl.weights[m]), Vs[m],
                                  opts(args.precision), want_ritz=False, want_saved=False)
        torch.cuda.synchronize()
        st = r["stats"]
        st["wall_s"] = time.perf_counter() - a
        st["m"] = m
        st["E"] = r["E"]
        st["status"] = r["status"]
        return st

    warm_steps = []
    for k in range(args.warmup):
        s = step(k)
        warm_steps.append(s)
        print("[bench] warmup %d: omega %.4g, %.2f s, COCG %.0f ms, iterations %d (max %d)" % (
            k, wl.omegas[s["m"]], s["wall_s"], s["cocg_kernel_ms"], s["cocg_iters_total"],
            s["cocg_iters_max"]), file=sys.stderr, flush=True)
    torch.cuda.synchronize()
    T0 = time.perf_counter()
    steps = []
    for k in range(args.warmup, args.warmup + args.steps):
        s = step(k)
        steps.append(s)
        print("[bench] step %d: omega %.4g, %.2f s, COCG %.0f ms, iterations %d (max %d), "
              "reliable updates %d, FP64 continuations %d, E_m %.12e" % (
                  k, wl.omegas[s["m"]], s["wall_s"], s["cocg_kernel_ms"], s["cocg_iters_total"],
                  s["cocg_iters_max"], s["refinements"], s["fp64_fallbacks"], s["E"]),
              file=sys.stderr, flush=True)
    torch.cuda.synchronize()
    T = time.perf_counter() - T0
    applies = sum(s["chi0_applies"] for s in steps)
    # Two classes of steps: the precision's own (in the mixed path the real-form FP64 kernel with an
    # exact residual per system, or the complex64 kernel where that does not run) and, in the mixed
    # path, the plain FP64 solves of the steps below mixed_min_omega.  Each
    # class is priced at its own kernel's algorithmic bytes over the steps whose only COCG launch is
    # that kernel (a step with FP64 continuations adds FP64 launches and is left out); the
    # roofline reports the class with the larger share of the timed region's kernel time.
    min_om = (args.mixed_min_omega if args.mixed_min_omega >= 0
              else L.default_options().mixed_min_omega) if args.precision == "mixed" else 0.0

    def kclass(s):
        return cycle_kernel_class(wl.omegas[s["m"]], args.precision, min_om)

    def kernel_entry(p):
        tsteps = [s for s in steps if kclass(s) == p]
        rsteps = [s for s in tsteps if s["cocg_launches"] == 1 and s["fp64_fallbacks"] == 0]
        n_before = sum(1 for s in warm_steps if kclass(s) == p)
        cocg_ms = sum(s["cocg_kernel_ms"] for s in rsteps)
        pit = sum(s["cocg_point_iters"] for s in rsteps)
        launches = len(rsteps)
        # a mixed step below mixed_min_omega runs the FP64 kernel
        shape, lowest = wl.cells[0].shape, min_om if p == "mixed" else 0.0
        nsys = c.n_occ * nr
        alg_pp = alg_bytes(p, shape, lowest, nsys)
        achieved = alg_pp * pit / (cocg_ms * 1e-3) / 1e9 if cocg_ms > 0 else 0.0
        avg_ms = cocg_ms / max(1, launches)
        traffic, tb = cocg_traffic(wl.name, p, pit / max(1, launches))
        entry = {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                 "frac": achieved / HBM_PEAK_GBS, "traffic": traffic,
                 "kernel": kernel_name(p, shape, lowest, nsys),
                 "launches": launches, "avg_launch_ms": avg_ms,
                 "launch_omegas": ["%.4g" % wl.omegas[s["m"]] for s in rsteps],
                 # this kernel's dispatches of the timed region within the whole run, in
                 # dispatch order (to match a kernel trace of the same command)
                 "dispatch_range": [n_before, n_before + len(tsteps)],
                 "steps_excluded_for_fp64_continuations": len(tsteps) - launches,
                 "traffic_bytes_per_point_iter": tb,
                 "traffic_GBs": (traffic / (avg_ms * 1e-3) / 1e9) if traffic else None,
                 "alg_bytes_per_point_iter": alg_pp,
                 "kernel_ms_in_timed_region": sum(s["cocg_kernel_ms"] for s in tsteps),
                 "timing": "HIP events on the launch stream"}
        return entry

    kinds = sorted({kclass(s) for s in steps})
    entries = {p: kernel_entry(p) for p in kinds}
    dom = max(kinds, key=lambda p: entries[p]["kernel_ms_in_timed_region"])
    roof = dict(entries[dom])
    roof["cocg_share_of_step"] = sum(s["cocg_kernel_ms"] for s in steps) * 1e-3 / T
    roof["other_kernels"] = [entries[p] for p in kinds if p != dom]
    per_freq = {}
    for s in steps:
        per_freq.setdefault(s["m"], []).append(s["wall_s"])
    out = {
        "metric": "chi0 block-applies/s and time-to-E_c, FP32-refined batched vs FP64, 1 GPU",
        "value": applies / T,
        "unit": "chi0 block-applies/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": 1e3 * T / args.steps,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": solve_dtype(args.precision, [c.shape], min_om),
        "data": "synthetic",
        "config": {"workload": wl.name, "grid": list(c.shape), "h": c.h, "n_occ": c.n_occ,
                   "n_r": nr, "n_freq": nf, "cocg_tol": wl.cocg_tol,
                   "systems_per_block_apply": c.n_occ * nr, "precision": args.precision,
                   "step": "one subspace iteration (one chi0 block-apply of %d vectors) at "
                           "frequency step mod %d" % (nr, nf),
                   "refine_tol": args.refine_tol or L.default_options().refine_tol,
                   "mixed_min_omega": min_om},
        "step_ms_per_frequency": {"%.4g" % wl.omegas[m]: 1e3 * float(np.mean(v))
                                  for m, v in sorted(per_freq.items())},
        "roofline": roof,
    }
    # time-to-E_c: rpa_energy from V0 at a fixed subspace count per frequency, every frequency
    # from V0 (batched-independent mode), in both precisions on the same inputs
    del Vs
    torch.cuda.empty_cache()
    V0 = torch.tensor(wl.V0[0], device=dev)
    ec = {}
    others = [args.precision] + ([p for p in ("mixed", "fp64") if p != args.precision]
                                 if args.compare == "other" else [])
    least_omega = (args.mixed_min_omega if args.mixed_min_omega >= 0
                   else L.default_options().mixed_min_omega)
    for p in others:
        o = dict(opts(p), subspace_iters=args.ec_iters, freq_mode=L.RPA_INDEPENDENT)
        torch.cuda.synchronize()
        a = time.perf_counter()
        r = api.rpa_energy(dc, nr, wl.omegas, wl.weights, [V0], o)
        torch.cuda.synchronize()
        t = time.perf_counter() - a
        st = r["stats"]
        ec[p] = dict(time_to_ec_s=t, E_c=float(r["E_c"][0]), status=r["status"],
                     chi0_block_applies_per_s=st["chi0_applies"] / t,
                     cocg_iters_total=st["cocg_iters_total"], cocg_iters_max=st["cocg_iters_max"],
                     fp64_fallbacks=st["fp64_fallbacks"], refinements=st["refinements"],
                     cocg_alg_GBs=alg_bytes(p, wl.cells[0].shape, least_omega) *
                     st["cocg_point_iters"] / (st["cocg_kernel_ms"] * 1e-3) / 1e9,
                     subspace_iters_per_freq=args.ec_iters, E_freq=r["E_freq"][0].tolist())
        print("[bench] time-to-E_c %s: %.2f s, E_c %.12e, iterations %d (max %d)" % (
            p, t, ec[p]["E_c"], st["cocg_iters_total"], st["cocg_iters_max"]), file=sys.stderr,
            flush=True)
        torch.cuda.empty_cache()
    out["time_to_ec_s"] = ec[args.precision]["time_to_ec_s"]
    out["time_to_ec_label"] = ("fixed count of %d subspace iteration(s) per frequency, every "
                               "frequency from V0 (no energy test)" % args.ec_iters)
    out["E_c"] = ec[args.precision]["E_c"]
    out["time_to_ec_runs"] = ec
    if len(ec) > 1:
        o_p = others[1]
        out["compare"] = {
            "precision": o_p,
            "time_to_ec_s": ec[o_p]["time_to_ec_s"],
            "chi0_block_applies_per_s": ec[o_p]["chi0_block_applies_per_s"],
            "E_c": ec[o_p]["E_c"],
            "E_c_rel_diff": abs(ec[o_p]["E_c"] - out["E_c"]) / abs(ec[o_p]["E_c"]),
            "time_to_ec_ratio_main_over_other": out["time_to_ec_s"] / ec[o_p]["time_to_ec_s"],
            "speedup_main_vs_other": ec[o_p]["time_to_ec_s"] / out["time_to_ec_s"],
        }
    if not args.no_cpu_baseline:
        t = time.perf_counter()
        ref = ec.get("fp64", ec[args.precision])
        U0 = api.rpa_apply_coulomb(dc, V0[:1].contiguous(), 1)[0].cpu().numpy()
        out["cpu_baseline"] = cpu_baseline_parallel(wl, U0, ref["cocg_iters_total"] / nf)
        print("[bench] cpu baseline %.1f s" % (time.perf_counter() - t), file=sys.stderr,
              flush=True)
    print(json.dumps(out), flush=True)


def run_energy(args):
    import torch

    from paper_2504_01816_amd import api, synth
    from paper_2504_01816_amd import lib as L

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    dev = "cuda:0"
    t0 = time.perf_counter()
    # the 48^3 and larger inputs get their ground states on the GPU (untimed)
    wl = synth.workload(args.config, device=dev if args.config in (2, 3, 4) else None)
    print("[bench] workload %s generated in %.1f s" % (wl.name, time.perf_counter() - t0),
          file=sys.stderr, flush=True)
    cells = [api.device_cell(c, dev) for c in wl.cells]
    V0 = [torch.tensor(v, device=dev) for v in wl.V0]
    prec = L.RPA_FP64 if args.precision == "fp64" else L.RPA_MIXED
    opts = dict(precision=prec, cocg_tol=wl.cocg_tol, subspace_iters=args.max_subspace,
                ec_tol=args.ec_tol, sq_order=args.sq_order, max_systems=args.max_systems,
                flags=L.RPA_FLAG_PRECOND if args.precond else 0, cocg_block=args.block,
                freq_mode=L.RPA_WARM if args.freq_mode == "warm" else L.RPA_INDEPENDENT)
    if wl.subspace_iters > 0:
        opts.update(subspace_iters=wl.subspace_iters, ec_tol=0.0)
    if args.refine_tol > 0:
        opts.update(refine_tol=args.refine_tol)

    def step(opts=opts):
        st = {"fwd_s": 0.0, "bwd_s": 0.0, "applies": 0, "cocg_ms": 0.0, "point_iters": 0.0,
              "launches": 0, "iters": None, "E": None}
        torch.cuda.synchronize()
        a = time.perf_counter()
        if args.cells_sequential and len(cells) > 1:
            # the cells one after another, each through its own rpa_energy call (the
            # comparison for the library's concurrent cells)
            parts = [api.rpa_energy([cc], [nr], wl.omegas, wl.weights, [v], opts,
                                    save=not args.no_backward)
                     for cc, nr, v in zip(cells, wl.n_r, V0)]
            res = {"stats": {k: sum(p["stats"][k] for p in parts)
                             for k in ("chi0_applies", "cocg_kernel_ms", "cocg_point_iters",
                                       "cocg_launches")},
                   "iters": np.concatenate([p["iters"] for p in parts]),
                   "E_c": np.concatenate([p["E_c"] for p in parts]),
                   "Vsave": sum((p["Vsave"] or [None] for p in parts), []) if not args.no_backward else None,
                   "Csave": sum((p["Csave"] or [None] for p in parts), []) if not args.no_backward else None}
        else:
            res = api.rpa_energy(cells, wl.n_r, wl.omegas, wl.weights, V0, opts,
                                 save=not args.no_backward)
        torch.cuda.synchronize()
        b = time.perf_counter()
        st["fwd_s"] = b - a
        for k in ("chi0_applies",):
            st["applies"] += res["stats"][k]
        st["cocg_ms"] += res["stats"]["cocg_kernel_ms"]
        st["point_iters"] += res["stats"]["cocg_point_iters"]
        st["launches"] += res["stats"]["cocg_launches"]
        st["iters"] = res["iters"].tolist()
        st["E"] = res["E_c"].tolist()
        if not args.no_backward:
            for ci, c in enumerate(cells):
                g, rc, s2 = api.rpa_energy_backward(c, wl.omegas, wl.weights, res["Vsave"][ci],
                                                    res["Csave"][ci], 1.0, opts)
                st["applies"] += s2["chi0_applies"]
                st["cocg_ms"] += s2["cocg_kernel_ms"]
                st["point_iters"] += s2["cocg_point_iters"]
                st["launches"] += s2["cocg_launches"]
            torch.cuda.synchronize()
            st["bwd_s"] = time.perf_counter() - b
        return st

    for w in range(args.warmup):
        s = step()
        print("[bench] warmup %d: %.2f s fwd, %.2f s bwd, subspace iters %s" %
              (w, s["fwd_s"], s["bwd_s"], s["iters"]), file=sys.stderr, flush=True)
    torch.cuda.synchronize()
    T0 = time.perf_counter()
    steps = []
    for k in range(args.steps):
        s = step()
        steps.append(s)
        print("[bench] step %d: %.2f s fwd, %.2f s bwd, applies %d, E_c %s" %
              (k, s["fwd_s"], s["bwd_s"], s["applies"], s["E"]), file=sys.stderr, flush=True)
    torch.cuda.synchronize()
    T = time.perf_counter() - T0
    applies = sum(s["applies"] for s in steps)
    cocg_ms = sum(s["cocg_ms"] for s in steps)
    pit = sum(s["point_iters"] for s in steps)
    launches = sum(s["launches"] for s in steps)
    min_om = opts.get("mixed_min_omega", L.default_options().mixed_min_omega)
    alg_pp = cells_alg_bytes(args.precision, wl, min_om)
    if args.precond or args.block >= 2:
        alg_pp = host_driven_bytes(args.precond, args.block, wl.cells[0].shape, fused_axis=64)
    alg = alg_pp * pit
    achieved = alg / (cocg_ms * 1e-3) / 1e9 if cocg_ms > 0 else 0.0
    avg_ms = cocg_ms / max(1, launches)
    timing = "HIP events on the launch stream"
    if len(cells) > 1:
        # cells run concurrently: their launches overlap, so the summed launch time overstates
        # the COCG time; the forward wall time bounds it from above instead
        fwd = sum(s["fwd_s"] for s in steps)
        achieved = alg / fwd / 1e9
        timing = ("forward wall time (cells one after another)" if args.cells_sequential
                  else "forward wall time (concurrent cells)")
    traffic, tb = cocg_traffic(wl.name, args.precision, pit / max(1, launches))
    kernel = "; ".join(dict.fromkeys(kernel_name(args.precision, x.shape, min_om) for x in wl.cells))

    def converged(iters):
        return subspace_converged(iters, opts["ec_tol"], opts["subspace_iters"])

    def label(iters):
        return ec_label(iters, opts["ec_tol"], opts["subspace_iters"])
    if args.precond or args.block >= 2:
        # the host-driven solvers: a launch is a whole solve of several kernels, and the
        # counters were taken on the plain kernel
        kernel = ("host-driven %s (all kernels of a solve)" %
                  ("block COCG" if args.block >= 2 else "preconditioned COCG"))
        traffic, tb = None, None
    out = {
        "metric": "chi0 block-applies/s and time-to-E_c, FP32-refined batched vs FP64, 1 GPU",
        "value": applies / T,
        "unit": "chi0 block-applies/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": 1e3 * T / args.steps,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": solve_dtype(args.precision, [x.shape for x in wl.cells], min_om),
        "data": "synthetic",
        "config": {"workload": wl.name, "grid": list(wl.cells[0].shape), "h": wl.cells[0].h,
                   "n_occ": wl.cells[0].n_occ, "n_r": wl.n_r[0], "n_freq": len(wl.omegas),
                   "cocg_tol": wl.cocg_tol, "ec_tol": opts["ec_tol"],
                   "backward": not args.no_backward, "precision": args.precision,
                   "freq_mode": args.freq_mode, "sq_order": args.sq_order,
                   "precond": bool(args.precond), "cocg_block": args.block},
        "time_to_ec_s": float(np.mean([s["fwd_s"] for s in steps])),
        "time_to_ec_label": label(steps[-1]["iters"]),
        "backward_s": float(np.mean([s["bwd_s"] for s in steps])),
        "E_c": steps[-1]["E"],
        "subspace_iters": steps[-1]["iters"],
        "converged": converged(steps[-1]["iters"]),
        "chi0_applies_per_step": applies / args.steps,
        "roofline": {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": achieved / HBM_PEAK_GBS, "traffic": traffic,
                     "kernel": kernel,
                     "launches": launches, "avg_launch_ms": avg_ms,
                     "traffic_bytes_per_point_iter": tb,
                     "traffic_GBs": (traffic / (avg_ms * 1e-3) / 1e9) if traffic else None,
                     "alg_bytes_per_point_iter": alg_pp,
                     "cocg_share_of_step": cocg_ms * 1e-3 / T, "timing": timing},
    }
    if args.compare == "other":
        # the metric's comparison: the same path and inputs in the other precision (complex64
        # state with float64 reliable updates against complex128); a preconditioned run is
        # compared with the plain FP64 solver instead, and so is a block COCG run
        if args.precond or args.block >= 2:
            other = "fp64"
            o2 = dict(opts, flags=0, cocg_block=0)
        else:
            other = "mixed" if args.precision == "fp64" else "fp64"
            o2 = dict(opts, precision=L.RPA_MIXED if other == "mixed" else L.RPA_FP64)
        step(o2)
        torch.cuda.synchronize()
        t = time.perf_counter()
        s2 = step(o2)
        torch.cuda.synchronize()
        t = time.perf_counter() - t
        out["compare"] = {
            "precision": other, "precond": False,
            "chi0_block_applies_per_s": s2["applies"] / t,
            "time_to_ec_s": s2["fwd_s"], "backward_s": s2["bwd_s"],
            "E_c": s2["E"], "subspace_iters": s2["iters"], "converged": converged(s2["iters"]),
            "time_to_ec_label": label(s2["iters"]),
            "E_c_rel_diff": [abs(a - b) / abs(b) for a, b in zip(s2["E"], steps[-1]["E"])],
            "cocg_alg_GBs": cells_alg_bytes(other, wl, min_om) * s2["point_iters"] / (s2["cocg_ms"] * 1e-3) / 1e9,
            "time_to_ec_ratio_vs_main": s2["fwd_s"] / out["time_to_ec_s"],
        }
        print("[bench] compare %s: %.2f s fwd, %.2f applies/s, E_c %s" % (
            other, s2["fwd_s"], out["compare"]["chi0_block_applies_per_s"], s2["E"]),
            file=sys.stderr, flush=True)
    if not args.no_cpu_baseline:
        t = time.perf_counter()
        out["cpu_baseline"] = cpu_baseline(wl)
        print("[bench] cpu baseline %.1f s" % (time.perf_counter() - t), file=sys.stderr,
              flush=True)
    print(json.dumps(out), flush=True)


def main():
    args = parse()
    if args.gpus != 1:
        print("bench.py runs on one GPU only; --gpus %d is not supported (sharding the "
              "Sternheimer systems across GPUs is described in the design notes, not "
              "implemented)" % args.gpus, file=sys.stderr)
        sys.exit(2)
    if args.mode == "cycle":
        run_cycle(args)
    else:
        run_energy(args)


if __name__ == "__main__":
    main()
