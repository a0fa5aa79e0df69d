"""Benchmark of the Lindblad master-equation / quantum-jump hot path on one MI355X.

Headline workload (one "step" = one full adaptive solve): the dissipative transverse-field Ising
chain, L = 8 (d = 256, Liouvillian 65,536 x 65,536 with 1,245,183 non-zeros), J = 1, h = 0.7,
gamma = 0.2, all spins up, t in [0, 10], <sigma_z^i> at 100 times, solved by the mixed-precision
CSR path (complex64 right-hand side and stages, FP64 step control / error norm / trace / expectations) at the
loosest tolerance whose result stays within 1e-4 of a tight FP64 oracle solution.
``value`` = Liouvillian right-hand-side evaluations per second over the timed solves.

The same JSON line carries: the FP64 single-solve path on the same problem, the rate of the solve's
right-hand side against the vector peak, the roofline of the fused SpMV-stage kernel (live, HIP
events; what a solve takes whose operators have no operator form) at this size and at an HBM-sized
Liouvillian (L = 10) beside the measured copy and read bandwidth, the 512-cavity parameter sweep (batched solves/s: all
in the dense form, and with the costliest cavities in the CSR form), the
quantum-jump ensemble (trajectories/s), the served request stream (p50/p99 latency over a load
sweep), the time-dependent, stochastic, Schrodinger and steady-state solvers, and the FP64 CPU
oracle timed on this host.

Usage: python bench.py [--gpus 1] [--steps K] [--warmup W] [--skip-extra] [--no-cpu]
                       [--only SECTIONS] [--sweep-forms POLICIES]
"""
import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

import workloads  # noqa: E402
import paper_2504_21440_amd as qt  # noqa: E402

HBM_PEAK_GBS = 8000.0
FP32_VECTOR_PEAK_TFLOPS = 157.3
METRIC = "Lindblad RHS evals/s + batched solves/s at 1e-4 error vs FP64; p50/p99 latency"
LADDER = [1e-4, 3e-5, 1e-5, 3e-6, 1e-6]


def log(*a):
    print("[bench]", *a, file=sys.stderr, flush=True)


def sz_ops(L):
    import scipy.sparse as sp
    ops = []
    for i in range(L):
        diag = np.array([1.0 if ((s >> (L - 1 - i)) & 1) == 0 else -1.0 for s in range(2 ** L)])
        ops.append(sp.diags(diag.astype(complex), 0, format="csr"))
    return ops


def up_ket(L):
    v = np.zeros(2 ** L, complex)
    v[0] = 1
    return v


def load_golden(name):
    with open(os.path.join(ROOT, "tests", "golden", name + ".json")) as f:
        g = json.load(f)
    return np.array(g["expect_re"]) + 1j * np.array(g["expect_im"])


CSR_SHAPES = [(l, r) for l in (4, 8, 16) for r in (1, 2, 4) if r <= l]
CSR_WIDE_SHAPES = [(4, 1), (8, 1), (8, 2), (16, 1)]  # also built with 16-byte matrix loads


def spmv_bytes(n, nnz, val_bytes):
    """Algorithmic HBM bytes of one CSR SpMV: values + column indices, row pointers, x read, y write."""
    return nnz * (val_bytes + 4) + (n + 1) * 4 + 2 * n * val_bytes


def calibrate(ctx, L_obj, p, prec, ref, tol=1e-4):
    """Loosest rtol in the ladder (atol = rtol/100) whose solution is within tol of the tight reference."""
    tl = workloads.tlist(p["t_end"], p["nt"])
    chosen = None
    for rt in LADDER:
        ex, st, _ = qt.mesolve(ctx, L_obj, up_ket(p["L"]), tl, sz_ops(p["L"]),
                               options=qt.opts(abstol=rt / 100, reltol=rt, precision=prec))
        err = float(np.abs(ex - ref).max())
        log(f"  calibrate prec={prec} rtol={rt:g}: err={err:.2e} steps={st['n_accept']}")
        if err <= tol:
            chosen = (rt, err)
            break
    return chosen


def time_plan(plan, steps, warmup):
    for _ in range(warmup):
        plan.run()
    t0 = time.perf_counter()
    for _ in range(steps):
        plan.run()
    dt = time.perf_counter() - t0
    return dt


def section_ising(ctx, steps, warmup):
    p = workloads.ising_single()
    H, cs = qt.model_ising(p["L"], p["J"], p["h"], p["gamma"])
    ref = load_golden("ising_l8_tight")
    tl = workloads.tlist(p["t_end"], p["nt"])
    out = {}
    for name, prec in [("mixed", qt.MIXED), ("fp64", qt.F64)]:
        Lo = qt.Liouvillian(ctx, H, cs, qt.FORM_CSR, prec)
        d, nnz, nbytes = Lo.info()
        cal = calibrate(ctx, Lo, p, prec, ref)
        rt, err = cal if cal else (1e-6, float("nan"))
        # untimed set-up: the autotuner picks the CSR tile shape for this size (unless its table
        # already holds one)
        o = qt.opts(abstol=rt / 100, reltol=rt, precision=prec, autotune=True)
        plan = qt.MePlan(ctx, [(Lo, up_ket(p["L"]), tl, sz_ops(p["L"]))], o)
        shape = plan.shape()
        dt = time_plan(plan, steps, warmup)
        ex, st, _ = plan.result(0)
        err = float(np.abs(ex - ref).max())
        n_rhs = st["n_rhs"]
        ms_stage = plan.time_rhs(reps=200)
        n = d * d
        vb = 8 if prec == qt.MIXED else 16
        b = spmv_bytes(n, nnz, vb)
        out[name] = {"rtol": rt, "atol": rt / 100, "max_err_vs_tight_fp64": err, "n_accept": st["n_accept"],
                     "n_reject": st["n_reject"], "n_rhs": n_rhs, "ms_per_solve": 1e3 * dt / steps,
                     "solves_per_s": steps / dt, "rhs_per_s": n_rhs * steps / dt,
                     "stage_kernel_ms": ms_stage, "spmv_bytes": b, "stage_kernel_GBs": b / (ms_stage * 1e-3) / 1e9,
                     "nnz": nnz, "n": n, "csr_shape": list(shape[:4])}
        log(f"ising L=8 {name}: {out[name]}")
        plan.close()
        Lo.close()
    return out


def section_ising_batch(ctx, rt, steps, warmup, n=16):
    """n L=8 chains (h = 0.3 + 0.08 i) advanced together by one plan, mixed precision at the
    accuracy-matched tolerance of the single chain: batched solves/s."""
    probs, Ls = [], []
    for p in workloads.ising_batch(n=n):
        H, cs = qt.model_ising(p["L"], p["J"], p["h"], p["gamma"])
        Lo = qt.Liouvillian(ctx, H, cs, qt.FORM_CSR, qt.MIXED)
        Ls.append(Lo)
        probs.append((Lo, up_ket(p["L"]), workloads.tlist(p["t_end"], p["nt"]), sz_ops(p["L"])))
    plan = qt.MePlan(ctx, probs, qt.opts(abstol=rt / 100, reltol=rt, precision=qt.MIXED, autotune=True))
    dt = time_plan(plan, steps, warmup)
    sts = [plan.result(i)[1] for i in range(n)]
    with open(os.path.join(ROOT, "tests", "golden", "ising_batch_members.json")) as f:
        members = json.load(f)["members"]
    err = max(float(np.abs(plan.result(m["index"])[0] - (np.array(m["expect_re"]) + 1j * np.array(m["expect_im"]))).max())
              for m in members)
    out = {"instances": n, "rtol": rt, "atol": rt / 100, "solves_per_s": n * steps / dt,
           "max_err_vs_fp64_oracle_members": err, "members_checked": [m["index"] for m in members],
           "ms_per_batch": 1e3 * dt / steps, "rhs_per_s": sum(s["n_rhs"] for s in sts) * steps / dt,
           "max_steps": max(s["n_accept"] + s["n_reject"] for s in sts), "csr_shape": list(plan.shape()[:4])}
    log(f"ising L=8 batch of {n}: {out}")
    plan.close()
    for Lo in Ls:
        Lo.close()
    return out


def section_kerr_single(ctx, reps=5):
    """The driven Kerr cavity (N = 20, Delta = 1, U = 0.5, F = 0.8, kappa = 1) in plain FP64 at the
    default tolerances (abstol 1e-8, reltol 1e-6), t in [0, 20] with <a^dag a> at 200 times, CSR form
    (400 Liouville rows, 2,280 non-zeros; one workgroup integrates it): RHS
    evaluations per second, solve time and steps, the error against the stored FP64 oracle solution
    (same integrator and tolerances), and the U = 0 variant against the coherent-state closed form
    alpha(t) = alpha_ss (1 - exp(-(i Delta + kappa/2) t)), alpha_ss = -i F / (i Delta + kappa/2)."""
    p = workloads.kerr_single()
    N = p["N"]
    tl = workloads.tlist(p["t_end"], p["nt"])
    rho0 = np.zeros((N, N), complex)
    rho0[0, 0] = 1
    num = np.diag(np.arange(N, dtype=float)).astype(complex)
    out = {"N": N, "n": N * N, "t_end": p["t_end"], "n_t": p["nt"], "abstol": 1e-8, "reltol": 1e-6}
    for U, key in [(p["U"], "U0.5"), (0.0, "U0")]:
        H, c = qt.model_kerr(N, p["delta"], U, p["F"], p["kappa"])
        Lo = qt.Liouvillian(ctx, H, c, qt.FORM_CSR, qt.F64)
        plan = qt.MePlan(ctx, [(Lo, rho0, tl, [num])], qt.opts(precision=qt.F64))
        dt = time_plan(plan, reps, 1)
        ex, st, _ = plan.result(0)
        if U != 0.0:
            err = float(np.abs(ex[0] - load_golden("kerr_n20_u05")[0]).max())
            ref_kind = "FP64 oracle, same tolerances"
        else:
            z = 1j * p["delta"] + p["kappa"] / 2
            al = (-1j * p["F"] / z) * (1 - np.exp(-z * tl))
            err = float(np.abs(ex[0] - np.abs(al) ** 2).max())
            ref_kind = "coherent-state closed form"
        out[key] = {"U": U, "ms_per_solve": 1e3 * dt / reps, "solves_per_s": reps / dt,
                    "rhs_per_s": st["n_rhs"] * reps / dt, "n_accept": st["n_accept"], "n_reject": st["n_reject"],
                    "n_rhs": st["n_rhs"], "stage_kernel_us": 1e3 * plan.time_rhs(reps=200), "nnz": Lo.info()[1],
                    "max_err": err, "reference": ref_kind}
        log(f"kerr N=20 {key}: {out[key]}")
        plan.close()
        Lo.close()
    return out


def section_hbm_spmv(ctx):
    """Fused SpMV-stage kernel on an HBM-sized Liouvillian (L = 10: 1,048,576 rows, 24.6 M nnz)."""
    out = {}
    H, cs = qt.model_ising(10, 1.0, 1.0, 0.1)
    tl = np.linspace(0, 0.1, 2)
    for name, prec, vb in [("mixed", qt.MIXED, 8), ("fp64", qt.F64, 16)]:
        Lo = qt.Liouvillian(ctx, H, cs, qt.FORM_CSR, prec)
        d, nnz, _ = Lo.info()
        plan = qt.MePlan(ctx, [(Lo, up_ket(10), tl, [])], qt.opts(precision=prec, autotune=True))
        shape = plan.shape()
        n = d * d
        b = spmv_bytes(n, nnz, vb)
        by_shape = {}
        for keep in (0, 1, 2):
            for xcd in (0, 1):
                for lpr, rg in (CSR_SHAPES if keep < 2 else CSR_WIDE_SHAPES):
                    plan.set_shape(lpr, rg, xcd, keep)
                    tag = f"{lpr}x{rg}" + ("x" if xcd else "") + ("", "k", "w")[keep]
                    by_shape[tag] = round(b / (plan.time_rhs(reps=20) * 1e-3) / 1e9, 1)
        plan.set_shape(*shape[:4])
        ms = plan.time_rhs(reps=50)
        gbs = b / (ms * 1e-3) / 1e9
        out[name] = {"n": n, "nnz": nnz, "bytes_per_launch": b, "ms_per_launch": ms, "GBs": gbs,
                     "frac_of_hbm_peak": gbs / HBM_PEAK_GBS, "csr_shape": list(shape[:4]),
                     "GBs_by_shape": by_shape}
        log(f"HBM SpMV L=10 {name}: {out[name]}")
        plan.close()
        Lo.close()
    return out


def kerr_spectral_estimate(p):
    """Estimate of the Kerr-cavity Liouvillian's spectral radius: the spread of the levels
    E_n = -delta n + U n (n - 1) / 2 (the coherent part's largest frequency), plus the damping
    (kappa N) and the drive (2 F sqrt N)."""
    n = np.arange(p["N"])
    lev = -p["delta"] * n + 0.5 * p["U"] * n * (n - 1)
    return np.ptp(lev) + p["kappa"] * p["N"] + 2.0 * p["F"] * np.sqrt(p["N"])


def kerr_dense_cost(p):
    """A-priori cost of one cavity's dense-form solve, in MFMA instructions.  An explicit
    Runge-Kutta step is held to h ~ 3 / rho(L), so the right-hand sides grow as t_end rho(L); each
    costs the MFMA instructions of the operator-form products at the padded size (P and X on every
    16 x 16 tile, C X^dag on the upper ones, real collapse operator)."""
    npad = -(-p["N"] // 16) * 16
    nt, kf = npad // 16, npad // 4
    return p["t_end"] * kerr_spectral_estimate(p) * (nt * nt * kf * 6 + nt * (nt + 1) // 2 * kf * 2)


def sweep_forms(sweep, policy):
    """Form per cavity.  "dense": all dense.  "n<K>": dense up to N = K, CSR above.  "stiff<f>": dense
    unless the cavity's estimated dense cost is at least f times the largest one's.  One cavity owns
    one CU in the dense form, so the stiffest cavities set that form's makespan; the CSR form
    spreads each of them over the whole chip (about 8 us per right-hand side alone, 13 us beside
    the dense buckets, against 20 us for one NP = 80 cavity on its CU)."""
    if policy == "dense":
        return [qt.FORM_DENSE] * len(sweep)
    if policy.startswith("n"):
        k = int(policy[1:])
        return [qt.FORM_DENSE if p["N"] <= k else qt.FORM_CSR for p in sweep]
    if policy.startswith("stiff"):
        f = float(policy[5:])
        cost = np.array([kerr_dense_cost(p) for p in sweep])
        return [qt.FORM_DENSE if c < f * cost.max() else qt.FORM_CSR for c in cost]
    raise ValueError(f"unknown sweep form policy {policy!r}")


def section_sweep(ctx, n=512, policy="dense"):
    """512 driven Kerr cavities, N ~ U{10..80}, mixed precision, one plan.  The policy (sweep_forms)
    picks each cavity's form; one workgroup integrates a cavity of either form."""
    sweep = workloads.kerr_sweep(n=n)
    forms = sweep_forms(sweep, policy)
    probs = []
    Ls = []
    for p, form in zip(sweep, forms):
        H, c = qt.model_kerr(p["N"], p["delta"], p["U"], p["F"], p["kappa"])
        Lo = qt.Liouvillian(ctx, H, c, form, qt.MIXED)
        Ls.append(Lo)
        rho0 = np.zeros((p["N"], p["N"]), complex)
        rho0[0, 0] = 1
        num = np.diag(np.arange(p["N"], dtype=float)).astype(complex)
        probs.append((Lo, rho0, workloads.tlist(p["t_end"], p["nt"]), [num]))
    o = qt.opts(abstol=1e-7, reltol=1e-5, precision=qt.MIXED, autotune=True)
    plan = qt.MePlan(ctx, probs, o)
    plan.run()
    t0 = time.perf_counter()
    plan.run()
    dt = time.perf_counter() - t0
    n_rhs = 0
    flops = 0.0
    res = []
    worst = (0, -1)
    for i, p in enumerate(sweep):
        ex, st, _ = plan.result(i)
        res.append(ex)
        n_rhs += st["n_rhs"]
        flops += st["n_rhs"] * 24.0 * p["N"] * (p["N"] + 1)
        worst = max(worst, (st["n_rhs"], i))
    with open(os.path.join(ROOT, "tests", "golden", "kerr_sweep_samples.json")) as f:
        samples = json.load(f)["instances"]
    err = max(float(np.abs(res[q["index"]] - (np.array(q["expect_re"]) + 1j * np.array(q["expect_im"]))).max())
              for q in samples)
    out = {"instances": n, "solves_per_s": n / dt, "ms_per_batch": dt * 1e3, "rhs_per_s": n_rhs / dt,
           "rtol": o.reltol, "atol": o.abstol, "form_policy": policy,
           "csr_instances": sum(1 for f in forms if f == qt.FORM_CSR),
           "max_err_vs_fp64_oracle_samples": err, "samples_checked": [q["index"] for q in samples]}
    if policy == "dense":
        # One workgroup integrates one cavity (k_res): 6 generator entries per element, one complex FMA each,
        # on the elements i <= j.  The stiffest cavity sets the makespan.
        nw, iw = worst
        out["algorithmic_TFLOPs_concurrent"] = flops / dt / 1e12
        out["frac_of_fp32_vector_peak_concurrent"] = flops / dt / 1e12 / FP32_VECTOR_PEAK_TFLOPS
        out["stiffest_instance"] = {"index": iw, "N": sweep[iw]["N"], "n_rhs": nw, "us_per_rhs": dt / nw * 1e6}
    else:
        out["csr_shape"] = list(plan.shape()[:4])
    plan.close()
    return out, sweep, res


def section_mc(ctx):
    """Quantum-jump ensemble: L = 10 chain, 10,000 trajectories, complex64 states with FP64 control."""
    p = workloads.ising_mc()
    H, cs = qt.model_ising(p["L"], p["J"], p["h"], p["gamma"])
    tl = workloads.tlist(p["t_end"], p["nt"])
    Sz = sum(sz_ops(p["L"]))
    me = load_golden("ising_l10_me")[0].real
    import scipy.sparse as sp
    Heff = sp.csr_matrix(H - 0.5j * sum(c.conj().T @ c for c in cs))
    d = Heff.shape[0]
    width = int(np.diff(Heff.indptr).max())  # ELL width of -i H_eff (entries per row)
    flops_rhs = 8.0 * d * width              # one complex FMA per stored entry
    out = {"ntraj": p["ntraj"], "d": d, "ell_width": width}
    for name, prec in [("mixed", qt.MIXED), ("fp64", qt.F64)]:
        o = qt.opts(abstol=1e-6, reltol=1e-4, precision=prec)
        plan = qt.McPlan(ctx, H, cs, up_ket(p["L"]), tl, [Sz], p["ntraj"], p["seed"], options=o)
        plan.run()
        t0 = time.perf_counter()
        plan.run()
        dt = time.perf_counter() - t0
        r = plan.result()
        z = np.abs(r["mean"][0].real - me)[1:] / r["se"][0, 1:]
        st = r["stats"]
        sec = {"seconds": dt, "trajectories_per_s": p["ntraj"] / dt, "traj_rhs_per_s": st["n_rhs"] / dt,
               "device_ms": st["device_ms"], "jumps_per_traj_mean": float(r["njumps"].mean()),
               "jumps_histogram": np.bincount(r["njumps"]).tolist(), "max_z_vs_oracle_me": float(z.max()),
               "points_over_3se": int((z > 3).sum()), "rtol": o.reltol, "atol": o.abstol}
        if prec == qt.MIXED:
            tf = st["n_rhs"] * flops_rhs / (st["device_ms"] * 1e-3) / 1e12
            sec["roofline"] = {"kernel": "k_mc<float,...> (one workgroup per trajectory; state and -i H_eff in registers)",
                               "bound": "alu", "flops_per_traj_rhs": flops_rhs,
                               "achieved_TFLOPs": tf, "peak_TFLOPs": FP32_VECTOR_PEAK_TFLOPS,
                               "frac": tf / FP32_VECTOR_PEAK_TFLOPS}
        out[name] = sec
        plan.close()
    log(f"mc: {out}")
    return out


def _serve_ops(p):
    """Host operators of one served request: (H, c_ops, initial state, tlist, [observable])."""
    if p["kind"] == "kerr":
        H, c = qt.model_kerr(p["N"], p["delta"], p["U"], p["F"], p["kappa"])
        rho0 = np.zeros((p["N"], p["N"]), complex)
        rho0[0, 0] = 1
        num = np.diag(np.arange(p["N"], dtype=float)).astype(complex)
        return H, c, rho0, workloads.tlist(p["t_end"], p["nt"]), [num]
    H, cs = qt.model_ising(p["L"], p["J"], p["h"], p["gamma"])
    return H, cs, up_ket(p["L"]), workloads.tlist(p["t_end"], p["nt"]), [sz_ops(p["L"])[0]]


def _serve_build(ctx, p, prec):
    """A request's assembly: host operators and the device Liouvillian (CSR form)."""
    H, cs, r0, tl, e = _serve_ops(p)
    return qt.Liouvillian(ctx, H, cs, qt.FORM_CSR, prec), r0, tl, e


def _serve_mixed(ctx, trace, o, steps_per_epoch=32):
    """Continuous batching: each request is assembled (operators and Liouvillian) when it arrives and
    submitted as soon as it is admitted; latency = completion - arrival, assembly included."""
    srv = qt.Server(ctx, pool_bytes=16 << 30, max_slots=1024, steps_per_epoch=steps_per_epoch, options=o)
    lat, asm, results, built = [], [], {}, {}
    waiting, tickets = list(range(len(trace))), {}
    t0 = time.perf_counter()
    while waiting or tickets:
        now = time.perf_counter() - t0
        while waiting and trace[waiting[0]]["arrival"] <= now:
            i = waiting[0]
            if i not in built:
                ta = time.perf_counter()
                built[i] = _serve_build(ctx, trace[i], qt.MIXED)
                asm.append(time.perf_counter() - ta)
            tk = srv.submit(*built[i])
            if tk is None:
                break  # no room yet: stays queued until requests retire
            tickets[tk] = waiting.pop(0)
        if not tickets:
            time.sleep(max(0.0, trace[waiting[0]]["arrival"] - (time.perf_counter() - t0)))
            continue
        srv.step()
        now = time.perf_counter() - t0
        for tk in list(tickets):
            r = srv.poll(tk)
            if r is not None:
                i = tickets.pop(tk)
                lat.append(now - trace[i]["arrival"])
                results[trace[i]["id"]] = r[0][0]
                built.pop(i)[0].close()
    span = time.perf_counter() - t0
    srv.close()
    return np.array(lat), span, results, np.array(asm)


def _serve_fp64_fifo(ctx, trace, o):
    """The plain FP64 single-solve path: one request at a time in arrival order, each assembled and
    solved by qt_mesolve."""
    lat, results = [], {}
    t0 = time.perf_counter()
    for p in trace:
        now = time.perf_counter() - t0
        if p["arrival"] > now:
            time.sleep(p["arrival"] - now)
        L, r0, tl, e = _serve_build(ctx, p, qt.F64)
        ex, _, _ = qt.mesolve(ctx, L, r0, tl, e, options=o)
        L.close()
        lat.append(time.perf_counter() - t0 - p["arrival"])
        results[p["id"]] = ex[0]
    return np.array(lat), time.perf_counter() - t0, results


def _serving_refs():
    """Stored FP64 oracle solutions (abstol 1e-10, reltol 1e-8) of the first requests of the stream."""
    path = os.path.join(ROOT, "tests", "golden", "serving_trace240.json")
    if not os.path.exists(path):
        return {}, None
    with open(path) as f:
        g = json.load(f)
    return {r["id"]: np.array(r["expect_re"][0]) + 1j * np.array(r["expect_im"][0]) for r in g["requests"]}, g


def _errors(results, refs):
    e = np.array([float(np.abs(results[i] - refs[i]).max()) for i in results if i in refs])
    if e.size == 0:
        return {"checked": 0}
    return {"checked": int(e.size), "max": float(e.max()), "p99": float(np.percentile(e, 99)),
            "median": float(np.median(e)), "over_1e-4": int((e > 1e-4).sum())}


def _serve_calibration_ids(trace, refs, n_kerr=4, n_ising=2):
    """The stiffest requests with stored references: the Kerr cavities with the largest U N^2 and the
    first L = 9 chains."""
    kerr = sorted((p for p in trace if p["kind"] == "kerr" and p["id"] in refs), key=lambda p: -p["U"] * p["N"] ** 2)
    ising = [p for p in trace if p["kind"] == "ising" and p["L"] == 9 and p["id"] in refs]
    return [p["id"] for p in kerr[:n_kerr]] + [p["id"] for p in ising[:n_ising]]


def _serve_calibrate(ctx, trace, refs, ids, prec):
    """Loosest ladder rtol (atol = rtol/100) whose solutions of the calibration requests are all within
    1e-4 of the stored references.  Mixed: one plan at the server's CSR launch shape; FP64: qt_mesolve
    one request at a time, as the single-solve path runs them."""
    if not ids:  # no stored references: the tolerance the server ran at before calibration existed
        return 1e-5, []
    byid = {p["id"]: p for p in trace}
    built = [_serve_build(ctx, byid[i], prec) for i in ids]
    chosen, rungs = None, []
    for rt in LADDER:
        o = qt.opts(abstol=rt / 100, reltol=rt, precision=prec)
        if prec == qt.MIXED:
            plan = qt.MePlan(ctx, built, o)
            plan.set_shape(8, 1, 0, 1)
            plan.run()
            res = {i: plan.result(k)[0][0] for k, i in enumerate(ids)}
            plan.close()
        else:
            res = {i: qt.mesolve(ctx, *b, options=o)[0][0] for i, b in zip(ids, built)}
        err = max(float(np.abs(res[i] - refs[i]).max()) for i in ids)
        rungs.append({"rtol": rt, "max_err": err})
        log(f"  serving calibration prec={prec} rtol={rt:g}: err={err:.2e}")
        if err <= 1e-4:
            chosen = rt
            break
    for b in built:
        b[0].close()
    return (chosen if chosen is not None else LADDER[-1]), rungs


def section_serving(ctx, n=240, qps=40.0, n_long=2000):
    """Poisson stream of 70% Kerr cavities (N 10..80) and 30% Ising chains (L 4..9), served with
    continuous batching in mixed precision through the CSR form (the Kerr operators are tridiagonal:
    the CSR right-hand side does far fewer flops than the dense form).  Each request is assembled
    when it arrives, so latencies include assembly.  Tolerances: for each path, the loosest ladder
    rtol whose solutions of the stiffest stored requests stay within 1e-4 of the oracle.  Every
    result of the first 240 requests is compared with its stored oracle solution after the timed
    window.  X = saturating throughput (all requests at once); the load sweep offers 0.25, 0.5, 0.7
    and 0.9 X; the plain FP64 single-solve path (qt_mesolve, one request at a time, FIFO) serves the
    same 240-request trace at 40 QPS as the mixed server; a 2,000-request stream runs at 0.7 X."""
    refs, _ = _serving_refs()
    cal_trace = workloads.serving_trace(n=n)
    ids = _serve_calibration_ids(cal_trace, refs)
    rt_m, rungs_m = _serve_calibrate(ctx, cal_trace, refs, ids, qt.MIXED)
    rt_f, rungs_f = _serve_calibrate(ctx, cal_trace, refs, ids, qt.F64)
    om_ = qt.opts(abstol=rt_m / 100, reltol=rt_m, precision=qt.MIXED)
    of_ = qt.opts(abstol=rt_f / 100, reltol=rt_f, precision=qt.F64)

    def summary(lat, span, res, asm, nreq):
        return {"solves_per_s": nreq / span, "makespan_s": span, "p50_s": float(np.percentile(lat, 50)),
                "p99_s": float(np.percentile(lat, 99)), "assembly_ms_p50": 1e3 * float(np.median(asm)),
                "errors_vs_oracle": _errors(res, refs)}

    lat, span, res, asm = _serve_mixed(ctx, workloads.serving_trace(n=n, qps=1e9), om_)
    x_sat = n / span
    out = {"requests": n, "calibration_requests": ids, "mixed_rtol": rt_m, "mixed_calibration": rungs_m,
           "fp64_rtol": rt_f, "fp64_calibration": rungs_f, "saturated": summary(lat, span, res, asm, n)}

    def at(q, nreq=n):
        lat, span, res, asm = _serve_mixed(ctx, workloads.serving_trace(n=nreq, qps=q), om_)
        return dict(summary(lat, span, res, asm, nreq), qps=q, requests=nreq)

    out["load_sweep"] = {f"{f}x": at(f * x_sat) for f in (0.25, 0.5, 0.7, 0.9)}
    out["at_qps"] = at(qps)
    lat_f, span_f, res_f = _serve_fp64_fifo(ctx, workloads.serving_trace(n=n, qps=qps), of_)
    out["fp64_single_fifo_at_qps"] = {"qps": qps, "requests": n, "solves_per_s": n / span_f, "makespan_s": span_f,
                                      "p50_s": float(np.percentile(lat_f, 50)),
                                      "p99_s": float(np.percentile(lat_f, 99)),
                                      "errors_vs_oracle": _errors(res_f, refs)}
    # the single-solve path is overloaded at this rate (arrivals outpace it), so its solves/s is its
    # saturated throughput, compared with the server's saturated throughput X
    out["saturated_mixed_vs_fp64_fifo_solves_per_s"] = x_sat / out["fp64_single_fifo_at_qps"]["solves_per_s"]
    out["long_stream_0.7x"] = at(0.7 * x_sat, n_long)
    log(f"serving: {out}")
    return out


def _optomech_ops(p):
    """Operators of the driven optomechanical system (cavity first), built with scipy."""
    import scipy.sparse as sp

    def destroy(N):
        return sp.diags(np.sqrt(np.arange(1, N, dtype=float)), 1, shape=(N, N), format="csr").astype(complex)

    a = sp.kron(destroy(p["Nc"]), sp.identity(p["Nm"]), format="csr")
    b = sp.kron(sp.identity(p["Nc"]), destroy(p["Nm"]), format="csr")
    ad, bd = a.conj().T, b.conj().T
    xa = (a + ad).tocsr()
    H0 = (p["wc"] * (ad @ a) + p["wm"] * (bd @ b) + 0.5 * p["g"] * (xa @ xa) @ (b + bd)).tocsr()
    c_ops = [np.sqrt(p["kappa"]) * a, np.sqrt(p["gamma"]) * b]
    return H0, xa, c_ops, (ad @ a).tocsr()


def section_td(ctx, n_sweep=64):
    """Time-dependent master equation: the driven optomechanical system (drive F cos(w_d t) on
    a + a^dag), one full solve over t in [0, 5/kappa] with 5000 saves in FP64 and mixed precision,
    then n_sweep drive frequencies over t in [0, 100] in one plan (mixed)."""
    p = workloads.optomech_td()
    H0, xa, c_ops, n_op = _optomech_ops(p)
    d = p["Nc"] * p["Nm"]
    rho0 = np.zeros((d, d), complex)
    rho0[0, 0] = 1.0
    tl = workloads.tlist(p["t_end"], p["nt"])
    coef = {"kind": "cos", "a": p["F"], "omega": p["wd"]}
    out = {"Nc": p["Nc"], "Nm": p["Nm"], "n": d * d, "t_end": p["t_end"], "n_t": p["nt"]}
    res = {}
    for name, prec in [("fp64", qt.F64), ("mixed", qt.MIXED)]:
        L = qt.Liouvillian(ctx, H0, c_ops, qt.FORM_CSR, prec, h_terms=[(xa, coef)])
        plan = qt.MePlan(ctx, [(L, rho0, tl, [n_op])], qt.opts(precision=prec, autotune=True))
        plan.run()
        t0 = time.perf_counter()
        plan.run()
        dt = time.perf_counter() - t0
        ex, st, _ = plan.result(0)
        res[name] = ex[0]
        out[name] = {"seconds": dt, "n_accept": st["n_accept"], "n_reject": st["n_reject"], "n_rhs": st["n_rhs"],
                     "rhs_per_s": st["n_rhs"] / dt, "nnz": L.info()[1], "csr_shape": list(plan.shape()[:4]),
                     "n_final": float(ex[0, -1].real)}
        plan.close()
        L.close()
    out["mixed_vs_fp64_max_abs"] = float(np.abs(res["mixed"] - res["fp64"]).max())
    ref = load_golden("optomech_full")[0]
    for name in ("fp64", "mixed"):
        out[name]["max_err_vs_fp64_oracle"] = float(np.abs(res[name] - ref).max())
    sweep = workloads.optomech_sweep(n=n_sweep)
    probs, Ls = [], []
    for q in sweep:
        Hq, xq, cq, nq = _optomech_ops(q)
        Lq = qt.Liouvillian(ctx, Hq, cq, qt.FORM_CSR, qt.MIXED,
                            h_terms=[(xq, {"kind": "cos", "a": q["F"], "omega": q["wd"]})])
        Ls.append(Lq)
        probs.append((Lq, rho0, workloads.tlist(q["t_end"], q["nt"]), [nq]))
    plan = qt.MePlan(ctx, probs, qt.opts(precision=qt.MIXED, autotune=True))
    plan.run()
    t0 = time.perf_counter()
    plan.run()
    dt = time.perf_counter() - t0
    rhs = sum(plan.result(i)[1]["n_rhs"] for i in range(len(probs)))
    out["sweep"] = {"instances": len(probs), "t_end": sweep[0]["t_end"], "seconds": dt,
                    "solves_per_s": len(probs) / dt, "rhs_per_s": rhs / dt, "csr_shape": list(plan.shape()[:4])}
    plan.close()
    for Lq in Ls:
        Lq.close()
    log(f"td: {out}")
    return out


def section_sde(ctx):
    """Stochastic Schrodinger and master equations under homodyne detection: the Jaynes-Cummings
    example (d = 40; SME n = 1,600), 500 trajectories, fixed step 1e-3 over t in [0, 2 pi]."""
    import scipy.sparse as sp
    from math import factorial
    p = workloads.jc_homodyne()
    N = p["N"]
    dst = sp.diags(np.sqrt(np.arange(1, N, dtype=float)), 1, shape=(N, N), format="csr").astype(complex)
    sm2 = sp.csr_matrix(np.array([[0, 0], [1, 0]], dtype=complex))
    sz2 = sp.csr_matrix(np.array([[1, 0], [0, -1]], dtype=complex))
    a = sp.kron(dst, sp.identity(2), format="csr")
    sm = sp.kron(sp.identity(N), sm2, format="csr")
    sz = sp.kron(sp.identity(N), sz2, format="csr")
    ad = a.conj().T
    H = (p["wc"] * (ad @ a) + 0.5 * p["wq"] * sz + p["g"] * (ad @ sm + a @ sm.conj().T)).tocsr()
    S = [np.sqrt(p["kappa"]) * a]
    X = (np.sqrt(p["kappa"]) * (a + ad)).tocsr()
    coh = np.array([np.exp(-p["alpha"] ** 2 / 2) * p["alpha"] ** n / np.sqrt(float(factorial(n))) for n in range(N)])
    psi0 = np.kron(coh, np.array([1.0, 0.0])).astype(complex)
    tl = workloads.tlist(p["t_end"], p["nt"])
    out = {"d": 2 * N, "ntraj": p["ntraj"], "dt": p["dt"], "t_end": p["t_end"], "n_t": p["nt"]}
    with open(os.path.join(ROOT, "tests", "golden", "jc_homodyne_traj.json")) as f:
        gold = json.load(f)
    means = {}
    C = [np.sqrt(p["gamma"]) * sm, (np.sqrt(p["kappa_phi"]) * (ad @ a)).tocsr()]
    for name, master, cops in [("sse", False, []), ("sme", True, C)]:
        for pname, prec in [("mixed", qt.MIXED), ("fp64", qt.F64)]:
            P = qt.SdePlan(ctx, H, S, psi0, tl, [X], p["ntraj"], p["seed"], p["dt"], c_ops=cops, master=master,
                           options=qt.opts(precision=prec))
            P.run()
            t0 = time.perf_counter()
            P.run()
            dt_ = time.perf_counter() - t0
            r = P.result(want_traj=(prec == qt.F64))
            if prec == qt.F64:
                g = gold[name]
                k = len(g["expect_re"])
                out[f"{name}_fp64_vs_oracle_first{k}"] = {
                    "expect_max_abs": float(np.abs(r["expect_tr"][:k] - (np.array(g["expect_re"]) + 1j * np.array(g["expect_im"]))).max()),
                    "current_max_abs": float(np.abs(r["measurement"][:k] - np.array(g["measurement"])).max())}
            out[f"{name}_{pname}"] = {"seconds": dt_, "trajectories_per_s": p["ntraj"] / dt_,
                                      "steps_per_s": r["stats"]["n_accept"] / dt_,
                                      "X_mean_final": float(r["mean"][0, -1].real),
                                      "J_mean_last_interval": float(r["measurement_mean"][0, -1])}
            means[(name, pname)] = r["mean"][0]
            P.close()
        out[f"{name}_mixed_vs_fp64_ensemble_max_abs"] = float(np.abs(means[(name, "mixed")] - means[(name, "fp64")]).max())
    log(f"sde: {out}")
    return out


def section_sesolve(ctx):
    """Schrodinger evolution of the closed L = 10 transverse-field chain (d = 1,024, J = 1, h = 1,
    all spins up, t in [0, 10], <sum sigma_z> at 100 times): one trajectory of the jump kernel with
    no collapse operators.  FP64 at the default tolerances; mixed at the loosest ladder rtol whose
    solution is within 1e-4 of the stored tight FP64 oracle solution."""
    p = workloads.ising_mc()
    H, _ = qt.model_ising(p["L"], p["J"], p["h"], p["gamma"])
    tl = workloads.tlist(p["t_end"], p["nt"])
    Sz = sum(sz_ops(p["L"]))
    ref = load_golden("sesolve_l10_tight")[0]
    out = {"L": p["L"], "d": 2 ** p["L"], "n_t": p["nt"], "t_end": p["t_end"]}
    rungs, chosen = [], None
    for rt in LADDER:
        o = qt.opts(abstol=rt / 100, reltol=rt, precision=qt.MIXED)
        ex, _ = qt.sesolve(ctx, H, up_ket(p["L"]), tl, [Sz], options=o)
        err = float(np.abs(ex[0] - ref).max())
        rungs.append({"rtol": rt, "max_err": err})
        if err <= 1e-4:
            chosen = o
            break
    out["mixed_calibration"] = rungs
    for name, o in [("fp64", qt.opts(precision=qt.F64)),
                    ("mixed", chosen or qt.opts(abstol=1e-8, reltol=1e-6, precision=qt.MIXED))]:
        qt.sesolve(ctx, H, up_ket(p["L"]), tl, [Sz], options=o)
        t0 = time.perf_counter()
        ex, st = qt.sesolve(ctx, H, up_ket(p["L"]), tl, [Sz], options=o)
        dt = time.perf_counter() - t0
        out[name] = {"seconds": dt, "n_accept": st["n_accept"], "n_rhs": st["n_rhs"], "rhs_per_s": st["n_rhs"] / dt,
                     "rtol": o.reltol, "atol": o.abstol, "sz_final": float(ex[0, -1].real),
                     "max_err_vs_tight_fp64_oracle": float(np.abs(ex[0] - ref).max())}
    log(f"sesolve: {out}")
    return out


def section_steady(ctx, n_kerr=64):
    """Steady states by relaxation (integrate until |L rho|_2 <= tol), FP64: the first n_kerr
    cavities with N <= 48 (the FP64 dense form's limit) of the 512-cavity sweep as one dense-form
    plan, and the L = 8 dissipative chain on the CSR form, both at tol 1e-6.  The residual of the
    integrated state settles near |L|_2 * atol * sqrt(n) (n = d^2), so atol sits well below
    tol / (|L|_2 sqrt(n)): |L|_2 is about 2.3e3 for the largest cavities and about 30 for the chain."""
    out = {}
    sweep = [p for p in workloads.kerr_sweep() if p["N"] <= 48][:n_kerr]
    probs = []
    for p in sweep:
        H, c = qt.model_kerr(p["N"], p["delta"], p["U"], p["F"], p["kappa"])
        Lo = qt.Liouvillian(ctx, H, c, qt.FORM_DENSE, qt.F64)
        rho0 = np.zeros((p["N"], p["N"]), complex)
        rho0[0, 0] = 1
        num = np.diag(np.arange(p["N"], dtype=float)).astype(complex)
        probs.append((Lo, rho0, np.array([0.0, 1000.0]), [num]))
    o = qt.opts(abstol=1e-13, reltol=1e-11, precision=qt.F64)
    plan = qt.MePlan(ctx, probs, o, steady_tol=1e-6)
    plan.run()
    t0 = time.perf_counter()
    plan.run()
    dt = time.perf_counter() - t0
    sts = [plan.result(i, check=False)[1] for i in range(n_kerr)]
    out["kerr_dense"] = {"instances": n_kerr, "N_max": max(p["N"] for p in sweep), "tol": 1e-6, "atol": o.abstol, "rtol": o.reltol, "seconds": dt,
                         "solves_per_s": n_kerr / dt, "rhs_per_s": sum(s["n_rhs"] for s in sts) / dt,
                         "steps_max": max(s["n_accept"] + s["n_reject"] for s in sts),
                         "converged": sum(1 for s in sts if s["status"] == 0)}
    plan.close()
    p = workloads.ising_single()
    H, cs = qt.model_ising(p["L"], p["J"], p["h"], p["gamma"])
    Lo = qt.Liouvillian(ctx, H, cs, qt.FORM_CSR, qt.F64)
    o = qt.opts(abstol=1e-12, reltol=1e-10, precision=qt.F64)
    qt.steadystate(ctx, Lo, up_ket(p["L"]), sz_ops(p["L"]), tol=1e-6, t_max=500.0, options=o)
    t0 = time.perf_counter()
    ex, st, _ = qt.steadystate(ctx, Lo, up_ket(p["L"]), sz_ops(p["L"]), tol=1e-6, t_max=500.0, options=o)
    dt = time.perf_counter() - t0
    out["ising_L8_csr"] = {"tol": 1e-6, "atol": o.abstol, "rtol": o.reltol, "seconds": dt, "n_accept": st["n_accept"],
                           "n_rhs": st["n_rhs"], "rhs_per_s": st["n_rhs"] / dt,
                           "sz_site1": float(ex[0].real)}
    Lo.close()
    log(f"steady: {out}")
    return out


def copy_calibration(mbytes):
    """One device-to-device copy of a known size (the HIP runtime's copy kernel), so that hardware
    traffic counters collected on this run can be scaled to bytes."""
    import ctypes
    rt = ctypes.CDLL("/opt/rocm/lib/libamdhip64.so")
    n = int(mbytes) << 20
    a, b = ctypes.c_void_p(), ctypes.c_void_p()
    assert rt.hipMalloc(ctypes.byref(a), ctypes.c_size_t(n)) == 0
    assert rt.hipMalloc(ctypes.byref(b), ctypes.c_size_t(n)) == 0
    assert rt.hipMemset(a, 1, ctypes.c_size_t(n)) == 0
    assert rt.hipMemcpy(b, a, ctypes.c_size_t(n), 3) == 0  # device to device
    assert rt.hipDeviceSynchronize() == 0
    rt.hipFree(a)
    rt.hipFree(b)
    log(f"copy calibration: {n} bytes device to device")


def kernel_source_digest():
    import hashlib
    src = os.path.join(ROOT, "paper_2504_21440_amd", "csrc")
    h = hashlib.sha256()
    for f in ("kernels_csr.hip", "csr_kernels.h", "qt_coef.h", "qt_csr.h", "qt_common.h"):
        with open(os.path.join(src, f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def profiled_traffic(kernel):
    """HBM-side bytes per dispatch of `kernel` from the committed counter summary, or None when the
    summary does not cover it or the kernel sources have changed since the counters were taken."""
    path = os.path.join(ROOT, "profiles", "k_csr_stage_L8.traffic.txt")
    if not os.path.exists(path):
        return None
    digest, table = None, {}
    with open(path) as f:
        for line in f:
            parts = line.split()
            if line.startswith("source_sha256_16:"):
                digest = parts[1]
            elif len(parts) == 5 and parts[1].startswith("k_csr_stage<"):
                table[parts[1]] = int(parts[4])
    if digest != kernel_source_digest():
        return None
    return table.get(kernel)


def _cpu_leg(name, budget):
    """One bounded timing of the FP64 oracle, run in a child process whose OMP_NUM_THREADS sets its
    threads (OpenMP over rows for single solves, over trajectories for ensembles).  Prints one JSON
    object."""
    import oracle
    from oracle import models as om
    oracle._load()

    def until(budget, items):
        t0, n, rhs, used = time.perf_counter(), 0, 0, []
        for it, fn in items:
            if n and time.perf_counter() - t0 >= budget:
                break
            r = fn()
            n += 1
            rhs += r
            used.append(it)
        return n, rhs, time.perf_counter() - t0, used

    def me(H, cs, rho0, tl, e):
        return lambda: oracle.mesolve(H, cs, rho0, tl, e)[1]["n_rhs"]

    if name == "kerr_n20":
        p = workloads.kerr_single()
        H, cs = om.kerr(p["N"], p["delta"], p["U"], p["F"], p["kappa"])
        f = me(H, cs, om.fock_dm(p["N"], 0), workloads.tlist(p["t_end"], p["nt"]), [om.number(p["N"])])
        n, rhs, dt, _ = until(budget, ((k, f) for k in range(10 ** 6)))
        r = {"unit": "solves/s", "value": n / dt, "rhs_per_s": rhs / dt, "seconds": dt, "sample": f"{n} full solves"}
    elif name in ("ising_l8", "ising_l8_window"):
        p = workloads.ising_single()
        H, cs = om.ising(p["L"], p["J"], p["h"], p["gamma"])
        e = [om.site_op(p["L"], i, om.sigmaz()) for i in range(p["L"])]
        tl = workloads.tlist(p["t_end"], p["nt"]) if name == "ising_l8" else np.linspace(0.0, 1.0, 11)
        f = me(H, cs, om.all_up_ket(p["L"]), tl, e)
        n, rhs, dt, _ = until(budget, ((k, f) for k in range(10 ** 6)))
        r = {"unit": "RHS evals/s", "value": rhs / dt, "solves": n, "rhs": rhs, "seconds": dt,
             "sample": f"{n} solves over t in [0, {tl[-1]:g}] ({rhs} RHS)"}
    elif name == "mc_l10":
        p = workloads.ising_mc()
        H, cs = om.ising(p["L"], p["J"], p["h"], p["gamma"])
        Sz = sum(om.site_op(p["L"], i, om.sigmaz()) for i in range(p["L"]))
        tl = workloads.tlist(p["t_end"], p["nt"])
        k = 4 * int(os.environ.get("OMP_NUM_THREADS", "1"))
        batches = ((b, (lambda b=b: int(oracle.mcsolve(H, cs, om.all_up_ket(p["L"]), tl, [Sz], k, p["seed"],
                                                         traj0=b * k, abstol=1e-6, reltol=1e-4)["njumps"].size)))
                   for b in range(10 ** 6))
        n, ntr, dt, _ = until(budget, batches)
        r = {"unit": "trajectories/s", "value": ntr / dt, "seconds": dt,
             "sample": f"{ntr} trajectories (mcsolve, rtol 1e-4)"}
    elif name in ("sweep", "serving"):
        items = workloads.kerr_sweep() if name == "sweep" else workloads.serving_trace(n=240)
        small = [q for q in items if (q["kind"] == "kerr" and q["N"] <= 40) or (q["kind"] == "ising" and q["L"] <= 6)]

        def solve(q):
            tl = workloads.tlist(q["t_end"], q["nt"])
            if q["kind"] == "kerr":
                H, cs = om.kerr(q["N"], q["delta"], q["U"], q["F"], q["kappa"])
                return me(H, cs, om.fock_dm(q["N"], 0), tl, [om.number(q["N"])])
            H, cs = om.ising(q["L"], q["J"], q["h"], q["gamma"])
            return me(H, cs, om.all_up_ket(q["L"]), tl, [om.site_op(q["L"], 0, om.sigmaz())])

        n, rhs, dt, used = until(budget, ((q, solve(q)) for q in small))
        sizes = [q.get("N", q.get("L")) for q in used]
        r = {"unit": "solves/s", "value": n / dt, "rhs_per_s": rhs / dt, "seconds": dt,
             "sample": f"{n} full solves of the first {'cavities' if name == 'sweep' else 'requests'} with "
                       f"N <= 40 / L <= 6 in order (sizes {sizes}); larger ones cost more per solve"}
    else:
        raise SystemExit(f"unknown cpu leg {name}")
    print(json.dumps(r), flush=True)


def _host_info():
    model = ""
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    return {"nproc": len(os.sched_getaffinity(0)), "cpu_model": model}


def _run_leg(name, threads, budget):
    import subprocess
    env = dict(os.environ, OMP_NUM_THREADS=str(threads))
    r = subprocess.run([sys.executable, os.path.abspath(__file__), "--cpu-leg", name, "--cpu-budget", str(budget)],
                       env=env, capture_output=True, text=True, check=True)
    out = json.loads(r.stdout.strip().splitlines()[-1])
    out["threads"] = threads
    return out


def cpu_oracle_baseline():
    """The FP64 oracle timed on this host: the headline chain at every thread (the bench line's
    cpu_baseline), and a bounded sample of every other workload at 1 thread and at every thread."""
    host = _host_info()
    nt = host["nproc"]
    head = _run_leg("ising_l8", nt, 10.0)
    legs = {}
    for name, budget in [("kerr_n20", 4.0), ("ising_l8_window", 6.0), ("mc_l10", 5.0), ("sweep", 5.0),
                         ("serving", 5.0)]:
        legs[name] = {f"{t}_threads": _run_leg(name, t, budget) for t in sorted({1, nt})}
        log(f"cpu oracle {name}: {legs[name]}")
    return {"value": head["value"], "unit": "RHS evals/s", "cores": nt, "kind": "oracle",
            "sample": head["sample"] + " of the L=8 chain (abstol 1e-8, reltol 1e-6, OpenMP over rows)",
            "seconds": head["seconds"], "host": host, "other_workloads": legs}


def copy_bandwidth(ctx, mbytes=2048, reps=20):
    """Achievable HBM bandwidth: the library's streaming copy kernel and the runtime's device-to-device
    copy (hipMemcpy) over mbytes MiB, timed with HIP events (bytes read plus bytes written per
    second)."""
    import ctypes
    rt = ctypes.CDLL("/opt/rocm/lib/libamdhip64.so")
    n = int(mbytes) << 20
    a, b, e0, e1 = ctypes.c_void_p(), ctypes.c_void_p(), ctypes.c_void_p(), ctypes.c_void_p()
    assert rt.hipMalloc(ctypes.byref(a), ctypes.c_size_t(n)) == 0
    assert rt.hipMalloc(ctypes.byref(b), ctypes.c_size_t(n)) == 0
    assert rt.hipMemset(a, 1, ctypes.c_size_t(n)) == 0
    assert rt.hipEventCreate(ctypes.byref(e0)) == 0 and rt.hipEventCreate(ctypes.byref(e1)) == 0
    assert rt.hipMemcpyAsync(b, a, ctypes.c_size_t(n), 3, None) == 0
    assert rt.hipEventRecord(e0, None) == 0
    for _ in range(reps):
        assert rt.hipMemcpyAsync(b, a, ctypes.c_size_t(n), 3, None) == 0
    assert rt.hipEventRecord(e1, None) == 0
    assert rt.hipEventSynchronize(e1) == 0
    ms = ctypes.c_float()
    assert rt.hipEventElapsedTime(ctypes.byref(ms), e0, e1) == 0
    rt.hipEventDestroy(e0)
    rt.hipEventDestroy(e1)
    rt.hipFree(a)
    rt.hipFree(b)
    gbs = 2.0 * n * reps / (ms.value * 1e-3) / 1e9
    kern = qt.measure_copy_bandwidth(ctx, n, reps)
    rd = qt.measure_read_bandwidth(ctx, n, reps)
    log(f"copy bandwidth: hipMemcpy {gbs:.0f} GB/s, streaming copy kernel {kern:.0f} GB/s, streaming read kernel "
        f"{rd:.0f} GB/s ({mbytes} MiB)")
    return {"GBs": kern, "kernel": "k_stream_copy (16-byte non-temporal loads and stores, 4 in flight per lane)",
            "hipMemcpy_GBs": gbs, "bytes_per_copy": n, "copies": reps, "frac_of_hbm_peak": kern / HBM_PEAK_GBS,
            "read_GBs": rd, "read_kernel": "k_stream_read (16-byte non-temporal loads, 4 in flight per lane)",
            "read_frac_of_hbm_peak": rd / HBM_PEAK_GBS}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--skip-extra", action="store_true")
    ap.add_argument("--only", default="",
                    help="comma list of extra sections: hbm,sweep,mc,serving,td,sde,sesolve,steady")
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--sweep-forms", default="dense,stiff0.6",
                    help="form policies of the 512-cavity sweep, one run each: dense (all dense), n<K> (dense up "
                         "to N = K, CSR above), stiff<f> (CSR for cavities whose estimated dense cost is at least "
                         "f times the largest)")
    ap.add_argument("--tune-in", default=os.path.join(ROOT, "paper_2504_21440_amd", "tuning", "mi355x.json"),
                    help="autotuner table loaded before measuring (size buckets it lacks are tuned live); "
                         "'' for none")
    ap.add_argument("--tune-out", default="", help="save the autotuner table after measuring")
    ap.add_argument("--copy-calib-mb", type=int, default=0,
                    help="also run one device-to-device copy of this many MiB (counter calibration)")
    ap.add_argument("--cpu-leg", default="", help=argparse.SUPPRESS)
    ap.add_argument("--cpu-budget", type=float, default=5.0, help=argparse.SUPPRESS)
    args = ap.parse_args()
    if args.cpu_leg:  # child process of the CPU baseline: the oracle only, no GPU
        _cpu_leg(args.cpu_leg, args.cpu_budget)
        return
    if args.gpus != 1:
        print("bench.py measures one GPU only: the library has no multi-GPU path (trajectories, sweep "
              "instances and served requests would shard by count across GPUs with one final FP64 "
              "all-reduce)", file=sys.stderr)
        sys.exit(2)
    if args.tune_in and os.path.exists(args.tune_in):
        qt.tune_load(args.tune_in)
    log("context")
    ctx = qt.Context(0)
    ising = section_ising(ctx, args.steps, args.warmup)
    copy = copy_bandwidth(ctx)
    mixed = ising["mixed"]
    log("ising batch")
    batch = section_ising_batch(ctx, mixed["rtol"], max(1, args.steps // 2), 1)
    extra = {}
    only = set(args.only.split(",")) if args.only else {"kerr", "hbm", "sweep", "mc", "serving", "td", "sde", "sesolve",
                                                       "steady"}
    if args.skip_extra:
        only = set()
    if "kerr" in only:
        log("kerr N=20 FP64")
        extra["kerr_n20_fp64"] = section_kerr_single(ctx)
    if "hbm" in only:
        log("hbm spmv")
        extra["spmv_hbm_L10"] = section_hbm_spmv(ctx)
        for v in extra["spmv_hbm_L10"].values():  # against what a pure streaming read reaches
            v["frac_of_measured_read"] = v["GBs"] / copy["read_GBs"]
    if "sweep" in only:
        log("sweep")
        for pol in [x for x in args.sweep_forms.split(",") if x]:
            key = "kerr_sweep_512" if pol == "dense" else f"kerr_sweep_512_{pol}"
            extra[key], _, _ = section_sweep(ctx, policy=pol)
    if "mc" in only:
        log("mc")
        extra["mcsolve_L10_10k"] = section_mc(ctx)
    if "serving" in only:
        log("serving")
        extra["serving"] = section_serving(ctx)
    if "td" in only:
        log("time-dependent")
        extra["td_optomechanics"] = section_td(ctx)
    if "sde" in only:
        log("stochastic")
        extra["homodyne_jc"] = section_sde(ctx)
    if "sesolve" in only:
        log("sesolve")
        extra["sesolve_L10"] = section_sesolve(ctx)
    if "steady" in only:
        log("steady states")
        extra["steadystate"] = section_steady(ctx)
    # kernel FORM of a single-problem plan: 1 streamed, 2 cached, 4 cached with 16-byte loads
    kname = "k_csr_stage<float,%d,%d,%d,3,false>" % (mixed["csr_shape"][0], mixed["csr_shape"][1],
                                                     (1, 2, 4)[mixed["csr_shape"][3]])
    matrix = {"bound": "hbm", "achieved": mixed["stage_kernel_GBs"], "peak": HBM_PEAK_GBS, "unit": "GB/s",
              "frac": mixed["stage_kernel_GBs"] / HBM_PEAK_GBS, "traffic": profiled_traffic(kname),
              "kernel": kname + " (fused SpMV + stage epilogue), L=8 Liouvillian, one launch = one SpMV",
              "algorithmic_bytes": mixed["spmv_bytes"],
              "regime": "timed alone: the solve applies the operators (k_op) instead; the 16 MB matrix stays in the "
                        "256 MB MALL between launches, so this launch is bound by latency, not HBM; the HBM "
                        "evidence is spmv_hbm_L10"}
    # the solve's own right-hand side: 8 flops per entry of the superoperator it stands for, over the whole solve
    tf = 8.0 * mixed["nnz"] * mixed["rhs_per_s"] / 1e12
    rl = {"bound": "latency", "achieved": tf, "peak": FP32_VECTOR_PEAK_TFLOPS, "unit": "TFLOP/s",
          "frac": tf / FP32_VECTOR_PEAK_TFLOPS,
          "kernel": "k_op<float,true,true,false,OP_SHORT> (operator form, upper triangle), L=8 chain, one launch = one stage",
          "regime": "us_per_rhs over the whole solve, launches and step control included; a stage is one launch of "
                    "160 workgroups, bound by the latency of a wave",
          "us_per_rhs": 1e6 / mixed["rhs_per_s"], "matrix_stage_kernel": matrix,
          "measured_copy_GBs": copy["GBs"], "measured_read_GBs": copy["read_GBs"]}
    line = {
        "metric": METRIC, "value": mixed["rhs_per_s"], "unit": "RHS evals/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": mixed["ms_per_solve"], "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "c64", "data": "synthetic",
        "config": {"workload": "dissipative TFIM chain L=8 mesolve, mixed precision, accuracy-matched to 1e-4",
                   "L": 8, "d": 256, "n": mixed["n"], "nnz": mixed["nnz"], "t_end": 10.0, "n_t": 100,
                   "rtol": mixed["rtol"], "atol": mixed["atol"], "parallelism": "single GPU"},
        "solves_per_s": mixed["solves_per_s"], "max_err_vs_fp64": mixed["max_err_vs_tight_fp64"],
        "fp64_single_solve": ising["fp64"], "mixed_detail": mixed,
        "mixed_batched_16xL8": batch,
        "batched_vs_fp64_single_solves_per_s": batch["solves_per_s"] / ising["fp64"]["solves_per_s"],
        "roofline": rl, "copy_bandwidth": copy,
    }
    line.update(extra)
    if args.tune_out:
        qt.tune_save(args.tune_out)
    if args.copy_calib_mb:
        copy_calibration(args.copy_calib_mb)
    if not args.no_cpu:
        log("cpu oracle baseline")
        line["cpu_baseline"] = cpu_oracle_baseline()
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
