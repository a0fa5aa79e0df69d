"""Workloads of the library as its users run them: what is prepared once, one pass, and its reference.

A case is a dict of plain values.  ``listed()`` names the standing ones, ``draw(rng)`` gives one more
of the same ranges.  ``prepare`` builds what a program holds before the call (operators, Liouvillian,
plan or server), ``run`` makes one pass through the public entry points and returns its outputs,
``exact`` computes the same outputs in 64 bits with torch and numpy alone.

Families:
  * ``me``: one master-equation problem in the CSR form (driven Kerr cavity or Ising chain), solved
    one-shot (``qt.mesolve``, planning included) or through a plan that is kept;
  * ``batch``: many problems in one plan, CSR or dense form;
  * ``td``: a driven optomechanical system (time-dependent Liouvillian);
  * ``se``: the Schroedinger equation; ``mc``: a quantum-jump ensemble; ``sde``: homodyne detection;
  * ``serve``: a burst of mixed requests through the continuous-batching server.

Mixed precision keeps the states and stages in complex64; its outputs are kept in 32 bits here too, and
only the recorded values are asked for (what the mode is for).  FP64 solves of the chain and of the
time-dependent system return the final state too; a cavity's stiff elements sit at the level its
error control admits, so cavities are asked for their recorded values.
"""
import math
import os

import numpy as np
import torch

import paper_2504_21440_amd as qt

_TABLE = os.path.join(os.path.dirname(os.path.abspath(qt.__file__)), "tuning", "mi355x.json")
_held = {}


def _context():
    """One context per process with the shipped tuning table, as a program would hold it."""
    if "ctx" not in _held:
        qt.tune_load(_TABLE)
        _held["ctx"] = qt.Context(0)
    return _held["ctx"]


# ---- the cases ------------------------------------------------------------------------------------
def listed():
    return [
        # the smallest calls: a lone small chain and the N = 20 cavity at the default tolerances,
        # solved one-shot, where launches, planning and latency are all there is
        dict(name="ising5_mixed_once", family="me", model="ising", size=5, precision="mixed", rtol=1e-5,
             t_end=10.0, nt=100, once=True),
        dict(name="kerr20_f64_once", family="me", model="kerr", size=20, precision="f64", rtol=1e-6, t_end=20.0,
             nt=200, once=True),
        # the ordinary single solve: the L = 8 chain of the benchmark line, in both precisions
        dict(name="ising8_mixed", family="me", model="ising", size=8, precision="mixed", rtol=1e-4, t_end=10.0,
             nt=100, once=False),
        # a parameter scan: 16 chains that differ in their fields, advanced together
        dict(name="ising8_batch16", family="batch", model="ising", form="csr", n=16, size_min=8, size_max=8,
             precision="mixed", rtol=1e-4, t_end=5.0, nt=50),
        # the largest Liouvillian: the L = 10 chain, whose matrix is sized for HBM
        dict(name="ising10_f64", family="me", model="ising", size=10, precision="f64", rtol=1e-6, t_end=2.0, nt=21,
             once=False),
        # parameter sweeps of cavities of many sizes in the dense form
        dict(name="kerr_sweep_dense", family="batch", model="kerr", form="dense", n=64, size_min=10, size_max=80,
             precision="mixed", rtol=1e-5, t_end=1.0, nt=21),
        dict(name="kerr_dense_f64", family="batch", model="kerr", form="dense", n=24, size_min=9, size_max=48,
             precision="f64", rtol=1e-6, t_end=4.0, nt=41),
        # the time-dependent example
        dict(name="optomech_f64", family="td", n=1, nc=10, nm=7, precision="f64", rtol=1e-6, t_end=60.0, nt=601),
        # quantum-jump and homodyne ensembles, the closed chain
        dict(name="mc_ising10", family="mc", model="ising", size=10, precision="mixed", rtol=1e-4, ntraj=10000,
             t_end=5.0, nt=51),
        dict(name="sme_jc20", family="sde", size=20, master=True, precision="mixed", ntraj=500, dt=1e-3, t_end=2.0,
             nt=128),
        dict(name="sesolve10_f64", family="se", size=10, precision="f64", rtol=1e-6, t_end=10.0, nt=100),
        # served traffic: 70% cavities, 30% chains, assembled when they are submitted
        dict(name="serve40", family="serve", n=40, precision="mixed", rtol=1e-5, t_end=4.0, nt=41),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    f = rng.choice(["me", "me", "me", "batch", "batch", "batch", "td", "mc", "mc", "sde", "se", "serve"])
    prec = rng.choice(["f64", "mixed"])
    rtol = rng.choice([1e-4, 1e-5, 1e-6]) if prec == "mixed" else 1e-6
    nt = rng.randint(2, 200)
    if f == "me":
        once = rng.random() < 0.5
        if rng.random() < 0.5:
            n = _log_int(rng, 5, 64)
            return dict(family=f, model="kerr", size=n, precision=prec, rtol=rtol, once=once, nt=nt,
                        t_end=round(rng.uniform(0.2, 1.0) * min(20.0, 4000.0 / n ** 2 + 1.0), 3))
        size = rng.randint(2, 10)
        return dict(family=f, model="ising", size=size, precision=prec, rtol=rtol, once=once and size < 10, nt=nt,
                    t_end=round(rng.uniform(0.2, 1.0) * (10.0 if size < 9 else 5.0 if size < 10 else 2.0), 3))
    if f == "batch":
        form = rng.choice(["dense", "dense", "csr"])
        if form == "csr" and rng.random() < 0.5:
            lo = rng.randint(3, 7)
            return dict(family=f, model="ising", form=form, n=_log_int(rng, 2, 24), size_min=lo,
                        size_max=min(8, lo + rng.randint(0, 3)), precision=prec, rtol=rtol, nt=nt,
                        t_end=round(rng.uniform(1.0, 5.0), 3))
        lo = rng.randint(4, 30)
        hi = min(lo + rng.randint(0, 50), 48 if prec == "f64" else 80)
        return dict(family=f, model="kerr", form=form, n=_log_int(rng, 2, 64), size_min=lo, size_max=max(lo, hi),
                    precision=prec, rtol=min(rtol, 1e-5), nt=min(nt, 60), t_end=round(rng.uniform(0.2, 1.0), 3))
    if f == "td":
        return dict(family=f, n=rng.choice([1, 1, 8]), nc=rng.randint(3, 10), nm=rng.randint(2, 7), precision=prec,
                    rtol=min(rtol, 1e-5), nt=2 * nt, t_end=round(rng.uniform(5.0, 50.0), 3))
    if f == "mc":
        if rng.random() < 0.5:
            return dict(family=f, model="kerr", size=_log_int(rng, 5, 60), precision=prec, rtol=rtol,
                        ntraj=_log_int(rng, 20, 2000), t_end=round(rng.uniform(0.5, 2.0), 3), nt=min(nt, 100))
        return dict(family=f, model="ising", size=rng.randint(3, 10), precision=prec, rtol=rtol,
                    ntraj=_log_int(rng, 20, 4000), t_end=round(rng.uniform(1.0, 5.0), 3), nt=min(nt, 100))
    if f == "sde":
        return dict(family=f, size=rng.randint(4, 24), master=rng.random() < 0.6, precision=prec,
                    ntraj=_log_int(rng, 20, 500), dt=1e-3, t_end=round(rng.uniform(0.2, 1.5), 3), nt=min(nt, 100))
    if f == "se":
        return dict(family=f, size=rng.randint(3, 11), precision=prec, rtol=rtol, nt=nt,
                    t_end=round(rng.uniform(1.0, 10.0), 3))
    return dict(family=f, n=rng.randint(4, 32), precision=prec, rtol=min(rtol, 1e-5), nt=min(nt, 60),
                t_end=round(rng.uniform(1.0, 3.0), 3))


# ---- parameters and operators -------------------------------------------------------------------------
def _prec(case):
    return qt.F64 if case["precision"] == "f64" else qt.MIXED


def _final(case):
    return case["precision"] == "f64" and (case["family"] == "td" or
                                           (case["family"] == "me" and case["model"] == "ising"))


def _opts(case):
    rtol = case.get("rtol", 1e-6)
    return qt.opts(abstol=rtol / 100, reltol=rtol, precision=_prec(case))


def _kerr(g, N, wide):
    if wide:  # the sweep's and the request stream's ranges
        p = (g.uniform(-2, 2), g.uniform(0, 1), g.uniform(0, 2), g.uniform(0.5, 2))
    else:
        p = (g.uniform(0.9, 1.1), g.uniform(0.45, 0.55), g.uniform(0.7, 0.9), g.uniform(0.9, 1.1))
    return dict(kind="kerr", N=int(N), delta=float(p[0]), U=float(p[1]), F=float(p[2]), kappa=float(p[3]))


def _ising(g, L, wide=False):
    return dict(kind="ising", L=int(L), J=1.0, h=float(g.uniform(0.3, 1.5) if wide else g.uniform(0.6, 0.8)),
                gamma=float(g.uniform(0.05, 0.5) if wide else g.uniform(0.15, 0.25)))


def _sizes(case):
    lo, hi, n = case["size_min"], case["size_max"], case["n"]
    return [int(round(lo + (hi - lo) * (k / (n - 1) if n > 1 else 1.0))) for k in range(n)]


def _params(case, seed):
    """The parameter records of a case's problems."""
    g = np.random.default_rng([int(seed), 17])
    f = case["family"]
    if f in ("me", "mc", "se"):
        m = case.get("model", "ising")
        return [_kerr(g, case["size"], False) if m == "kerr" else _ising(g, case["size"])]
    if f == "batch":
        return [_kerr(g, n, True) if case["model"] == "kerr" else _ising(g, n, True) for n in _sizes(case)]
    if f == "serve":
        return [_kerr(g, 10 + int(70 * ((k * 7) % 10 + g.uniform()) / 10), True) if k % 10 < 7
                else _ising(g, 4 + (k * 5) % 6, True) for k in range(case["n"])]
    if f == "td":
        return [dict(kind="optomech", g=0.05, kappa=0.01, gamma=0.01, F=float(g.uniform(0.08, 0.12)),
                     wd=float(g.uniform(0.8, 1.2))) for _ in range(case["n"])]
    return [dict(kind="jc", g=float(g.uniform(0.08, 0.12)), kappa=float(g.uniform(0.9, 1.1)), gamma=2.0,
                 kappa_phi=0.3, alpha=2.0, seed=int(g.integers(1 << 40)))]


def _operators(p):
    """(H, c_ops) as scipy CSR matrices from the library's model builders."""
    if p["kind"] == "kerr":
        return qt.model_kerr(p["N"], p["delta"], p["U"], p["F"], p["kappa"])
    return qt.model_ising(p["L"], p["J"], p["h"], p["gamma"])


def _diagonal(like, d):
    """Sparse diagonal matrix of the type of `like`."""
    n = len(d)
    return type(like)((np.asarray(d, complex), np.arange(n), np.arange(n + 1)), shape=(n, n))


def _sz(L, i):
    return 1.0 - 2.0 * ((np.arange(2 ** L) >> (L - 1 - i)) & 1)


def _observables(p):
    """Diagonals of the recorded operators: <a^dag a>, or <sigma_z> of every site."""
    return [np.arange(p["N"], dtype=float)] if p["kind"] == "kerr" else [_sz(p["L"], i) for i in range(p["L"])]


def _start(d):
    v = np.zeros(d, complex)
    v[0] = 1.0
    return v


def _tl(case):
    return np.linspace(0.0, case["t_end"], case["nt"])


def _destroy(n):
    return np.diag(np.sqrt(np.arange(1, n, dtype=float)), 1).astype(complex)


def _optomech(case, p):
    a = np.kron(_destroy(case["nc"]), np.eye(case["nm"]))
    b = np.kron(np.eye(case["nc"]), _destroy(case["nm"]))
    x = a + a.T
    H = 1.0 * a.T @ a + 2.0 * b.T @ b + 0.5 * p["g"] * (x @ x) @ (b + b.T)
    return H, x, [math.sqrt(p["kappa"]) * a, math.sqrt(p["gamma"]) * b], a.T @ a


def _jc(case, p):
    N = case["size"]
    a = np.kron(_destroy(N), np.eye(2))
    sm = np.kron(np.eye(N), np.array([[0, 0], [1, 0]], complex))
    sz = np.kron(np.eye(N), np.diag([1.0, -1.0]))
    H = 5.0 * a.T @ a + 2.5 * sz + p["g"] * (a.T @ sm + a @ sm.T)
    S = [math.sqrt(p["kappa"]) * a]
    C = [math.sqrt(p["gamma"]) * sm, math.sqrt(p["kappa_phi"]) * (a.T @ a)] if case["master"] else []
    X = math.sqrt(p["kappa"]) * (a + a.T)
    coh = np.array([math.exp(-p["alpha"] ** 2 / 2) * p["alpha"] ** n / math.sqrt(math.factorial(n)) for n in range(N)])
    psi = np.kron(coh, [1.0, 0.0]).astype(complex)
    return H, S, C, X, psi / np.linalg.norm(psi)


# ---- what a program holds, and one pass -----------------------------------------------------------------
def prepare(case, seed):
    ctx, prec, f = _context(), _prec(case), case["family"]
    ps, tl, o = _params(case, seed), _tl(case), _opts(case)
    s = dict(case=case, ctx=ctx, tl=tl, o=o, keep=[])
    if f in ("me", "batch"):
        form = qt.FORM_DENSE if case.get("form") == "dense" else qt.FORM_CSR
        probs = []
        for p in ps:
            H, cs = _operators(p)
            L = qt.Liouvillian(ctx, H, cs, form, prec)
            s["keep"].append(L)
            probs.append((L, _start(H.shape[0]), tl, [_diagonal(H, v) for v in _observables(p)]))
        s["probs"] = probs
        if not case.get("once"):
            s["plan"] = qt.MePlan(ctx, probs, o)
    elif f == "td":
        probs = []
        for p in ps:
            H, x, cs, n = _optomech(case, p)
            L = qt.Liouvillian(ctx, H, cs, qt.FORM_CSR, prec,
                               h_terms=[(x, {"kind": "cos", "a": p["F"], "omega": p["wd"]})])
            s["keep"].append(L)
            probs.append((L, _start(H.shape[0]), tl, [n]))
        s["probs"], s["plan"] = probs, qt.MePlan(ctx, probs, o)
    elif f == "se":
        H, _ = _operators(ps[0])
        s["args"] = (H, _start(H.shape[0]), tl, [_diagonal(H, sum(_observables(ps[0])))])
    elif f == "mc":
        H, cs = _operators(ps[0])
        obs = _observables(ps[0])
        s["plan"] = qt.McPlan(ctx, H, cs, _start(H.shape[0]), tl, [_diagonal(H, sum(obs))], case["ntraj"],
                              20250430 + int(seed), o)
    elif f == "sde":
        H, S, C, X, psi = _jc(case, ps[0])
        s["plan"] = qt.SdePlan(ctx, H, S, psi, tl, [X], case["ntraj"], ps[0]["seed"], case["dt"], c_ops=C,
                               master=case["master"], options=o)
    else:
        reqs = []
        for p in ps:
            H, cs = _operators(p)
            reqs.append((H, cs, _start(H.shape[0]), [_diagonal(H, _observables(p)[0])]))
        s["reqs"] = reqs
        s["server"] = qt.Server(ctx, pool_bytes=2 << 30, max_slots=256, steps_per_epoch=32, options=o)
    return s


def _kept(s, *outs):
    """Outputs in the precision of the solve."""
    if s["case"]["precision"] == "f64":
        return list(outs)
    return [x.astype(np.complex64 if x.dtype.kind == "c" else np.float32) for x in outs]


def run(s):
    f, final = s["case"]["family"], _final(s["case"])
    if f == "me" and s["case"]["once"]:
        ex, _, rho = qt.mesolve(s["ctx"], *s["probs"][0], options=s["o"], want_final=final)
        return _kept(s, ex, rho) if final else _kept(s, ex)
    if f in ("me", "batch", "td"):
        s["plan"].run()
        got = [s["plan"].result(i, want_final=final) for i in range(len(s["probs"]))]
        outs = [np.concatenate([r[k].ravel() for r in got]) for k in ((0, 2) if final else (0,))]
        return _kept(s, *outs)
    if f == "se":
        ex, _ = qt.sesolve(s["ctx"], *s["args"], options=s["o"])
        return _kept(s, ex)
    if f in ("mc", "sde"):
        s["plan"].run()
        r = s["plan"].result()
        return _kept(s, r["mean"], r["se"]) + (_kept(s, r["measurement_mean"]) if f == "sde" else [])
    form, prec, srv, out, tickets = qt.FORM_CSR, s["o"].precision, s["server"], {}, {}
    waiting = list(range(len(s["reqs"])))
    while waiting or tickets:
        while waiting:
            H, cs, psi, e = s["reqs"][waiting[0]]
            L = qt.Liouvillian(s["ctx"], H, cs, form, prec)
            t = srv.submit(L, psi, s["tl"], e)
            if t is None:
                L.close()
                break
            tickets[t] = (waiting.pop(0), L)
        srv.step()
        for t in list(tickets):
            r = srv.poll(t)
            if r is not None:
                i, L = tickets.pop(t)
                out[i] = r[0][0]
                L.close()
    return _kept(s, np.stack([out[i] for i in range(len(s["reqs"]))]))


# ---- the work a pass cannot do without ---------------------------------------------------------------
def _superop(p, case):
    """(d, entries of the sparse generator, right-hand sides per unit time of an explicit pair)."""
    if p["kind"] == "kerr":
        N, U, F, k = p["N"], p["U"], p["F"], p["kappa"]
        lv = p["delta"] * np.arange(N) + 0.5 * U * np.arange(N) * (np.arange(N) - 1)
        rate = (lv.max() - lv.min()) + k * N + 2 * F * math.sqrt(N)
        return N, 6 * N * N, 6 * max(2.0, rate / 3.3)
    if p["kind"] == "ising":
        L = p["L"]
        return 2 ** L, 4 ** L * (1 + 2 * L + L / 4), 6 * max(4.0, (L - 1 + L * p["h"]) * 0.9)
    d = case["nc"] * case["nm"]
    return d, 15 * d * d, 6 * (case["nc"] + 2.0 * case["nm"])


def work(case):
    ps, f, nt = _params(case, 1), case["family"], case["nt"]
    val = 16 if case["precision"] == "f64" else 8
    nbytes = flops = 0.0
    for p in ps:
        if f in ("mc", "se"):
            d, _, rate = _superop(p, case)
            nnz = d * (1 + (p["L"] if p["kind"] == "ising" else 2))
            n = case.get("ntraj", 1)
            flops += n * 8.0 * nnz * rate * 0.5 * case["t_end"]
            nbytes += 20.0 * nnz + 16.0 * n * nt
        elif f == "sde":
            d = 2 * case["size"]
            rows, nnz = (d * d, 14.0 * d * d) if case["master"] else (d, 6.0 * d)
            flops += case["ntraj"] * case["t_end"] / case["dt"] * 8.0 * nnz
            nbytes += case["ntraj"] * (val * rows + 24.0 * nt)
        else:
            d, nnz, rate = _superop(p, case)
            ne = p["L"] if f in ("me", "batch") and p["kind"] == "ising" else 1
            flops += 8.0 * nnz * rate * case["t_end"]
            nbytes += 2.0 * val * d * d + 20.0 * d * 12 + 16.0 * ne * nt
    return {"bytes": float(nbytes), "flops": float(flops)}


# ---- the same outputs in 64 bits ---------------------------------------------------------------------
_DEV = "cuda" if torch.cuda.is_available() else "cpu"


def _t(x):
    return torch.as_tensor(np.asarray(x), dtype=torch.complex128, device=_DEV)


def _gather(C):
    """Collapse operators [b][d][d] with at most one entry per row, in the same columns: those columns
    [d] and the values [b][d]."""
    k = np.argmax(np.abs(C).sum(axis=0), axis=-1)
    return k, C[:, np.arange(len(k)), k]


def _evolve(Hs, cs, tl, obs, drive=None):
    """Taylor propagation (order 40, steps of |L| h <= 6) of a batch of d x d problems that share their
    size: Hs [b][d][d], cs a list of [b][d][d] with one entry per row and common columns, obs a list of
    [b][d] diagonals, drive (operators [b][d][d], amplitudes [b], frequencies [b]).  Returns the
    expectation values [b][n_obs][n_t] and the final states [b][d][d], from |0><0|."""
    b, d = Hs.shape[:2]
    lam = np.linalg.eigvalsh(Hs)
    mid = 0.5 * (lam[:, 0] + lam[:, -1])
    G = -1j * (Hs - mid[:, None, None] * np.eye(d))
    ops, norm = [], lam[:, -1] - lam[:, 0]
    for C in cs:
        k, v = _gather(C)
        ops.append((torch.as_tensor(k, device=_DEV), _t(v[:, :, None] * v[:, None, :].conj())))
        G = G - 0.5 * C.conj().transpose(0, 2, 1) @ C
        norm = norm + 2.0 * np.abs(v).max(axis=1) ** 2
    if drive is not None:
        norm = norm + 2.0 * drive[1] * np.linalg.norm(drive[0], 2, axis=(1, 2))
    bound, K = float(norm.max()), 40
    G, O = _t(G), torch.stack([_t(o) for o in obs], 1)
    r = torch.zeros(b, d, d, dtype=torch.complex128, device=_DEV)
    r[:, 0, 0] = 1.0
    if drive is not None:
        D = -1j * _t(drive[0])
        amp, om = _t(drive[1])[:, None, None], np.asarray(drive[2])

    def rhs(x):
        p = torch.matmul(G, x)
        p = p + p.conj().transpose(1, 2)
        for k, w in ops:
            p = p + w * x[:, k][:, :, k]
        return p

    ex = [(O * torch.diagonal(r, dim1=1, dim2=2)[:, None]).sum(-1)]
    for q in range(len(tl) - 1):
        dt = float(tl[q + 1] - tl[q])
        n = max(1, math.ceil(dt * bound / 6.0))
        h = dt / n
        for s in range(n):
            term, acc, past = r, r.clone(), [r]
            if drive is not None:
                t0 = tl[q] + s * h
                ph = np.array([(om * h) ** j / math.factorial(j) * np.cos(om * t0 + 0.5 * math.pi * j)
                               for j in range(K)])
                ph = torch.as_tensor(ph, device=_DEV).to(torch.complex128)[:, :, None, None] * amp
            for k in range(1, K + 1):
                nxt = rhs(term)
                if drive is not None:
                    y = sum(ph[j] * past[k - 1 - j] for j in range(min(k, 16)))
                    z = torch.matmul(D, y)
                    nxt = nxt + z + z.conj().transpose(1, 2)
                term = nxt * (h / k)
                acc = acc + term
                if drive is not None:
                    past.append(term)
            r = acc
        ex.append((O * torch.diagonal(r, dim1=1, dim2=2)[:, None]).sum(-1))
    return torch.stack(ex, -1).cpu().numpy(), r.cpu().numpy()


def _exact_me(case, ps):
    """Expectation values and final states of every record, problems of one kind padded and batched."""
    tl, out = _tl(case), {}
    for kind in ("kerr", "ising"):
        ids = [i for i, p in enumerate(ps) if p["kind"] == kind]
        groups = {}
        for i in ids:  # cavities pad to the next multiple of 16, chains group by length
            key = -(-ps[i]["N"] // 16) * 16 if kind == "kerr" else 2 ** ps[i]["L"]
            groups.setdefault(key, []).append(i)
        for d, g in groups.items():
            Hs, C, obs = [], None, None
            for i in g:
                H, cs = _operators(ps[i])
                n = H.shape[0]
                pad = lambda M: np.pad(M.toarray(), (0, d - n))  # noqa: E731
                Hs.append(pad(H))
                C = [[] for _ in cs] if C is None else C
                for k, c in enumerate(cs):
                    C[k].append(pad(c))
                o = [np.pad(v, (0, d - n)) for v in _observables(ps[i])]
                obs = [[] for _ in o] if obs is None else obs
                for k, v in enumerate(o):
                    obs[k].append(v)
            ex, fin = _evolve(np.stack(Hs), [np.stack(c) for c in C], tl, [np.stack(o) for o in obs])
            for j, i in enumerate(g):
                n = ps[i]["N"] if kind == "kerr" else d
                out[i] = (ex[j], fin[j, :n, :n])
    return [out[i] for i in range(len(ps))]


def _exact_se(case, p):
    H, _ = _operators(p)
    tl, d = _tl(case), H.shape[0]
    A = torch.sparse_csr_tensor(torch.as_tensor(H.indptr.astype(np.int64)), torch.as_tensor(H.indices.astype(np.int64)),
                                torch.as_tensor(H.data * -1j), size=(d, d))
    o = torch.as_tensor(sum(_observables(p)))
    bound = float(np.abs(H).sum(axis=1).max())
    x = torch.as_tensor(_start(d))
    ex = [(o * x.abs() ** 2).sum()]
    for q in range(len(tl) - 1):
        dt = float(tl[q + 1] - tl[q])
        n = max(1, math.ceil(dt * bound / 6.0))
        for _ in range(n):
            term, acc = x, x.clone()
            for k in range(1, 41):
                term = torch.mv(A, term) * (dt / n / k)
                acc = acc + term
            x = acc
        ex.append((o * x.abs() ** 2).sum())
    return torch.stack(ex).numpy().astype(complex)[None]


def _philox(c0, c1, c2, c3, seed):
    m = np.uint64(0xFFFFFFFF)
    k0, k1 = np.uint64(seed & 0xFFFFFFFF), np.uint64(seed >> 32)
    c = [np.asarray(v, np.uint64) for v in (c0, c1, c2, c3)]
    for _ in range(10):
        p0, p1 = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
        c = [(p1 >> np.uint64(32)) ^ c[1] ^ k0, p1 & m, (p0 >> np.uint64(32)) ^ c[3] ^ k1, p0 & m]
        k0, k1 = (k0 + np.uint64(0x9E3779B9)) & m, (k1 + np.uint64(0xBB67AE85)) & m
    return c


def _u01(a, b):
    return ((a >> np.uint64(5)).astype(float) * 67108864.0 + (b >> np.uint64(6)).astype(float) + 0.5) * 2.0 ** -53


def _exact_sde(case, p):
    """Platen's derivative-free strong scheme for one measured operator, all trajectories at once."""
    H, S, C, X, psi = _jc(case, p)
    S, tl, n, master = S[0], _tl(case), case["ntraj"], case["master"]
    d = len(psi)
    G = -1j * H - 0.5 * sum(M.conj().T @ M for M in C + [S])
    Gt, St, Xt = _t(G), _t(S), _t(X)
    gat = [(torch.as_tensor(k, device=_DEV), _t(np.outer(v[0], v[0].conj())))
           for k, v in (_gather(M[None]) for M in C + [S])]
    traj = np.arange(n, dtype=np.uint64)
    if master:
        x = _t(np.outer(psi, psi.conj())).repeat(n, 1, 1)

        def drift(x):
            y = torch.matmul(Gt, x)
            y = y + y.conj().transpose(1, 2)
            for k, w in gat:
                y = y + w * x[:, k][:, :, k]
            return y

        def noise(x):
            y = torch.matmul(St, x)
            y = y + y.conj().transpose(1, 2)
            mu = torch.diagonal(y, dim1=1, dim2=2).sum(-1).real[:, None, None]
            return y - mu * x, mu

        value = lambda x: torch.diagonal(torch.matmul(Xt, x), dim1=1, dim2=2).sum(-1)  # noqa: E731
        size = lambda x: torch.diagonal(x, dim1=1, dim2=2).sum(-1).real[:, None, None]  # noqa: E731
    else:
        x = _t(psi).repeat(n, 1)

        def image(x):
            y = x @ St.T.contiguous()
            return y, 2.0 * (x.conj() * y).sum(-1, keepdim=True).real / (x.abs() ** 2).sum(-1, keepdim=True)

        def drift(x):
            y, mu = image(x)
            return x @ Gt.T.contiguous() + 0.5 * mu * y - 0.125 * mu * mu * x

        def noise(x):
            y, mu = image(x)
            return y - 0.5 * mu * x, mu

        value = lambda x: (x.conj() * (x @ Xt.T.contiguous())).sum(-1) / (x.abs() ** 2).sum(-1)  # noqa: E731
        size = lambda x: (x.abs() ** 2).sum(-1, keepdim=True).sqrt()  # noqa: E731
    shape = (n,) + (1,) * (x.dim() - 1)
    ex, cur, step = [value(x)], [], 0
    for q in range(len(tl) - 1):
        length = float(tl[q + 1] - tl[q])
        ns = max(1, math.ceil(length / case["dt"] - 1e-9))
        h = length / ns
        tot = 0.0
        for _ in range(ns):
            c = _philox(traj & np.uint64(0xFFFFFFFF), traj >> np.uint64(32), np.full(n, step, np.uint64),
                        np.ones(n, np.uint64), p["seed"])
            z = np.sqrt(-2.0 * np.log(_u01(c[0], c[1]))) * np.cos(2.0 * math.pi * _u01(c[2], c[3]))
            dw = torch.as_tensor(math.sqrt(h) * z, device=_DEV).reshape(shape)
            step += 1
            a, (b, mu) = drift(x), noise(x)
            tot = tot + mu * h + dw
            y = x + h * a + dw * b + (noise(x + h * a + math.sqrt(h) * b)[0] - b) * ((dw * dw - h) / (2 * math.sqrt(h)))
            x = y / size(y)
        ex.append(value(x))
        cur.append(tot.reshape(n) / length)
    ex, cur = torch.stack(ex, 1).cpu().numpy(), torch.stack(cur, 1).cpu().numpy()
    return [ex.mean(0)[None], ex.real.std(0, ddof=1)[None] / math.sqrt(n), cur.mean(0)[None]]


def exact(case, seed):
    f, ps = case["family"], _params(case, seed)
    if f == "mc":
        return None  # whole jump ensembles: minutes in numpy
    if f == "se":
        return [_exact_se(case, ps[0])]
    if f == "sde":
        return _exact_sde(case, ps[0])
    if f == "td":
        M = [_optomech(case, p) for p in ps]
        ex, fin = _evolve(np.stack([m[0] for m in M]), [np.stack([m[2][k] for m in M]) for k in range(2)], _tl(case),
                          [np.stack([np.diag(m[3]).real for m in M])],
                          drive=(np.stack([m[1] for m in M]), np.array([p["F"] for p in ps]),
                                 np.array([p["wd"] for p in ps])))
        got = [(ex[i], fin[i]) for i in range(len(ps))]
    else:
        got = _exact_me(case, ps)
    if f == "serve":
        return [np.stack([e[0] for e, _ in got])]
    if f == "me" and case["once"]:
        return list(got[0][:1 + _final(case)])
    return [np.concatenate([r[k].ravel() for r in got]) for k in range(1 + _final(case))]
