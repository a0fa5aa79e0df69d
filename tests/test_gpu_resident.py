"""The resident solver (one workgroup per small problem) against the FP64 oracle at the edges of its
kernel classes: elements per workgroup (256, 512, 1,024, 1,536, 2,048 and 3,584 upper-triangle elements),
generator entries per element (6 and 16, and one more, which another solver takes), both forms and
precisions, and what it shares with the other solvers (rejections, given first step, one save time,
many and off-diagonal operators, several problems of several classes at once).

Tolerances: the integrator is the oracle's own at the same tolerances, so FP64 results differ by
rounding only (1e-9 allows it to grow through a few thousand steps); mixed precision is held to the
library's bar of 1e-4."""
import numpy as np
import pytest
import scipy.sparse as sp

import oracle
from oracle import models as om
import paper_2504_21440_amd as qt

pytestmark = pytest.mark.gpu
TOL = {qt.F64: 1e-9, qt.MIXED: 1e-4}


@pytest.fixture(scope="module")
def ctx():
    print("[gpu] resident: creating context", flush=True)
    c = qt.Context(0)
    yield c
    c.close()


def _kerr(N, seed):
    g = np.random.default_rng(seed)
    return om.kerr(N, g.uniform(-1, 1), 0.3 * 20.0 / N, g.uniform(0.5, 1.0), g.uniform(0.8, 1.2))


def _check(ctx, H, cs, rho0, tl, e_ops, prec, form, resident=True, **kw):
    o = dict(abstol=1e-8, reltol=1e-6, **kw)
    ref = oracle.mesolve(H, cs, rho0, tl, e_ops, abstol=1e-8, reltol=1e-6, **kw)[0]
    L = qt.Liouvillian(ctx, H, cs, form, prec)
    ex, st, fin = qt.mesolve(ctx, L, rho0, tl, e_ops, options=qt.opts(precision=prec, **o), want_final=True)
    assert st["status"] == 0
    assert np.abs(ex - ref).max() <= TOL[prec], np.abs(ex - ref).max()
    assert abs(np.trace(fin) - 1.0) <= TOL[prec]
    if resident:  # the solver's states are Hermitian exactly
        np.testing.assert_array_equal(fin, fin.conj().T)
    L.close()
    return st


@pytest.mark.parametrize("prec", [qt.F64, qt.MIXED])
@pytest.mark.parametrize("form", [qt.FORM_CSR, qt.FORM_DENSE])
@pytest.mark.parametrize("N", [1, 2, 3, 22, 23, 31, 32, 44, 45, 48, 54, 55, 63, 64, 80])
def test_cavity_at_class_edges(ctx, N, form, prec):
    if form == qt.FORM_DENSE and prec == qt.F64 and N > 48:
        pytest.skip("the FP64 dense form ends at 48")
    print(f"[gpu] resident cavity N={N} form={form} prec={prec}", flush=True)
    H, cs = _kerr(N, N)
    tl = np.linspace(0.0, 0.3, 4)
    e = [om.number(N), om.destroy(N) + om.destroy(N).conj().T] if N > 1 else [om.qeye(1)]
    _check(ctx, H, cs, om.fock_dm(N, 0), tl, e, prec, form, resident=prec == qt.MIXED or N <= 54)


@pytest.mark.parametrize("prec", [qt.F64, qt.MIXED])
@pytest.mark.parametrize("width", [7, 16, 17])
@pytest.mark.parametrize("d", [22, 31, 44])
def test_entries_per_element(ctx, d, width, prec):
    """Operators whose generator has 7, 16 or 17 entries in its longest rows: two or more channels on
    distinct shifted diagonals beside a tridiagonal Hamiltonian."""
    print(f"[gpu] resident width d={d} width={width} prec={prec}", flush=True)
    g = np.random.default_rng(100 * d + width)
    off = g.normal(size=d - 1)
    H = sp.diags([g.normal(size=d), off, off], [0, 1, -1], format="csr").astype(complex)
    cs = [sp.diags(0.3 * g.normal(size=d - 1 - k), 1 + k, format="csr").astype(complex) for k in range(width - 5)]
    psi = g.normal(size=d) + 1j * g.normal(size=d)
    _check(ctx, H, cs, psi / np.linalg.norm(psi), np.linspace(0.0, 1.0, 5), [om.number(d)], prec, qt.FORM_CSR,
           resident=width <= 16)


@pytest.mark.parametrize("prec", [qt.F64, qt.MIXED])
def test_options_and_operators(ctx, prec):
    print(f"[gpu] resident options prec={prec}", flush=True)
    L = 4
    H, cs = om.ising(L, 1.0, 0.7, 0.4)
    e = [om.site_op(L, i % L, (om.sigmaz, om.sigmax)[i // L % 2]()) for i in range(11)]
    e.append(sp.csr_matrix(np.random.default_rng(3).normal(size=(16, 16)).astype(complex)))  # 256 entries
    rho = np.diag(np.arange(1.0, 17.0)).astype(complex) / 136.0
    # uneven save times, a first step far too large (rejections), then one save time only
    st = _check(ctx, H, cs, rho, np.array([0.0, 1.5, 1.501, 2.0, 3.0]), e, prec, qt.FORM_CSR, h0=1.5)
    assert st["n_reject"] > 0
    Lv = qt.Liouvillian(ctx, H, cs, qt.FORM_CSR, prec)
    ex, st, _ = qt.mesolve(ctx, Lv, rho, [0.3], e[:2])
    assert st["n_accept"] == 0 and abs(ex[0, 0] - np.trace(e[0] @ rho)) <= 1e-6
    with pytest.raises(qt.QtError) as err:
        qt.mesolve(ctx, Lv, rho, [0.0, 5.0], e[:1], options=qt.opts(precision=prec, max_steps=3))
    assert err.value.code == qt.QT_EMAXSTEPS
    # an initial state that is not Hermitian stays with the CSR solver
    bad = rho.copy()
    bad[0, 1] += 0.1
    ref = oracle.mesolve(H, cs, bad, np.linspace(0, 1, 3), e[:2])[0]
    got = qt.mesolve(ctx, Lv, bad, np.linspace(0, 1, 3), e[:2])[0]
    assert np.abs(got - ref).max() <= (1e-9 if prec == qt.F64 else 1e-4)


@pytest.mark.parametrize("prec", [qt.F64, qt.MIXED])
def test_batch_server_and_reruns_are_bitwise_the_lone_solve(ctx, prec):
    """Problems of several classes and one that is not resident, in one plan, run twice with the
    stage timing and the autotuner between (which overwrite the solvers' vectors), and the same
    problems through a server in epochs of 5 steps: all bitwise the lone solves."""
    print(f"[gpu] resident batch / server prec={prec}", flush=True)
    tl = np.linspace(0.0, 0.5, 6)
    o = qt.opts(precision=prec)
    probs = []
    for N, form in [(10, qt.FORM_CSR), (30, qt.FORM_DENSE), (24, qt.FORM_CSR), (40, qt.FORM_DENSE), (45, qt.FORM_CSR)]:
        H, cs = _kerr(N, 7 * N)
        probs.append((qt.Liouvillian(ctx, H, cs, form, prec), om.fock_dm(N, 0), tl, [om.number(N)]))
    H, cs = om.ising(6, 1.0, 0.7, 0.2)
    probs.append((qt.Liouvillian(ctx, H, cs, qt.FORM_CSR, prec), om.all_up_ket(6), tl,
                  [om.site_op(6, 1, om.sigmaz())]))
    plan = qt.MePlan(ctx, probs, o)
    plan.set_shape(8, 1, 0, 2)  # the server's launch shape, for the chain
    lone = []
    for p in probs:
        q = qt.MePlan(ctx, [p], o)
        q.set_shape(8, 1, 0, 2)
        q.run()
        lone.append(q.result(0)[0])
        q.close()
    for _ in range(2):
        plan.run()
        for i, ref in enumerate(lone):
            np.testing.assert_array_equal(plan.result(i)[0], ref)
        plan.time_rhs(2)
        plan.autotune(2)
        plan.set_shape(8, 1, 0, 2)
    plan.close()
    srv = qt.Server(ctx, pool_bytes=64 << 20, max_slots=8, steps_per_epoch=5, options=o)
    tickets = [srv.submit(*p) for p in probs]
    got = {}
    for _ in range(10000):
        srv.step()
        for i, t in enumerate(tickets):
            if i not in got:
                r = srv.poll(t)
                if r is not None:
                    got[i] = r[0]
        if len(got) == len(probs):
            break
    for i, ref in enumerate(lone):
        np.testing.assert_array_equal(got[i], ref)
    srv.close()
