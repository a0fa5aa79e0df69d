"""The staged solver's operator-form right-hand side (kernels_op.hip) against the FP64 oracle at the edges of
its tiles (64 columns, 4 or 8 rows), its row rule (d = 256), its table widths (the widest it takes, and one
more, which the matrix kernels take) and of what it accepts (one entry per row and channel, an exactly
Hermitian initial state); problems of different widths in one launch against the lone solves, bitwise.

Tolerances: as for the other solvers, the oracle's own integrator at the same tolerances: 1e-9 in FP64,
the library's bar of 1e-4 in mixed precision."""
import numpy as np
import pytest
import scipy.sparse as sp

import oracle
import paper_2504_21440_amd as qt

pytestmark = pytest.mark.gpu
TOL = {qt.F64: 1e-9, qt.MIXED: 1e-4}


@pytest.fixture(scope="module")
def ctx():
    print("[gpu] operator form: creating context", flush=True)
    c = qt.Context(0)
    yield c
    c.close()


def _model(d, w, nc, seed, two=False):
    """H of at most w off-diagonals per row, nc channels of one entry in half of the rows (two: the first
    channel has a row of two entries), a ket, and a Hermitian operator."""
    g = np.random.default_rng(seed)
    H = sp.diags(g.normal(size=d), format="lil").astype(complex)
    for q in range(w // 2):  # pairs at distance q + 1, and far ones
        s = q + 1 if q % 2 == 0 else d // 2 - q
        v = 0.5 * (g.normal(size=d - s) + 1j * g.normal(size=d - s))
        H.setdiag(v, s)
        H.setdiag(v.conj(), -s)
    if w % 2:
        v = np.zeros(d - 1, complex)
        v[::2] = 0.4j  # a matching: one more entry in every row
        s = d - 1 if d < 3 else 1
        H.setdiag(H.diagonal(s) + v[:d - s], s)
        H.setdiag(H.diagonal(-s) + v[:d - s].conj(), -s)
    cs = []
    for c in range(nc):
        rows = np.flatnonzero(g.random(d) < 0.5)
        C = sp.csr_matrix((0.3 * (g.normal(size=rows.size) + 1j * g.normal(size=rows.size)),
                           (rows, g.permutation(d)[:rows.size])), shape=(d, d))
        if two and c == 0:
            C = sp.csr_matrix(C + sp.csr_matrix(([0.2, 0.2], ([0, 0], [1, 2])), shape=(d, d)))
        cs.append(C)
    psi = g.normal(size=d) + 1j * g.normal(size=d)
    e = sp.diags([g.normal(size=d), np.full(d - 1, 0.5), np.full(d - 1, 0.5)], [0, 1, -1], format="csr")
    return sp.csr_matrix(H), cs, psi / np.linalg.norm(psi), [e.astype(complex)]


def _offdiagonal_hermitian(m):
    m = m - np.diag(np.diag(m))
    return np.array_equal(m, m.conj().T)


@pytest.mark.parametrize("prec", [qt.F64, qt.MIXED])
@pytest.mark.parametrize("d,w,nc", [(128, 4, 0), (129, 12, 12), (130, 6, 5), (191, 10, 3), (192, 1, 2), (193, 8, 8),
                                    (255, 2, 2), (256, 2, 2), (257, 2, 2), (321, 8, 4)])
def test_sizes_and_widths(ctx, d, w, nc, prec):
    print(f"[gpu] operator form d={d} w={w} nc={nc} prec={prec}", flush=True)
    H, cs, psi, e = _model(d, w, nc, 1000 * d + 10 * w + nc)
    tl = np.linspace(0.0, 0.3, 4)
    ref = oracle.mesolve(H, cs, psi, tl, e, abstol=1e-8, reltol=1e-6)[0]
    L = qt.Liouvillian(ctx, H, cs, qt.FORM_CSR, prec)
    ex, st, fin = qt.mesolve(ctx, L, psi, tl, e, options=qt.opts(precision=prec, abstol=1e-8, reltol=1e-6), want_final=True)
    assert np.abs(ex - ref).max() <= TOL[prec], np.abs(ex - ref).max()
    if d > 128:
        assert _offdiagonal_hermitian(fin)
    L.close()


@pytest.mark.parametrize("prec", [qt.F64, qt.MIXED])
@pytest.mark.parametrize("what", ["wide", "channels", "two entries", "not Hermitian"])
def test_what_the_matrix_kernels_keep(ctx, what, prec):
    print(f"[gpu] operator form left out: {what} prec={prec}", flush=True)
    d = 132
    H, cs, psi, e = _model(d, 14 if what == "wide" else 8, 13 if what == "channels" else 5, 17, two=what == "two entries")
    rho = np.outer(psi, psi.conj())
    if what == "not Hermitian":
        rho[0, 1] += 1e-3
    tl = np.linspace(0.0, 0.3, 3)
    ref = oracle.mesolve(H, cs, rho, tl, e, abstol=1e-8, reltol=1e-6)[0]
    ex = qt.mesolve(ctx, qt.Liouvillian(ctx, H, cs, qt.FORM_CSR, prec), rho, tl, e,
                    options=qt.opts(precision=prec, abstol=1e-8, reltol=1e-6))[0]
    assert np.abs(ex - ref).max() <= TOL[prec], np.abs(ex - ref).max()


@pytest.mark.parametrize("prec", [qt.F64, qt.MIXED])
def test_widths_and_sizes_in_one_launch(ctx, prec):
    """A plan and a server hold problems whose tables differ in width (2, 8, 10, 12) and rows per wave, with one
    of the matrix kernels among them."""
    print(f"[gpu] operator form mixed widths prec={prec}", flush=True)
    tl = np.linspace(0.0, 0.2, 5)
    o = qt.opts(precision=prec)
    probs, keep = [], []
    for d, w, nc in [(140, 2, 1), (300, 8, 2), (165, 10, 10), (130, 12, 12), (90, 14, 2), (257, 2, 12)]:
        H, cs, psi, e = _model(d, w, nc, d + w)
        keep.append(qt.Liouvillian(ctx, H, cs, qt.FORM_CSR, prec))
        probs.append((keep[-1], psi, tl, e))
    lone = []
    for p in probs:
        q = qt.MePlan(ctx, [p], o)
        q.set_shape(8, 1, 0, 2)  # the server's launch shape, for the matrix kernels
        q.run()
        lone.append(q.result(0)[0])
        q.close()
    plan = qt.MePlan(ctx, probs, o)
    plan.set_shape(8, 1, 0, 2)
    for _ in range(2):
        plan.run()
        for i, ref in enumerate(lone):
            np.testing.assert_array_equal(plan.result(i)[0], ref)
        plan.time_rhs(2)  # every problem through the matrix kernels, on the run's vectors
    plan.close()
    srv = qt.Server(ctx, pool_bytes=256 << 20, max_slots=8, steps_per_epoch=5, options=o)
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


@pytest.mark.parametrize("prec", [qt.F64, qt.MIXED])
def test_lanes_shrink_as_problems_finish(ctx, prec):
    """Operator-form and matrix problems in one plan run in two lanes on two streams; each drops its finished
    members by itself (six early, two late, one last): bitwise the lone solves, twice."""
    print(f"[gpu] operator form lanes prec={prec}", flush=True)
    o = qt.opts(precision=prec, reltol=1e-4)
    probs, keep = [], []
    for d, w, nc in [(130, 2, 1), (72, 14, 2)]:
        for t in [0.1, 0.1, 0.1, 0.1, 0.1, 0.1, 4.0, 4.0, 40.0]:
            H, cs, psi, e = _model(d, w, nc, d + w)
            keep.append(qt.Liouvillian(ctx, H, cs, qt.FORM_CSR, prec))
            probs.append((keep[-1], psi, np.linspace(0.0, t, 3), e))
    lone = {}
    plan = qt.MePlan(ctx, probs, o)
    plan.set_shape(8, 1, 0, 2)
    for _ in range(2):
        plan.run()
        for i, p in enumerate(probs):
            key = (i // 9, p[2][-1])
            if key not in lone:
                q = qt.MePlan(ctx, [p], o)
                q.set_shape(8, 1, 0, 2)
                q.run()
                lone[key] = q.result(0)[0]
                q.close()
            np.testing.assert_array_equal(plan.result(i)[0], lone[key])
    plan.close()
