"""Operator form of the staged solver: diagonal collapse operators lose nothing that the assembled matrix keeps.

Dephasing C = sqrt(g) n of a coherent state leaves every population as it is: the decay of rho_ii and the jump
into it cancel.  They cancel in FP64 before the one rounding of the element's factor, so k_ii is exactly 0
and a population only sees the rounding of the trace's renormalisation: 1e-6 of itself in mixed precision,
1e-12 in FP64.  (With rounded operator entries 2e-7 of the rate 0.1 n^2 was left: after t = 20 populations were
off by 7e-4 of the largest.)  The second channel set has rows on and off the diagonal in one operator;
there the oracle's integrator at the same tolerances is the reference (1e-9 in FP64, 1e-4 in mixed precision)."""
from math import lgamma

import numpy as np
import pytest
import scipy.sparse as sp

import oracle
from oracle import models as om
import paper_2504_21440_amd as qt

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    print("[gpu] operator precision: creating context", flush=True)
    c = qt.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("prec", [qt.F64, qt.MIXED])
@pytest.mark.parametrize("d", [160, 272])
def test_dephasing_keeps_populations(ctx, d, prec):
    print(f"[gpu] operator precision dephasing d={d} prec={prec}", flush=True)
    n = np.arange(d)
    al = 7.0
    psi = np.exp(-0.5 * al ** 2 + n * np.log(al) - 0.5 * np.array([lgamma(k + 1.0) for k in n])).astype(complex)
    psi /= np.linalg.norm(psi)
    N = om.number(d)
    t = 20.0 if d == 160 else 7.0
    L = qt.Liouvillian(ctx, sp.csr_matrix(0.3 * N), [sp.csr_matrix(np.sqrt(0.1) * N)], qt.FORM_CSR, prec)
    ex, st, fin = qt.mesolve(ctx, L, psi, np.array([0.0, t]), [N], options=qt.opts(precision=prec, abstol=1e-8, reltol=1e-6),
                             want_final=True)
    L.close()
    p0 = np.abs(psi) ** 2
    bar = 1e-12 if prec == qt.F64 else 1e-6
    assert np.abs(np.diag(fin).real - p0).max() <= bar * p0.max()
    assert np.abs(ex[0, 1] - ex[0, 0]) <= bar * (n * p0).sum()


@pytest.mark.parametrize("prec", [qt.F64, qt.MIXED])
@pytest.mark.parametrize("d", [130, 258])
def test_channels_on_and_off_the_diagonal(ctx, d, prec):
    print(f"[gpu] operator precision mixed channels d={d} prec={prec}", flush=True)
    g = np.random.default_rng(d)
    v = 0.4 * g.normal(size=d - 1)
    H = sp.diags([g.normal(size=d), v, v], [0, 1, -1], format="csr").astype(complex)
    cs = []
    for c in range(3):
        col = np.where(g.random(d) < 0.5, np.arange(d), g.permutation(d))  # half of the rows keep their own column
        val = 0.5 * (g.normal(size=d) + 1j * g.normal(size=d))
        cs.append(sp.csr_matrix((val, (np.arange(d), col)), shape=(d, d)))
    cs.append(cs[0])  # and a channel that repeats another
    psi = g.normal(size=d) + 1j * g.normal(size=d)
    psi /= np.linalg.norm(psi)
    e = [sp.diags(np.linspace(0, 1, d)).astype(complex).tocsr()]
    tl = np.linspace(0.0, 0.3, 4)
    ref = oracle.mesolve(H, cs, psi, tl, e, abstol=1e-8, reltol=1e-6)[0]
    L = qt.Liouvillian(ctx, H, cs, qt.FORM_CSR, prec)
    ex = qt.mesolve(ctx, L, psi, tl, e, options=qt.opts(precision=prec, abstol=1e-8, reltol=1e-6))[0]
    L.close()
    assert np.abs(ex - ref).max() <= (1e-9 if prec == qt.F64 else 1e-4), np.abs(ex - ref).max()


def _unit_channels(d, seed):
    """Channels whose entries are a complex factor times +-1 and +-i (short column entries), one of them on the
    diagonal."""
    g = np.random.default_rng(seed)
    v = 0.4 * g.normal(size=d - 1)
    H = sp.diags([g.normal(size=d), v, v], [0, 1, -1], format="csr").astype(complex)
    cs = []
    for s, f in [(1, np.sqrt(0.2)), (2, np.sqrt(0.3) * np.exp(0.7j)), (d // 2, 0.3j)]:
        cs.append(sp.csr_matrix(sp.diags(f * g.choice([1, -1, 1j, -1j], size=d - s), s, shape=(d, d))))
    psi = g.normal(size=d) + 1j * g.normal(size=d)
    return H, cs, psi / np.linalg.norm(psi)


@pytest.mark.parametrize("prec", [qt.F64, qt.MIXED])
def test_kernel_variants_in_one_launch(ctx, prec):
    """Channels with short column entries, without, and with diagonal entries: alone, all in one plan, and two
    kinds in another, bitwise the same; the short ones against the oracle."""
    print(f"[gpu] operator precision variants prec={prec}", flush=True)
    o = qt.opts(precision=prec)
    tl = np.linspace(0.0, 0.3, 4)
    probs = []

    def add(H, cs, psi):
        d = H.shape[0]
        e = [sp.diags(np.linspace(0, 1, d)).astype(complex).tocsr()]
        probs.append((qt.Liouvillian(ctx, H, cs, qt.FORM_CSR, prec), psi, tl, e))
        return H, cs, psi, tl, e

    short = [add(*_unit_channels(d, d)) for d in (130, 258)]
    g = np.random.default_rng(3)
    for d in (140, 300):
        H, cs, psi = _unit_channels(d, d)
        add(H, [sp.csr_matrix(sp.diags(0.4 * g.normal(size=d - 1), 1, shape=(d, d)).astype(complex))], psi)
        add(H, cs[:1] + [sp.csr_matrix(sp.diags(0.4 * g.normal(size=d)).astype(complex))], psi)
    lone = []
    for p in probs:
        q = qt.MePlan(ctx, [p], o)
        q.run()
        lone.append(q.result(0, want_final=True))
        q.close()
    for k, s in enumerate(short):
        ref = oracle.mesolve(*s)[0]
        assert np.abs(lone[k][0] - ref).max() <= (1e-9 if prec == qt.F64 else 1e-4)
    for pick in (range(len(probs)), [0, 2], [1, 3], [0, 1]):
        plan = qt.MePlan(ctx, [probs[i] for i in pick], o)
        plan.run()
        for k, i in enumerate(pick):
            got = plan.result(k, want_final=True)
            np.testing.assert_array_equal(got[0], lone[i][0])
            np.testing.assert_array_equal(got[2], lone[i][2])
        plan.close()
    for p in probs:
        p[0].close()
