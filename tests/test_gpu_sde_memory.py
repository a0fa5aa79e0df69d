"""The stochastic kernel that reads its operators from memory (several measured operators, or wider ones than
the register kernels hold), at the edges of its rows per thread (state lengths 256, 512, 1,024, 2,048, 4,096),
trajectory by trajectory against the FP64 oracle with the same Wiener increments: within 1e-8 (currents
1e-6) in FP64, the bars of the other stochastic tests, and 1e-4 (currents 1e-3) in mixed precision."""
import numpy as np
import pytest
import scipy.sparse as sp

import oracle
from oracle import models as om
import paper_2504_21440_amd as qt

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    print("[gpu] sde memory: creating context", flush=True)
    c = qt.Context(0)
    yield c
    c.close()


def _check(res, ref, prec, k):
    f64 = prec == qt.F64
    assert np.abs(res["expect_tr"][:k] - ref["expect_tr"]).max() <= (1e-8 if f64 else 1e-4)
    assert np.abs(res["measurement"][:k] - ref["measurement"]).max() <= (1e-6 if f64 else 1e-3)
    assert res["stats"]["status"] == 0


@pytest.mark.parametrize("prec", [qt.F64, qt.MIXED])
@pytest.mark.parametrize("d,m,ntraj", [(40, 8, 3), (256, 2, 3), (257, 3, 3), (512, 2, 3), (513, 2, 300), (1024, 3, 300),
                                       (1025, 1, 3), (1025, 2, 3), (1500, 2, 3), (2048, 3, 3), (2049, 2, 3), (3400, 2, 3)])
def test_kets_with_several_measured_operators(ctx, d, m, ntraj, prec):
    """m = 1 measures one operator of one entry per row (the register kernels' case)."""
    print(f"[gpu] sde memory SSE d={d} m={m} ntraj={ntraj} prec={prec}", flush=True)
    g = np.random.default_rng(d + m)
    v = 0.3 * g.uniform(-1, 1, d - 1)
    H = sp.diags([g.uniform(-1, 1, d), v, v], [0, 1, -1], format="csr").astype(complex)
    up = sp.diags(np.full(d - 1, 0.6), 1, format="csr").astype(complex)
    S = [sp.csr_matrix(up / np.sqrt(m)) if k % 2 == 0 else sp.csr_matrix(0.2 * up.conj().T + 0.1 * k * om.qeye(d))
         for k in range(m)]
    psi = g.normal(size=d) + 1j * g.normal(size=d)
    psi /= np.linalg.norm(psi)
    tl = np.linspace(0.0, 0.3, 4)
    e = [sp.diags(np.linspace(0, 1, d)).astype(complex).tocsr(), sp.csr_matrix(up + up.conj().T)]
    ref = oracle.ssesolve(H, S, psi, tl, e, 3, 23, 2e-3)
    res = qt.ssesolve(ctx, H, S, psi, tl, e, ntraj, 23, 2e-3, options=qt.opts(precision=prec), want_traj=True)
    _check(res, ref, prec, 3)


@pytest.mark.parametrize("prec", [qt.F64, qt.MIXED])
@pytest.mark.parametrize("d,m,ntraj", [(6, 2, 3), (16, 2, 3), (17, 2, 3), (23, 2, 300), (32, 3, 3), (33, 2, 300), (45, 2, 3),
                                       (46, 2, 3), (58, 2, 3), (64, 1, 3)])
def test_master_equations_with_several_measured_operators(ctx, d, m, ntraj, prec):
    """n = d^2: a driven cavity, two quadratures (m = 2) and a number measurement (m = 3); m = 1 at d = 64 is
    longer than the register kernels hold."""
    print(f"[gpu] sde memory SME d={d} m={m} ntraj={ntraj} prec={prec}", flush=True)
    a = om.destroy(d)
    H = sp.csr_matrix(0.3 * om.number(d) + 0.4 * (a + a.conj().T))
    C = [0.3 * om.number(d) / d]
    S = [np.sqrt(0.4) * a, np.sqrt(0.3) * 1j * a, 0.2 * om.number(d) / d][:m]
    rho = np.diag(np.exp(-0.5 * np.arange(d))).astype(complex)
    rho /= np.trace(rho)
    tl, e = np.array([0.0, 0.03, 0.2]), [om.number(d), sp.csr_matrix(a + a.conj().T)]
    ref = oracle.smesolve(H, C, S, rho, tl, e, 3, 41, 2e-3)
    res = qt.smesolve(ctx, H, C, S, rho, tl, e, ntraj, 41, 2e-3, options=qt.opts(precision=prec), want_traj=True)
    _check(res, ref, prec, 3)


@pytest.mark.parametrize("prec", [qt.F64, qt.MIXED])
@pytest.mark.parametrize("d", [40, 600, 2100])
def test_no_measured_operator(ctx, d, prec):
    """A closed system: Euler steps of the renormalised ket, the oracle's to rounding."""
    print(f"[gpu] sde memory SSE d={d} m=0 prec={prec}", flush=True)
    g = np.random.default_rng(d)
    v = 0.3 * g.uniform(-1, 1, d - 1)
    H = sp.diags([g.uniform(-1, 1, d), v, v], [0, 1, -1], format="csr").astype(complex)
    psi = g.normal(size=d) + 1j * g.normal(size=d)
    psi /= np.linalg.norm(psi)
    tl, e = np.linspace(0.0, 0.3, 4), [sp.diags(np.linspace(0, 1, d)).astype(complex).tocsr()]
    ref = oracle.ssesolve(H, [], psi, tl, e, 2, 23, 2e-3)
    res = qt.ssesolve(ctx, H, [], psi, tl, e, 2, 23, 2e-3, options=qt.opts(precision=prec), want_traj=True)
    assert np.abs(res["expect_tr"] - ref["expect_tr"]).max() <= (1e-8 if prec == qt.F64 else 1e-4)
    assert res["stats"]["status"] == 0
