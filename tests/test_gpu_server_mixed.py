"""Served requests of every kind at once: matrix-core requests (dense form, generators too wide for the resident
kernel) of one and of five padded sizes, resident ones, and small and large CSR requests on the matrix kernels
and in operator form, one step an epoch and many.  Each result equals the lone solve of a plan at the server's
launch shape, bitwise."""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle import models as om
import paper_2504_21440_amd as qt

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    print("[gpu] server mixed: creating context", flush=True)
    c = qt.Context(0)
    yield c
    c.close()


def _full(d, seed):
    """A full Hamiltonian and one collapse operator: matrix cores in dense form, matrix kernels in CSR form."""
    g = np.random.default_rng(seed)
    h = 0.05 * (g.normal(size=(d, d)) + 1j * g.normal(size=(d, d)))
    return sp.csr_matrix(h + h.conj().T), [sp.csr_matrix(np.sqrt(0.3) * om.destroy(d))]


@pytest.mark.parametrize("prec", [qt.F64, qt.MIXED])
@pytest.mark.parametrize("sizes,steps", [([20], 4), ([10, 20, 36, 52, 70], 1), ([10, 20, 36, 52, 70], 9)])
def test_every_kind_of_request_together(ctx, sizes, steps, prec):
    print(f"[gpu] server mixed sizes={sizes} steps={steps} prec={prec}", flush=True)
    if prec == qt.F64:
        sizes = [d for d in sizes if d <= 40]
    tl = np.linspace(0.0, 0.4, 4)
    o = qt.opts(precision=prec)
    probs, keep = [], []

    def add(H, cs, form, psi):
        keep.append(qt.Liouvillian(ctx, H, cs, form, prec))
        probs.append((keep[-1], psi, tl, [om.number(H.shape[0])]))

    def fock(d, k=1):
        return np.eye(d, dtype=complex)[k]

    for d in sizes:
        add(*_full(d, d), qt.FORM_DENSE, fock(d))
    for N, form in [(12, qt.FORM_DENSE), (20, qt.FORM_CSR), (50, qt.FORM_CSR)]:
        H, cs = qt.model_kerr(N, 1.0, 0.5, 0.8, 1.0)
        add(H, cs, form, fock(N))
    for L in (6, 8):
        H, cs = qt.model_ising(L, 1.0, 0.7, 0.2)
        add(H, cs, qt.FORM_CSR, om.all_up_ket(L))
    H, cs = qt.model_kerr(140, 0.02, 0.0, 0.1, 0.05)
    add(H, cs, qt.FORM_CSR, fock(140))
    lone = []
    for p in probs:
        q = qt.MePlan(ctx, [p], o)
        if p[0].form == qt.FORM_CSR:
            q.set_shape(8, 1, 0, 2)
        q.run()
        lone.append(q.result(0)[0])
        q.close()
    srv = qt.Server(ctx, pool_bytes=256 << 20, max_slots=16, steps_per_epoch=steps, options=o)
    tickets = [srv.submit(*p) for p in probs]
    got = {}
    for _ in range(20000):
        srv.step()
        for i, t in enumerate(tickets):
            if i not in got:
                r = srv.poll(t)
                if r is not None:
                    got[i] = r[0]
        if len(got) == len(probs):
            break
    srv.close()
    assert len(got) == len(probs)
    for i, ref in enumerate(lone):
        np.testing.assert_array_equal(got[i], ref)
    for L in keep:
        L.close()
