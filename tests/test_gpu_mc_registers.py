"""The trajectory kernels that hold A in registers, at the edges of what they take (rows per workgroup
256, 512, 1,024, in complex64 2,048; entries per row 4, 8, 12 and one more, which the kernels that read A
from memory take), trajectory by trajectory against the FP64 oracle with the same Philox stream: the same
jump counts, channels and times within 1e-8 (the bars of the other trajectory tests), expectation values
within 1e-6 in FP64 and 1e-4 in mixed precision."""
import numpy as np
import pytest
import scipy.sparse as sp

import oracle
import paper_2504_21440_amd as qt

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    print("[gpu] mc registers: creating context", flush=True)
    c = qt.Context(0)
    yield c
    c.close()


def _problem(d, width):
    """A banded Hamiltonian of `width` entries in A's longest rows (odd: the diagonal and pairs; even:
    one extra pair that wraps only some rows), two lowering channels of different strength."""
    g = np.random.default_rng(1000 * width + d)
    k = (width - 1) // 2
    offs = list(range(1, k + 1))
    diags = {0: g.uniform(-1, 1, d)}
    for o in offs:
        v = 0.4 * g.uniform(-1, 1, d - o)
        diags[o], diags[-o] = v, v
    H = sp.diags(list(diags.values()), list(diags.keys()), shape=(d, d), format="lil").astype(complex)
    if width % 2 == 0:  # couples disjoint far pairs: one more entry in their rows
        far = d // 2 + k
        for i in range(min(5, d - far)):
            H[i, i + far] = H[i + far, i] = 0.2
    cs = [sp.diags(np.full(d - 1, s), 1, shape=(d, d), format="csr").astype(complex) for s in (0.9, 0.6)]
    n = sp.diags(np.linspace(0.0, 1.0, d), 0, format="csr").astype(complex)
    x = sp.diags([np.ones(d - 1), np.ones(d - 1)], [1, -1], format="csr").astype(complex)
    psi = np.exp(-0.5 * ((np.arange(d) - 0.7 * d) / (0.05 * d + 2.0)) ** 2).astype(complex)
    return sp.csr_matrix(H), cs, psi / np.linalg.norm(psi), [n, x]


@pytest.mark.parametrize("prec", [qt.F64, qt.MIXED])
@pytest.mark.parametrize("d,width", [(255, 3), (256, 4), (257, 5), (256, 8), (512, 9), (513, 12), (1000, 13),
                                     (1023, 3), (1024, 8), (1024, 12), (1025, 12), (2048, 11), (2049, 3)])
def test_trajectories_at_variant_edges(ctx, d, width, prec):
    print(f"[gpu] mc registers d={d} width={width} prec={prec}", flush=True)
    H, cs, psi, e = _problem(d, width)
    tl = np.array([0.0, 0.4, 0.41, 1.5])
    kw = dict(max_jump_record=8)
    ref = oracle.mcsolve(H, cs, psi, tl, e, 3, 11, abstol=1e-8, reltol=1e-6, **kw)
    got = qt.mcsolve(ctx, H, cs, psi, tl, e, 3, 11, options=qt.opts(precision=prec), want_traj=True, **kw)
    if prec == qt.F64:
        np.testing.assert_array_equal(got["njumps"], ref["njumps"])
        assert ref["njumps"].sum() > 0
        for j in range(3):
            m = ref["njumps"][j]
            np.testing.assert_array_equal(got["jump_channels"][j, :m], ref["jump_channels"][j, :m])
            assert np.abs(got["jump_times"][j, :m] - ref["jump_times"][j, :m]).max(initial=0.0) <= 1e-8
    assert np.abs(got["expect_tr"] - ref["expect_tr"]).max() <= (1e-6 if prec == qt.F64 else 1e-4)
