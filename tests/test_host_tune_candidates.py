"""The launch shapes the autotuner measures: every built shape of the load kinds it may choose among, whatever the
size of the problem and however often the plan has been laid out or tuned before."""
import ctypes

import pytest

import paper_2504_21440_amd as qt


class _Shape(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("lpr", "rg", "xcd", "keep")]


def _candidates(single, fold):
    out = (_Shape * 64)()
    n = qt.lib()["_ZN2qt14csr_candidatesEPNS_8CsrShapeEibb"](out, 64, ctypes.c_bool(single), ctypes.c_bool(fold))
    return [(s.lpr, s.rg, s.xcd, s.keep) for s in out[:n]]


@pytest.mark.parametrize("single", [False, True])
def test_a_plan_that_may_fold_measures_every_shape_of_the_folding_kind(single):
    every, fold = _candidates(single, False), _candidates(single, True)
    assert fold == [s for s in every if s[3] == 2]
    assert len(set(every)) == len(every)
    # the shapes of one load kind: both block orders for a lone problem, and more than one tile
    assert len({s[:2] for s in fold}) >= 4
    assert len(fold) == len({s[:2] for s in fold}) * (2 if single else 1)
    assert {s[3] for s in every} == {0, 1, 2}
