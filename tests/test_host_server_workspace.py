"""The device memory a server asks for beside its request pool: one workgroup table (two int32 arrays of the
table capacity) for each of its three lanes of staged requests, and the slots' records."""
import pytest

import paper_2504_21440_amd as qt


@pytest.mark.parametrize("prec,es", [(qt.MIXED, 8), (qt.F64, 16)])
@pytest.mark.parametrize("pool,slots", [(1 << 30, 8), (16 << 30, 256)])
def test_workspace_holds_three_tables(pool, slots, prec, es):
    cap = 256
    while cap < pool // (11 * es * 32) + slots:  # 32 rows a workgroup at the server's launch shape
        cap *= 2
    extra = qt.server_workspace(pool, slots, 8, qt.opts(precision=prec)) - pool
    assert 3 * 8 * cap <= extra <= 3 * 8 * cap + 4096 * slots + 65536
