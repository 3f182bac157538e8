"""The benchmark's result line (no GPU): the byte count of the one-pass DSS."""
import numpy as np
import pytest

import bench


@pytest.mark.parametrize("p,n", [(1, 1), (1, 2), (2, 3), (3, 4), (7, 2)])
def test_one_pass_dss_moves_every_shared_copy_once(p, n):
    ids = [np.arange(n)[:, None] * p + np.arange(p + 1) for _ in range(3)]
    g = [np.bincount(x.ravel())[x].ravel() for x in ids]              # copies of every 1D node, per copy
    mult = g[0][:, None, None] * g[1][None, :, None] * g[2][None, None, :]
    assert bench.op_bytes("dss_once", p, n, 8) == 2 * 8 * int((mult > 1).sum())
    assert bench.OP_OF["dss"] == "dss_once" and bench.OP_OF["dss_axis"] == "dss"
