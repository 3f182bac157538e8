"""The whole DSS in one pass (by storage blocks and node rows) against the
three axis passes of the cascade: bitwise equal in FP64 and FP32 (the same sums
in the same order), within one rounding per pass in 2-byte storage, and against
the oracle's S = G G^T; on meshes whose rows and layers meet the 64-cell blocks
in every way, with directions of a single cell."""
import numpy as np
import pytest

from oracle import operators
from tests.gpu_util import graded, note, to_dev, to_np

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1), (1, 5, 3), (5, 1, 3), (5, 3, 1), (65, 2, 2), (64, 2, 2), (63, 3, 2), (2, 33, 2), (2, 2, 17),
          (5, 5, 5), (130, 1, 2)]


@pytest.fixture(scope="module")
def F():
    import torch
    from paper_2607_02335_amd import fem
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    fem.lib()
    return fem


@pytest.mark.parametrize("p", [1, 2, 3, 4, 7])
@pytest.mark.parametrize("n", SHAPES)
def test_dss_equals_the_axis_passes(F, p, n):
    m, w, rng = graded(p, n, 900 + p)
    P = F.Problem(p, n, w)
    v = rng.uniform(-1, 1, (m.ncells, m.n1 ** 3))
    for prec in (0, 1, 2, 3):
        note(f"dss rows p={p} n={n} prec={prec}")
        vd = P.pack(to_dev(v.ravel()), prec)
        s = P.dss(vd)
        ax = vd.clone()
        for axis in (2, 1, 0):
            P.dss_axis(ax, axis)
        if prec <= 1:
            assert bool((s == ax).all())
        got = to_np(P.unpack(s))
        ref = operators.dss(m, to_np(P.unpack(vd)))
        # at most 8 terms below 1: eps of the storage (half an ulp of 8) times
        # the roundings (FP64 and FP32: 7 sums; 2-byte storage: the last store)
        tol = {0: 8 * 7 * 1.2e-16, 1: 8 * 7 * 6e-8, 2: 8 * 2.0 ** -8, 3: 8 * 2.0 ** -11}[prec]
        assert np.abs(got - ref).max() <= tol
        # continuous bit for bit
        np.testing.assert_array_equal(to_np(P.unpack(P.gather(P.extract(s), prec))), got)
