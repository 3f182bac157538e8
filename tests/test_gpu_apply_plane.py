"""The output-plane apply (p >= 4 in 4-byte arithmetic, p = 4, 5 and the p = 6
mass apply in FP64, the default): the
Laplace and mass applies and the residual of a smoother step against the
oracle on ragged and one-cell meshes, and batches (of one degree and of mixed
degrees) against each problem alone, bit for bit."""
import numpy as np
import pytest

from oracle import operators
from tests.gpu_util import check_err, graded, note, to_dev, to_np

pytestmark = pytest.mark.gpu

TOL = {0: 1e-12, 1: 1e-5, 2: 1e-2, 3: 2e-3}


@pytest.fixture(scope="module")
def F():
    import torch
    from paper_2607_02335_amd import fem
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    fem.lib()
    return fem


@pytest.mark.parametrize("p", [4, 5, 6, 7])
@pytest.mark.parametrize("n", [(1, 1, 1), (3, 2, 2), (65, 1, 1), (13, 5, 2)])
@pytest.mark.parametrize("prec", [1, 2, 3])
def test_apply_against_the_oracle(F, p, n, prec):
    note(f"apply plane p={p} n={n} prec={prec}")
    m, w, rng = graded(p, n, 820 + p)
    P = F.Problem(p, n, w)
    xd = P.gather(to_dev(rng.uniform(-1, 1, m.nglob)), prec)
    x = to_np(P.extract(xd))
    # copies are summed after rounding: each carries its own storage error
    # relative to the largest copy, bounded by 8 copies of the entry bound
    y = to_np(P.scatter(P.apply(xd)))
    ref = operators.apply_global(m, x)
    if np.abs(ref).max() > 0:
        check_err(y, ref, 8 * TOL[prec], f"apply plane p={p} n={n} prec={prec}")
    else:
        np.testing.assert_array_equal(y, 0.0)
    # padding cells stay zero
    yd = P.apply(xd)
    assert bool((P.pack(P.unpack(yd).reshape(-1), prec) == yd).all())


@pytest.mark.parametrize("p", [4, 5, 6, 7])
@pytest.mark.parametrize("n", [(1, 1, 1), (3, 2, 2), (13, 5, 2)])
@pytest.mark.parametrize("prec", [1, 2, 3])
def test_mass_and_residual(F, p, n, prec):
    """The mass apply against the oracle, and a two-sweep smoother step (whose
    second sweep takes the residual) against the same step in FP64, which has
    another apply."""
    note(f"apply plane mass, residual p={p} n={n} prec={prec}")
    m, w, rng = graded(p, n, 840 + p)
    P = F.Problem(p, n, w)
    xd = P.pack(to_dev(rng.uniform(-1, 1, m.ncells * m.n1 ** 3)), prec)
    y = to_np(P.unpack(P.mass_apply(xd)))
    ref = operators.mass_cells(m, to_np(P.unpack(xd)))
    if np.abs(ref).max() > 0:
        check_err(y, ref, TOL[prec], f"mass plane p={p} n={n} prec={prec}")
    else:
        np.testing.assert_array_equal(y, 0.0)
    s = to_np(P.unpack(P.smoother_step(xd, sweeps=2, omega=0.125)))
    s64 = to_np(P.unpack(P.smoother_step(P.pack(P.unpack(xd).reshape(-1)), sweeps=2, omega=0.125)))
    # the second sweep's residual is rounded to storage before the patch solves:
    # its error passes through the sum over up to 8 patches
    if np.abs(s64).max() > 0:
        check_err(s, s64, 8 * TOL[prec], f"residual plane p={p} n={n} prec={prec}")
    else:
        np.testing.assert_array_equal(s, 0.0)


@pytest.mark.parametrize("prec", [1, 2, 3])
@pytest.mark.parametrize("degrees", [(7, 7, 7), (4, 4), (7, 3, 2, 7)])
def test_batch_equals_single(F, degrees, prec):
    note(f"apply plane batch {degrees} prec={prec}")
    shapes = [(13, 5, 4), (1, 1, 1), (3, 7, 5), (65, 1, 2)]
    B = F.Batch([(p, shapes[i], None) for i, p in enumerate(degrees)])
    rng = np.random.default_rng(99)
    xs = [P.pack(to_dev(rng.uniform(-1, 1, int(np.prod(shapes[i])) * (p + 1) ** 3)), prec)
          for i, (P, p) in enumerate(zip(B.problems, degrees))]
    ys = [P.cell_vector(prec) for P in B.problems]
    B.apply(xs, ys)
    for P, x, y in zip(B.problems, xs, ys):
        assert bool((P.apply(x) == y).all())
    B.close()


@pytest.mark.parametrize("p", [4, 5, 6])
@pytest.mark.parametrize("n", [(1, 1, 1), (3, 2, 2), (65, 1, 1), (13, 5, 2)])
def test_fp64(F, p, n):
    test_apply_against_the_oracle(F, p, n, 0)
    test_mass_and_residual(F, p, n, 0)
    # the smoother's second sweep by the library's own parts: the residual's
    # copies round as its terms do, in another order
    m, w, rng = graded(p, n, 860 + p)
    P = F.Problem(p, n, w)
    r = P.pack(to_dev(rng.uniform(-1, 1, m.ncells * m.n1 ** 3)))
    s1 = 0.125 * P.patch_inverse(r)
    s2 = s1 + 0.125 * P.patch_inverse(r - P.apply(s1))
    s = P.smoother_step(r, sweeps=2, omega=0.125)
    if min(n) > 1:
        check_err(to_np(P.unpack(s)), to_np(P.unpack(s2)), 8 * TOL[0], f"smoother plane p={p} n={n}")
    else:
        assert not bool(s.any())                       # no interior vertex


@pytest.mark.parametrize("degrees", [(4, 4, 4), (5, 5), (6, 6), (7, 3, 2, 7)])
def test_fp64_batch_equals_single(F, degrees):
    test_batch_equals_single(F, degrees, 0)
