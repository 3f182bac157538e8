"""The assembly by storage blocks (the restriction of the patch inverse) on
meshes whose rows, layers and last layer meet the 64-cell blocks in every way:
rows longer than, equal to and shorter than a block, a block holding several
rows or layers, a last layer that starts inside a block, one cell per row."""
import numpy as np
import pytest

from oracle import operators, patches
from tests.gpu_util import check_err, graded, note, to_dev, to_np

pytestmark = pytest.mark.gpu

# the bounds of the parity tests (largest entry and 2-norm)
TOL = {0: 1e-12, 1: 1e-5, 2: 1e-2}

SHAPES = [(65, 2, 2), (64, 2, 2), (63, 3, 2), (32, 2, 3), (2, 33, 2), (2, 2, 17), (5, 5, 5), (130, 2, 2), (4, 4, 4)]


@pytest.fixture(scope="module")
def F():
    import torch
    from paper_2607_02335_amd import fem
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    fem.lib()
    return fem


@pytest.mark.parametrize("p", [1, 2, 3, 5])
@pytest.mark.parametrize("n", SHAPES)
def test_patch_inverse_over_block_shapes(F, p, n):
    if p == 5 and n[0] * n[1] * n[2] > 70:
        n = (n[0] // 2 if n[0] > 20 else n[0], n[1] // 2 + 1, 2)
    m, w, rng = graded(p, n, 700 + p)
    P = F.Problem(p, n, w)
    ref_op = patches.SchwarzFactors(m)
    rc = rng.uniform(-1, 1, (m.ncells, m.n1 ** 3)) * ~operators.boundary_copies(m)
    for prec in (0, 1, 2):
        note(f"assemble blocks p={p} n={n} prec={prec}")
        rd = P.pack(to_dev(rc.ravel()), prec)
        z = to_np(P.unpack(P.patch_inverse(rd)))
        ref = ref_op(operators.scatter(m, to_np(P.unpack(rd))))
        check_err(z, ref[m.dofs], TOL[prec], f"assemble blocks p={p} n={n} prec={prec}")


def test_block_shapes_batched_equal_single(F):
    import torch
    specs = [(7, (9, 2, 2)), (3, (65, 2, 2)), (2, (2, 33, 2)), (3, (3, 3, 3)), (7, (2, 3, 4))]
    for prec, dt in ((0, torch.float64), (1, torch.float32)):
        note(f"assemble blocks batched prec={prec}")
        B = F.Batch([(p, n, None) for p, n in specs])
        rng = np.random.default_rng(12)
        rs = [Q.gather(to_dev(rng.uniform(-1, 1, Q.global_len)), prec) for Q in B.problems]
        zs = [Q.cell_vector(prec) for Q in B.problems]
        B.patch_inverse(rs, zs)
        for Q, (p, n), r, z in zip(B.problems, specs, rs, zs):
            np.testing.assert_array_equal(to_np(F.Problem(p, n).patch_inverse(r)), to_np(z))
