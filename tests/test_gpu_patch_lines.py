"""Patch solves for p >= 4 (one wavefront per patch, four patches per
workgroup) where the patch count leaves 1, 2, 3 and 0 wavefronts of the last
workgroup without a patch, for every number of lines per lane."""
import numpy as np
import pytest

from oracle import operators, patches
from tests.gpu_util import check_err, graded, note, to_dev, to_np

pytestmark = pytest.mark.gpu

# the bounds of the parity tests: 1e-12 (FP64), 1e-5 (FP32), 1e-2 (BF16),
# 2e-3 (FP16) relative to the largest entry and in the 2-norm
TOL = {0: 1e-12, 1: 1e-5, 2: 1e-2, 3: 2e-3}


@pytest.fixture(scope="module")
def F():
    import torch
    from paper_2607_02335_amd import fem
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    fem.lib()
    return fem


@pytest.mark.parametrize("p", [4, 5, 6, 7])
@pytest.mark.parametrize("n", [(2, 2, 2), (4, 2, 2), (2, 4, 3), (2, 3, 3)])
@pytest.mark.parametrize("prec", [0, 1, 2, 3])
def test_patch_counts_against_the_oracle(F, p, n, prec):
    note(f"patch lines p={p} n={n} prec={prec}")
    m, w, rng = graded(p, n, 500 + p)
    P = F.Problem(p, n, w)
    # patch inverses of unit residuals are up to 1/lambda_min, about 1e2 here: in range of FP16
    rc = rng.uniform(-1, 1, (m.ncells, m.n1 ** 3)) * ~operators.boundary_copies(m)
    rd = P.pack(to_dev(rc.ravel()), prec)
    z = to_np(P.unpack(P.patch_inverse(rd)))
    ref = patches.SchwarzFactors(m)(operators.scatter(m, to_np(P.unpack(rd))))
    check_err(z, ref[m.dofs], TOL[prec], f"patch lines p={p} n={n} prec={prec}")
