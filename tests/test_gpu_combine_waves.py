"""The p >= 4 combine with one wavefront per global node row (the default)
against the one per (storage block, node plane) that large 4-byte outputs take:
a batch whose output is past the line between them gives each problem's own
result bit for bit, with and without accumulation; and meshes with and without
interior vertices in each direction equal the other two forms."""
import numpy as np
import pytest

from tests.gpu_util import graded, note, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import torch
    from paper_2607_02335_amd import fem
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    fem.lib()
    return fem


@pytest.mark.parametrize("prec,count", [(1, 3), (2, 5)])          # 166 and 138 MB of output
def test_large_batch_equals_single_problems(F, prec, count):
    import torch
    n = (48, 48, 48)
    note(f"combine waves batch prec={prec} x{count}")
    B = F.Batch([(4, n, None)] * count)
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    rs = [(torch.rand(P.cell_len, generator=g, device="cuda", dtype=torch.float64) - 0.5).to(F.torch_dtype(prec))
          for P in B.problems]
    zs = [P.cell_vector(prec) for P in B.problems]
    B.patch_inverse(rs, zs)
    for P, r, z in zip(B.problems, rs, zs):
        assert bool((P.patch_inverse(r) == z).all())
    B.close()


@pytest.mark.parametrize("p", [4, 5, 6, 7])
@pytest.mark.parametrize("n", [(1, 1, 1), (1, 3, 2), (33, 1, 2), (9, 2, 1), (2, 2, 2), (17, 3, 2), (65, 2, 3)])
@pytest.mark.parametrize("prec", [0, 1, 2, 3])
def test_waves_equal_the_other_forms(F, p, n, prec):
    note(f"combine waves p={p} n={n} prec={prec}")
    m, w, rng = graded(p, n, 700 + p)
    P = F.Problem(p, n, w)
    rd = P.pack(to_dev(rng.uniform(-1, 1, m.ncells * m.n1 ** 3)), prec)
    z = P.patch_inverse(rd)
    s = P.smoother_step(rd, sweeps=2, omega=0.125)
    assert bool(z.isfinite().all())
    if min(n) == 1:
        assert not bool(z.any())                       # no interior vertex
    try:
        for form in (1, 2):
            F.set_option(F.OPT_COMBINE_PER_CELL, form)
            assert bool((P.patch_inverse(rd) == z).all())
            assert bool((P.smoother_step(rd, sweeps=2, omega=0.125) == s).all())
    finally:
        F.set_option(F.OPT_COMBINE_PER_CELL, 0)
