"""The register apply with one wavefront per output plane (meshes of few
storage blocks) against the form with one wavefront per block: the leading
layers of a large uniform mesh see the same cell values, so their results are
the same bit for bit; and small ragged meshes against the oracle."""
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


@pytest.mark.parametrize("p", [2, 3])
@pytest.mark.parametrize("prec", [0, 1, 2])
def test_split_equals_whole_cells(F, p, prec):
    import torch
    note(f"apply split p={p} prec={prec}")
    n = (32, 32, 200)                            # 3200 blocks: one wavefront per block
    k = 8                                        # its first 8 layers alone: 128 blocks, split
    w = [np.full(32, 1.0 / 32)] * 2 + [np.full(200, 1.0 / 32)]
    big = F.Problem(p, n, w)
    small = F.Problem(p, (32, 32, k), [w[0], w[1], w[2][:k]])
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    x = torch.rand(big.cell_len, generator=g, device="cuda", dtype=torch.float64).to(F.torch_dtype(prec))
    xs = x[:small.cell_len].clone()
    # all but the small mesh's last layer (its upper boundary)
    inner = small.cell_len // k * (k - 1)
    assert bool((big.apply(x)[:inner] == small.apply(xs)[:inner]).all())
    assert bool((big.mass_apply(x)[:inner] == small.mass_apply(xs)[:inner]).all())


@pytest.mark.parametrize("p", [2, 3])
@pytest.mark.parametrize("n", [(1, 1, 1), (3, 5, 2), (65, 1, 1), (13, 5, 4)])
@pytest.mark.parametrize("prec", [0, 1, 2, 3])
def test_split_against_the_oracle(F, p, n, prec):
    note(f"apply split p={p} n={n} prec={prec}")
    m, w, rng = graded(p, n, 950 + p)
    P = F.Problem(p, n, w)
    xd = P.gather(to_dev(rng.uniform(-1, 1, m.nglob)), prec)
    y = to_np(P.scatter(P.apply(xd)))
    x = to_np(P.extract(xd))
    ref = operators.apply_global(m, x)
    if np.abs(ref).max() > 0:
        # copies are summed after rounding: each carries its own storage error
        # relative to the largest copy, bounded by 8 copies of the entry bound
        check_err(y, ref, 8 * TOL[prec], f"apply split p={p} n={n} prec={prec}")
    else:
        assert not np.any(y)


@pytest.mark.parametrize("p", [2, 3])
def test_split_equals_whole_cells_fp16(F, p):
    test_split_equals_whole_cells(F, p, 3)
