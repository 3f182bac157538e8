"""The residual of a smoother's second sweep: the register kernel's two forms
(one wavefront per output plane on meshes of few storage blocks, one per block
otherwise) bit for bit against each other, and the output-plane kernel (p >= 4)
against the oracle's two sweeps in every precision."""
import numpy as np
import pytest

from oracle import operators, patches
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
@pytest.mark.parametrize("prec", [0, 1, 2, 3])
def test_split_residual_equals_whole_cells(F, p, prec):
    """Two sweeps reach a few layers of cells, so the leading layers of a large
    mesh and of its first layers alone have the same values."""
    import torch
    note(f"residual split p={p} prec={prec}")
    n, k = (32, 32, 200), 16                     # 3200 blocks: whole cells; 256: split
    w = [np.full(32, 1.0 / 32)] * 2 + [np.full(n[2], 1.0 / 32)]
    big = F.Problem(p, n, w)
    small = F.Problem(p, (32, 32, k), [w[0], w[1], w[2][:k]])
    g = torch.Generator(device="cuda")
    g.manual_seed(6)
    r = (torch.rand(big.cell_len, generator=g, device="cuda", dtype=torch.float64) - 0.5).to(F.torch_dtype(prec))
    inner = small.cell_len // k * (k - 6)        # a sweep passes two layers on, and the residual none
    zb = big.smoother_step(r, sweeps=2, omega=0.125)[:inner]
    zs = small.smoother_step(r[:small.cell_len].clone(), sweeps=2, omega=0.125)[:inner]
    assert bool(zb.any()) and bool((zb == zs).all())


@pytest.mark.parametrize("p", [4, 5, 6, 7])
@pytest.mark.parametrize("n", [(3, 2, 2), (9, 2, 4)])
@pytest.mark.parametrize("prec", [0, 1, 2, 3])
def test_second_sweep_against_the_oracle(F, p, n, prec):
    note(f"residual plane p={p} n={n} prec={prec}")
    m, w, rng = graded(p, n, 870 + p)
    P = F.Problem(p, n, w)
    rd = P.pack(to_dev(rng.uniform(-1, 1, m.ncells * m.n1 ** 3)), prec)
    S = patches.SchwarzFactors(m)
    rg = operators.scatter(m, to_np(P.unpack(rd)))
    z1 = 0.125 * S(rg)
    z2 = z1 + 0.125 * S(rg - operators.apply_global(m, z1))
    z = to_np(P.unpack(P.smoother_step(rd, sweeps=2, omega=0.125)))
    # the first sweep's result and the residual are rounded to storage: their
    # errors pass through the sum over up to 8 patches
    check_err(z, z2[m.dofs], 8 * TOL[prec], f"second sweep p={p} n={n} prec={prec}")
