"""The coarse correction at the edges of its kernels: meshes with one storage
block and with a ragged one, coarse planes and columns at the largest size of
the plane solve and just beyond it (the pass solve), single-vertex planes, and
the same problems in one server beside each other."""
import numpy as np
import pytest

from oracle import operators, twolevel
from tests.gpu_util import check_err, graded, note, to_dev, to_np

pytestmark = pytest.mark.gpu

# 1e-11: the fast diagonalisation carries rounding errors of eps times the
# condition number of the coarse operator, about (n / pi)^2 times the square of
# the grading (up to 3) and a small count of sums: 1e-16 * 850 * 9 * 10
TOL = {0: 1e-11, 1: 1e-5}


@pytest.fixture(scope="module")
def F():
    import torch
    from paper_2607_02335_amd import fem
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    fem.lib()
    return fem


SHAPES = [(1, (88, 3, 2)), (1, (92, 3, 3)), (2, (3, 92, 2)), (1, (2, 3, 65)), (1, (3, 2, 66)), (3, (2, 2, 2)),
          (2, (8, 4, 2)), (4, (13, 5, 3)), (7, (2, 9, 4)), (2, (34, 2, 3))]


@pytest.mark.parametrize("p,n", SHAPES)
@pytest.mark.parametrize("prec", [0, 1])
def test_two_level_at_the_edges_of_the_coarse_solve(F, p, n, prec):
    note(f"coarse shapes p={p} n={n} prec={prec}")
    m, w, rng = graded(p, n, 300 + p)
    P = F.Problem(p, n, w)
    rc = rng.uniform(-1, 1, (m.ncells, m.n1 ** 3)) * ~operators.boundary_copies(m)
    rd = P.pack(to_dev(rc.ravel()), prec)
    z = to_np(P.unpack(P.two_level(rd, sweeps=1, omega=0.2)))
    ref = twolevel.TwoLevel(m, 0.2, 1, 1)(operators.scatter(m, to_np(P.unpack(rd))))
    check_err(z, ref[m.dofs], TOL[prec], f"two-level p={p} n={n} prec={prec}")


def test_server_beside_a_mesh_beyond_the_plane_solve(F):
    """A solve whose coarse planes fit takes the pass solve when one beside it
    does not: the same bits as alone."""
    meshes = [(2, (5, 4, 6)), (2, (92, 2, 2)), (3, (4, 4, 4)), (7, (3, 2, 3))]
    fs = [np.random.default_rng(40 + i).uniform(-1, 1, (n[0] * p + 1) * (n[1] * p + 1) * (n[2] * p + 1))
          for i, (p, n) in enumerate(meshes)]
    S = F.Server(hbm_budget=2 << 30, max_active=8, smoother_prec=F.F32, sweeps=1, omega=0.2, precond=F.PC_TWO_LEVEL)
    tickets = [S.submit(p, n, f) for (p, n), f in zip(meshes, fs)]
    got = {}
    while len(got) < len(tickets):
        S.step()
        for t in S.finished():
            got[t] = S.poll(t)[0]
    S.close()
    for t, (p, n), f in zip(tickets, meshes, fs):
        note(f"server beside p={p} n={n}")
        P = F.Problem(p, n)
        u, _ = P.pcg_solve(P.mass_apply(P.gather(to_dev(f))), rtol=1e-8, maxit=2000, smoother_prec=F.F32, sweeps=1,
                           omega=0.2, precond=F.PC_TWO_LEVEL)
        np.testing.assert_array_equal(got[t], to_np(P.extract(u)))
