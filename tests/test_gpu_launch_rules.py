"""Rules that pick a kernel or its launch: the same results on both sides of
each line, and no launch that a rule says is not needed."""
import numpy as np
import pytest

from oracle import operators
from tests.gpu_util import check_err, graded, note, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import torch
    from paper_2607_02335_amd import fem
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    fem.lib()
    return fem


def _launches(F, label, call):
    import torch
    torch.cuda.synchronize()
    F.trace_enable(True)
    try:
        call()
        torch.cuda.synchronize()
        return sum(k["launches"] for k in F.trace_read() if k["label"] == label)
    finally:
        F.trace_enable(False)


@pytest.mark.parametrize("p", [4, 5, 6, 7])
@pytest.mark.parametrize("prec", [0, 1, 2, 3])
def test_pi_fused_has_no_effect_from_degree_4(F, p, prec):
    note(f"pi_fused p={p} prec={prec}")
    m, w, rng = graded(p, (3, 4, 2), 30 + p)
    P = F.Problem(p, m.n, w)
    r = P.pack(to_dev(rng.uniform(-1, 1, m.ncells * m.n1 ** 3)), prec)
    z = P.patch_inverse(r)
    try:
        for v in range(5):
            F.set_option(F.OPT_PI_FUSED, v)
            assert bool((P.patch_inverse(r) == z).all()), v
    finally:
        F.set_option(F.OPT_PI_FUSED, -1)


@pytest.mark.parametrize("prec", [0, 1])
def test_autotune_times_a_launch_once(F, prec):
    """Kernels without a persistent grid are timed with one cap: a warm-up and
    three runs of each kernel, the first index."""
    note(f"autotune prec={prec}")
    B = F.Batch([(p, (5, 4, 3), None) for p in (2, 4, 7, 7)])
    choice = {}
    n = _launches(F, "pi_solve", lambda: choice.update(B.autotune(prec)))
    # degrees 4 and 7: one kernel; degree 2: three kernels with a patch solve
    # launch of their own (the fused sweeps have none)
    assert n == 4 * (1 + 1 + 3)
    assert all(pi % 2 == 0 for _, pi in choice.values()), choice
    B.close()


@pytest.mark.parametrize("p", [4, 5, 6, 7])
@pytest.mark.parametrize("prec", [0, 1, 2, 3])
def test_padding_cells_take_no_part(F, p, prec):
    """Whatever a vector holds in its padding cells, the applies and the residual
    write zero there and the same values elsewhere."""
    import torch
    note(f"padding p={p} prec={prec}")
    m, w, rng = graded(p, (3, 2, 2), 890 + p)
    P = F.Problem(p, m.n, w)
    x = P.pack(to_dev(rng.uniform(-1, 1, m.ncells * m.n1 ** 3)), prec)
    bad = x.clone().view(-1, 64)
    bad[:, m.ncells:] = float("nan")
    bad = bad.view(-1)
    for f in (P.apply, P.mass_apply, lambda v: P.smoother_step(v, sweeps=2, omega=0.125)):
        y = f(x)
        assert not bool(y.view(-1, 64)[:, m.ncells:].any())
        assert bool((f(bad) == y).all())


@pytest.mark.parametrize("n", [(17, 17, 17), (18, 17, 17)])
def test_fp64_mass_on_both_sides_of_the_plane_limit(F, n):
    """The FP64 mass apply at p = 6 takes the output planes from 80 storage
    blocks on."""
    note(f"plane limit n={n}")
    m, w, rng = graded(6, n, 886)
    assert (m.ncells + 63) // 64 in (77, 82)
    P = F.Problem(6, n, w)
    xd = P.pack(to_dev(rng.uniform(-1, 1, m.ncells * m.n1 ** 3)))
    y = to_np(P.unpack(P.mass_apply(xd)))
    check_err(y, operators.mass_cells(m, to_np(P.unpack(xd))), 1e-12, f"mass n={n}")


@pytest.mark.parametrize("p", [1, 2, 3])
def test_streamed_assembly_equals_cached(F, p):
    """FP64 vectors of 96 MiB and more are read past the caches: the leading
    layers of such a mesh against those layers alone."""
    import torch
    note(f"streamed assembly p={p}")
    e = 128 if p == 1 else 64
    per_layer = e * e * (p + 1) ** 3 * 8
    nz, k = (96 << 20) // per_layer + 2, 6
    assert per_layer * nz >= 96 << 20 > per_layer * k
    w = [np.full(e, 1.0 / e)] * 2 + [np.full(nz, 1.0 / e)]
    big = F.Problem(p, (e, e, nz), w)
    small = F.Problem(p, (e, e, k), [w[0], w[1], w[2][:k]])
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    r = torch.rand(big.cell_len, generator=g, device="cuda", dtype=torch.float64) - 0.5
    inner = small.cell_len // k * (k - 2)
    assert bool((big.patch_inverse(r)[:inner] == small.patch_inverse(r[:small.cell_len].clone())[:inner]).all())


@pytest.mark.parametrize("p,n", [(5, (34, 33, 34)), (7, (25, 24, 24))])
def test_large_fp64_combine_equals_the_others(F, p, n):
    note(f"large combine p={p} n={n}")
    import torch
    P = F.Problem(p, n)
    assert P.cell_len * 8 > 56 << 20
    g = torch.Generator(device="cuda")
    g.manual_seed(8)
    r = torch.rand(P.cell_len, generator=g, device="cuda", dtype=torch.float64) - 0.5
    z = P.patch_inverse(r)
    F.set_option(F.OPT_COMBINE_PER_CELL, 1)
    try:
        assert bool((P.patch_inverse(r) == z).all())
    finally:
        F.set_option(F.OPT_COMBINE_PER_CELL, 0)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("degrees", [(2, 3), (7, 3, 2)])
def test_many_rows_batch_equals_single(F, degrees, prec):
    """Above the number of node rows from which a mixed-degree assembly gives a
    wavefront four of them, and without degree 7 the solves without its body."""
    note(f"many rows {degrees} prec={prec}")
    shapes = [(17, 16, 15), (14, 15, 16), (3, 3, 65)] if 7 in degrees else [(29, 28, 31), (30, 33, 27), (3, 130, 5)]
    specs = [(degrees[i % len(degrees)], shapes[i % 3]) for i in range(24)]
    specs += [(degrees[(i + 1) % len(degrees)], shapes[i % 3]) for i in range(12)]
    assert sum(p * p * (a * b * c // 64) for p, (a, b, c) in specs) > 32768
    B = F.Batch([(p, n, None) for p, n in specs])
    rng = np.random.default_rng(14)
    rs = [Q.gather(to_dev(rng.uniform(-1, 1, Q.global_len)), prec) for Q in B.problems]
    zs = [Q.cell_vector(prec) for Q in B.problems]
    B.patch_inverse(rs, zs)
    for Q, r, z in zip(B.problems, rs, zs):
        assert bool((Q.patch_inverse(r) == z).all())
    B.close()


@pytest.mark.parametrize("pc,per_precond", [(0, 2), (3, 2)])
def test_solve_stops_without_a_spare_patch_inverse(F, pc, per_precond):
    """The last allowed iteration queues no preconditioner ahead of reading its
    residual: one preconditioner for p_0, one per iteration but the last."""
    note(f"solve launches pc={pc}")
    m, w, rng = graded(3, (6, 5, 4), 77)
    P = F.Problem(3, m.n, w)
    b = P.mass_apply(P.gather(to_dev(rng.uniform(-1, 1, m.nglob))))
    for maxit in (1, 2, 3):
        def solve():
            _, info = P.pcg_solve(b, rtol=1e-14, maxit=maxit, precond=pc, sweeps=2 if pc == 0 else 1,
                                  omega=0.125 if pc == 0 else 0.2, raise_on_error=False)
            assert info["iters"] == maxit
        assert _launches(F, "pi_solve", solve) == maxit * per_precond


@pytest.mark.parametrize("sp", [0, 1])
def test_head_start_changes_no_iterate(F, sp):
    """A solve to the tolerance and the same solve cut at each iteration end
    at the same residuals (whichever iterations queue work ahead)."""
    note(f"solve iterates sp={sp}")
    m, w, rng = graded(3, (6, 5, 4), 78)
    P = F.Problem(3, m.n, w)
    b = P.mass_apply(P.gather(to_dev(rng.uniform(-1, 1, m.nglob))))
    u, info = P.pcg_solve(b, rtol=1e-8, maxit=200, smoother_prec=sp)
    k = info["iters"]
    v, cut = P.pcg_solve(b, rtol=1e-30, maxit=k, smoother_prec=sp, raise_on_error=False)
    assert cut["iters"] == k and cut["relres"] == info["relres"]
    assert bool((u == v).all())
