"""The benchmark's result line (no GPU): the byte count of the one-pass DSS, and
a line short enough to be kept whole."""
import itertools
import json

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


def _workload(p, n):
    ks = [dict(label=l, p=p, prec=0, launches=50, total_ms=3.193294979631901, avg_us=63.865899592638016 + i)
          for i, l in enumerate(("apply", "pi_assemble", "pi_combine", "pi_solve"))]
    r = dict(p=p, n=n, unique_dofs=(n * p + 1) ** 3, cell_dofs=(n * (p + 1)) ** 3, s_per_step=0.00024992994000001546,
             kernels=ks, esize=8, csize=8, apply_s=7.314315795898438e-05, pi_s=0.0001615540313720703)
    r["ops"] = bench.op_table(r)
    r["roofline_by_kernel"] = bench.kernel_table(r)
    return r


def test_summary_is_short_and_keeps_the_figures():
    x = 0.123456789012345678
    solves = {a + b: dict(iters=115, p50_s=0.0633123456789, p99_s=x, relres=x)
              for a, b in itertools.product(("", "two_level_"), ("fp64", "fp32", "bf16", "fp16"))}
    paper = {f"q{p}_128": {k: dict(s=x, unique_gdofs=103.123456789, gbs=x) for k in ("mass", "dss", "assembled_mass")}
             for p in (2, 3, 7)}
    layout = {f"q{p}_{n}": [dict(B=2 ** k, mass_s=x, mass_tile=32, mass_unique_gdofs=147.123456, dss_s=x,
                                 dss_unique_gdofs=182.123456) for k in range(8)]
              for p, n in ((2, 160), (3, 128), (4, 96), (5, 80))}
    extra = dict(q3_64=_workload(3, 64), q2_96=_workload(2, 96), q7_24=_workload(7, 24), q7_solve=solves,
                 batch_256=dict(s_per_pass_mixed=0.0085123456, s_per_pass_per_degree=0.0080612345,
                                launches="per_degree", unique_gdofs=33.612345678, autotuned={"7": [0, 0]}),
                 paper_kernels=paper, layout_sweep=layout,
                 serve=dict(requests=10000, wall_s=49.94729742199999, steps=126709, failures=0, failed=[],
                            p50_latency_s=0.007033097270271682, p99_latency_s=0.23276776760850712, mean_iters=15.1892,
                            solved_unique_dofs_per_s=82474807.93996984, hbm_high_water_bytes=11971055360,
                            host_seconds={"server_step": x}))
    out = bench.summary(extra)
    # the line's other fields take about 2,100 characters
    assert len(json.dumps(out)) < 4000
    assert out["q3_64"]["kernels_us"]["pi_solve"] == 66.87
    assert out["q7_solve_iters_p50_ms"]["two_level_fp32"] == [115, 63.31]
    assert out["batch_256"]["ms_mixed"] == 8.512
    assert out["mass_dss_assembled_unique_gdofs"]["q7_128"] == [103.1] * 3
    assert out["layout_mass_dss_unique_gdofs"]["q5_80"]["64"] == [147.1, 182.1]
    assert out["serve"]["steps"] == 126709 and out["serve"]["p99_latency_s"] == 0.2328
    assert bench.summary({"q3_64": _workload(3, 64)}).keys() == {"q3_64"}
