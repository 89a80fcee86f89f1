"""Three-right-hand-side solves at the sizes where a super-row of 128 rows
changes: one tile, one ragged pair, the head of the chain with and without a
second tile row, an odd last tile row, and several super-rows; FP64 factor and
both refined modes, the first solve (forward inside the factorization) and a
second with the factor kept (forward as a launch of its own)."""
import numpy as np
import pytest

import pd_inputs as P
from gpu_util import dev, gpu_context, host, oracle_model, rel

pytestmark = pytest.mark.gpu

# condition numbers below 1e4 and FP64 vectors; the refined modes are held to a
# residual of 1e-12, so that their error is at most 1e4 times that
MODES = {"fp64": "PD_FP64", "fp32": "PD_FP32_IR", "bf16": "PD_BF16_IR"}
TOL = {"fp64": 1e-10, "fp32": 1e-8, "bf16": 1e-8}


# region sizes m = (nx + 1) (ny + 1) of one layer: 4 .. 441
@pytest.mark.parametrize("nx,ny", [(1, 1), (6, 8), (7, 7), (12, 4), (10, 10), (15, 7), (12, 9),
                                   (18, 9), (15, 15), (18, 16), (20, 20)])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
def test_solves_match_oracle(nx, ny, prec):
    import torch
    import paper_2008_01541_amd as pd
    sc = P.scene_small(nx, ny, 3, h=1.0, region_top_layers=1, seed=nx * ny)
    om = oracle_model(sc)
    ctx = gpu_context(sc)
    if prec != "fp64":
        ctx.set_refinement(max_steps=100, tol=1e-12, fallback=False)
    rng = np.random.default_rng(2)
    m = ctx.m
    for k in range(3):
        g = rng.normal(size=(3, m))
        u = torch.empty(3 * m, dtype=torch.float64, device="cuda")
        ctx.global_solve(dev(g), u, getattr(pd, MODES[prec]))
        want = np.linalg.solve(om.schur(), g.T).T
        assert rel(host(u, (3, -1)), want) <= TOL[prec], f"solve {k}"


def test_first_solve_in_place():
    """The right-hand side is packed for the factorization, and the sentinel of
    the backward solve put in its place, by one kernel."""
    import torch
    sc = P.scene_small(14, 9, 3, h=1.0, region_top_layers=1, seed=4)
    om = oracle_model(sc)
    g = np.random.default_rng(6).normal(size=(3, om.i2.size))
    want = np.linalg.solve(om.schur(), g.T).T
    ctx = gpu_context(sc)
    u = dev(g)
    ctx.global_solve(u, u)
    assert rel(host(u, (3, -1)), want) <= TOL["fp64"]
    u = dev(g)
    ctx.global_solve(u, u)                      # factor kept
    assert rel(host(u, (3, -1)), want) <= TOL["fp64"]
    torch.cuda.synchronize()
