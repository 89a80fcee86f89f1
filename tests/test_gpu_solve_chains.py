"""Triangular solves on both sides of the rule that takes short chains of
super-rows (128 rows, up to six) tile row by tile row: the last super-row full,
ragged, of one tile row and of one row; FP64 and float factor against the
oracle, and a second solve in the bits of the first."""
import numpy as np
import pytest

import pd_inputs as P
from gpu_util import dev, gpu_context, host, oracle_model, rel

pytestmark = pytest.mark.gpu

# condition numbers below 1e4; FP64 vectors, the refined mode to a residual of 1e-12
TOL = {"fp64": 1e-10, "fp32": 1e-8}


# region sizes (nx + 1) (ny + 1) of one layer: 256, 288, 385, 513, 645, 720, 768,
# 775, 836, 900, 1,025 (2, 3, 4, 5, 6, 6, 6, 7, 7, 8 and 9 super-rows)
@pytest.mark.parametrize("nx,ny", [(15, 15), (17, 15), (34, 10), (26, 18), (42, 14), (23, 29),
                                   (31, 23), (30, 24), (37, 21), (29, 29), (40, 24)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_solves_match_oracle(nx, ny, prec):
    import torch
    import paper_2008_01541_amd as pd
    sc = P.scene_small(nx, ny, 2, h=1.0, region_top_layers=1, seed=nx + ny)
    om = oracle_model(sc)
    ctx = gpu_context(sc)
    mode = pd.PD_FP64
    if prec == "fp32":
        mode = pd.PD_FP32_IR
        ctx.set_refinement(max_steps=100, tol=1e-12, fallback=False)
    g = np.random.default_rng(8).normal(size=(3, ctx.m))
    want = np.linalg.solve(om.schur(), g.T).T
    u = torch.empty(3 * ctx.m, dtype=torch.float64, device="cuda")
    bits = []
    for k in range(3):                          # the first: forward inside the factorization
        ctx.global_solve(dev(g), u, mode)
        assert rel(host(u, (3, -1)), want) <= TOL[prec], f"solve {k}"
        bits.append(u.clone())
    assert torch.equal(bits[1], bits[2])
    ctx.close()
