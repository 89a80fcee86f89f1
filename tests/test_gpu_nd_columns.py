"""Sweeps of the nested-dissection factor at the supernode sizes where the
products change: columns of less than a step, of a step and a bit, of several
steps, four and one per wave, and boundaries with a ragged end."""
import numpy as np
import pytest

import pd_inputs as P
from gpu_util import dev, gpu_context, host, oracle_model, rel
from oracle import schur as osch

pytestmark = pytest.mark.gpu

TOL = 1e-10      # inverses of fronts of condition below 1e4, as in the other tests


# leaf sizes: supernodes of up to leaf nodes; one supernode of all 1,904 or 1,694
# interior nodes at the largest
@pytest.mark.parametrize("leaf", [3, 33, 64, 130, 255, 300, 600, 1100, 5000])
@pytest.mark.parametrize("nx,ny", [(16, 15), (10, 21)])
def test_sweeps_match_oracle(leaf, nx, ny):
    import torch
    sc = P.scene_small(nx, ny, 9, h=1.0, region_top_layers=2, seed=leaf)
    om = oracle_model(sc, build_schur=False)
    ctx = gpu_context(sc, interior="nd", nd_leaf=leaf)
    rng = np.random.default_rng(leaf)
    f = rng.normal(size=(3, sc.n_nodes))
    y2 = torch.empty(3 * ctx.m, dtype=torch.float64, device="cuda")
    ctx.condense_rhs(dev(f), y2)
    _, want = osch.forward_sub(om.lu11, om.A21, f[:, om.i1].T, f[:, om.i2].T)
    assert rel(host(y2, (3, -1)), want.T) <= TOL
    d2 = rng.normal(size=(3, ctx.m))
    x0 = rng.normal(size=(3, sc.n_nodes))
    xd = dev(x0)
    ctx.backsub(dev(d2), xd)
    x = x0.copy()
    x[:, om.i1] += osch.back_sub(om.lu11, om.A12, f[:, om.i1].T, d2.T).T
    x[:, om.i2] += d2
    assert rel(host(xd, (3, -1)), x) <= TOL
