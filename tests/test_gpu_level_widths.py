"""Level sweeps past 1,024 nodes a level, where a part of Z_k is read after the
wait: the edges of the instances (1,280 and 1,792 nodes; those of 1,024, 1,536
and 2,048 are in test_gpu_level_sweeps) against the oracle's solves."""
import numpy as np
import pytest

import pd_inputs as P
from gpu_util import dev, gpu_context, host, oracle_model, rel
from oracle import schur as osch

pytestmark = pytest.mark.gpu

# relative error of the order of the levels' condition (below 1e4) times 1e-16
TOL = 1e-10


# (nx + 1) (ny + 1) = 1,280, 1,281, 1,792 and 1,798 nodes a level
@pytest.mark.parametrize("nx,ny", [(39, 31), (60, 20), (55, 31), (57, 30)])
def test_instance_edges(nx, ny):
    import torch
    sc = P.scene_small(nx, ny, 4, h=1.0, region_top_layers=1, seed=nx)
    om = oracle_model(sc, build_schur=False)
    ctx = gpu_context(sc)
    rng = np.random.default_rng(5)
    y2 = torch.empty(3 * ctx.m, dtype=torch.float64, device="cuda")
    for _ in range(2):                          # both copies of the published vectors
        f = rng.normal(size=(3, sc.n_nodes))
        ctx.condense_rhs(dev(f), y2)
        _, want = osch.forward_sub(om.lu11, om.A21, f[:, om.i1].T, f[:, om.i2].T)
        assert rel(host(y2, (3, -1)), want.T) <= TOL
        d2 = rng.normal(size=(3, ctx.m))
        xd = dev(np.zeros((3, sc.n_nodes)))
        ctx.backsub(dev(d2), xd)
        want = np.zeros((3, sc.n_nodes))
        want[:, om.i1] = osch.back_sub(om.lu11, om.A12, f[:, om.i1].T, d2.T).T
        want[:, om.i2] = d2
        assert rel(host(xd, (3, -1)), want) <= TOL
    ctx.close()
