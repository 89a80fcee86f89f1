"""Level sweeps at the widths where their kernels change: the edges of the
blocks of 16 rows, of each kernel instance (128, 256, 512, 1,024, 1,536 and
2,048 nodes a level), one level past the widest (a launch per step again),
levels of unequal width, and repeated sweeps in any order (the published
vectors alternate between two copies)."""
import numpy as np
import pytest

import pd_inputs as P
from gpu_util import dev, gpu_context, host, oracle_model, rel
from oracle import schur as osch

pytestmark = pytest.mark.gpu

# The solves go through inverses of the level blocks: a relative error of the
# order of their condition (below 1e4 here) times 1e-16, as in the other tests
TOL = 1e-10


def grid(nx, ny, nz, layers=1):
    return lambda: P.scene_small(nx, ny, nz, h=1.0, region_top_layers=layers, seed=nx + ny)


# (nx + 1) (ny + 1) nodes a level
SCENES = {
    "w4": grid(1, 1, 6), "w15": grid(2, 4, 3), "w16": grid(3, 3, 4), "w17": grid(16, 0 + 1, 3),
    "w128": grid(15, 7, 5), "w130": grid(12, 9, 4), "w256": grid(15, 15, 4), "w270": grid(14, 17, 3),
    "w512": grid(31, 15, 3), "w527": grid(30, 16, 4), "w1024": grid(31, 31, 3),
    "w1056": grid(31, 32, 3), "w1536": grid(47, 31, 3), "w1551": grid(46, 32, 3),
    "w2048": grid(63, 31, 3), "w2079": grid(62, 32, 3), "one level": grid(9, 8, 2),
}


@pytest.mark.parametrize("name", list(SCENES))
def test_sweeps_match_oracle_at_every_width(name):
    import torch
    sc = SCENES[name]()
    om = oracle_model(sc, build_schur=False)
    ctx = gpu_context(sc)
    rng = np.random.default_rng(11)
    y2 = torch.empty(3 * ctx.m, dtype=torch.float64, device="cuda")

    def condense(f):
        ctx.condense_rhs(dev(f), y2)
        _, want = osch.forward_sub(om.lu11, om.A21, f[:, om.i1].T, f[:, om.i2].T)
        assert rel(host(y2, (3, -1)), want.T) <= TOL

    def backsub(f):
        d2 = rng.normal(size=(3, ctx.m))
        x0 = rng.normal(size=(3, sc.n_nodes))
        xd = dev(x0)
        if f is None:
            d2 = d2.astype(np.float32)
            ctx.warmstart_apply(dev(d2), 1.0, xd)
            f, d2 = np.zeros((3, sc.n_nodes)), d2.astype(np.float64)
        else:
            ctx.backsub(dev(d2), xd)
        want = x0.copy()
        want[:, om.i1] += osch.back_sub(om.lu11, om.A12, f[:, om.i1].T, d2.T).T
        want[:, om.i2] += d2
        assert rel(host(xd, (3, -1)), want) <= TOL

    f1, f2 = rng.normal(size=(2, 3, sc.n_nodes))
    condense(f1)
    first = y2.clone()
    condense(f1)                                # a fixed order: the same bits again
    assert torch.equal(first, y2)
    condense(f2)
    backsub(f2)
    backsub(f2)
    backsub(None)
    backsub(None)
    condense(f1)
    backsub(f1)


def test_sweep_replays_match_eager():
    import torch
    sc = P.scene_small(12, 9, 6, h=1.0, region_top_layers=2, seed=7)
    ctx = gpu_context(sc)
    rng = np.random.default_rng(3)
    f = dev(rng.normal(size=(3, sc.n_nodes)))
    d2 = dev(rng.normal(size=(3, ctx.m)))
    y2 = torch.empty(3 * ctx.m, dtype=torch.float64, device="cuda")
    x = torch.zeros(3 * sc.n_nodes, dtype=torch.float64, device="cuda")
    ctx.condense_rhs(f, y2)
    ctx.backsub(d2, x)
    want_y, want_x = y2.clone(), x.clone()
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    ctx.set_stream(s)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        ctx.condense_rhs(f, y2)
        ctx.backsub(d2, x)
    ctx.set_stream(torch.cuda.current_stream())
    for rep in range(5):
        x.zero_()
        y2.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y2, want_y) and torch.equal(x, want_x), f"replay {rep}"
        x.zero_()                                # eager sweeps between the replays
        ctx.condense_rhs(f, y2)
        if rep & 1:
            ctx.backsub(d2, x)
            torch.cuda.synchronize()
            assert torch.equal(x, want_x)
        torch.cuda.synchronize()
