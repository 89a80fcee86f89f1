"""The penalty lists where the kernel's storage changes: 16-bit keys in LDS up to
8,192 penalties, 32-bit ones from there on, keys past the room in LDS, counters
that just fit it (150^2 rows) and that do not (151^2); the contact forces against
a plain sum."""
import numpy as np
import pytest

import pd_inputs as P
from gpu_util import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_pen,unused", [(20, 8192, 0.8), (20, 8192, 0.2), (20, 8193, 0.8),
                                            (20, 8193, 0.2), (149, 3000, 0.2), (150, 3000, 0.2)])
def test_forces(n, n_pen, unused):
    import torch
    from paper_2008_01541_amd import PDContext
    sc = P.scene_small(n, n, 1, region_top_layers=1)
    ctx = PDContext(sc.rest, sc.tets, sc.region, sc.dirichlet, sc.mu)
    m = ctx.m
    assert m == (n + 1) ** 2
    rng = np.random.default_rng(n + n_pen)
    start = rng.integers(0, m - 40, n_pen)
    idx = (start[:, None] + np.argsort(rng.random((n_pen, 40)), axis=1)[:, :8]).astype(np.int32)
    idx[rng.random(idx.shape) < unused] = -1
    w = rng.standard_normal(idx.shape)
    c = np.where(rng.random(n_pen) < 0.9, 1.0e3 * rng.random(n_pen), 0.0)
    c[-1] = 1.0e3                              # the largest keys are used
    t = rng.standard_normal((3, n_pen))
    x2 = rng.standard_normal((3, m))
    fcol = torch.empty(3 * m, dtype=torch.float64, device="cuda")
    ctx.collision_update(dev(idx), dev(w), dev(c), dev(t), dev(x2), fcol)
    got = host(fcol, (3, m))
    ctx.close()
    wz, ii = np.where(idx >= 0, w, 0.0), np.maximum(idx, 0)
    r = np.einsum("ps,dps->dp", wz, x2[:, ii]) - t
    ref, size = np.zeros((3, m)), np.zeros((3, m))
    for d in range(3):
        np.add.at(ref[d], ii, -(c * r[d])[:, None] * wz)
        np.add.at(size[d], ii, np.abs((c * r[d])[:, None] * wz))
    # a row adds n terms whose sizes add up to `size`; each term has eight products
    terms = np.bincount(ii[idx >= 0], minlength=m).max() + 16
    assert np.abs(got - ref).max() <= terms * np.finfo(float).eps * size.max()
