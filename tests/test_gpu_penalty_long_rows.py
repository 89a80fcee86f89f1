"""Rows that very many penalty slots name, whose keys a wave sorts instead of a
lane: on both sides of the rule (96 keys), at powers of two and past them, with
16- and 32-bit keys in LDS and with the keys in memory.  The forces add a row's
terms in the order of its keys, so that wrongly ordered keys change bits."""
import numpy as np
import pytest

import pd_inputs as P
from gpu_util import dev, host

pytestmark = pytest.mark.gpu


def penalties(m, lengths, extra, rng):
    """Row 40 a (a = 0, 1, ..) in lengths[a] slots, seven random rows of the other
    half of the region beside each, and extra penalties of eight random rows."""
    rows = np.repeat(40 * np.arange(len(lengths)), lengths)
    rows = rows[rng.permutation(rows.size)]
    n = rows.size + extra
    idx = rng.integers(m // 2, m, (n, 8)).astype(np.int32)
    idx[:, 1:] = (idx[:, :1] - m // 2 + 1 + np.arange(7)) % (m - m // 2) + m // 2    # distinct
    idx[extra:, 3] = rows
    return idx


@pytest.mark.parametrize("lengths,extra,n", [
    ((95, 96, 97, 1), 0, 20), ((127, 128, 129), 0, 20), ((255, 256, 257, 300), 0, 20),
    ((1023, 1024, 1025), 0, 20), ((2049,), 0, 20), ((4500, 1, 40), 0, 20),
    ((700, 97), 5200, 20),                                # the keys do not fit LDS
    ((700, 97, 260), 0, 151),                             # nor the counters
])
def test_forces_in_key_order(lengths, extra, n):
    import torch
    from paper_2008_01541_amd import PDContext
    sc = P.scene_small(n, n, 1, region_top_layers=1)
    ctx = PDContext(sc.rest, sc.tets, sc.region, sc.dirichlet, sc.mu)
    m = ctx.m
    rng = np.random.default_rng(sum(lengths))
    idx = penalties(m, lengths, extra, rng)
    n_pen = idx.shape[0]
    w = rng.standard_normal(idx.shape)
    c = 1.0e3 * rng.random(n_pen) + 1.0
    t = rng.standard_normal((3, n_pen))
    x2 = rng.standard_normal((3, m))
    fcol = torch.empty(3 * m, dtype=torch.float64, device="cuda")

    def forces(idle):
        """With idle penalties that are not active behind the others."""
        pad = lambda a, v: np.concatenate([a, np.full((*a.shape[:-1], idle), v)], axis=-1)
        ctx.collision_update(dev(np.concatenate([idx, np.full((idle, 8), -1, np.int32)])),
                             dev(np.concatenate([w, np.zeros((idle, 8))])), dev(pad(c, 0.0)),
                             dev(pad(t, 0.0)), dev(x2), fcol)
        return host(fcol, (3, m)).copy()

    got = forces(0)
    for idle in (0, 0, 9000, 9000):                       # 9,000: 32-bit keys
        assert np.array_equal(forces(idle), got)
    ctx.close()
    r = np.einsum("ps,dps->dp", w, x2[:, idx]) - t
    ref, size = np.zeros((3, m)), np.zeros((3, m))
    for d in range(3):
        np.add.at(ref[d], idx, -(c * r[d])[:, None] * w)
        np.add.at(size[d], idx, np.abs((c * r[d])[:, None] * w))
    terms = np.bincount(idx.ravel(), minlength=m).max() + 16
    assert np.abs(got - ref).max() <= terms * np.finfo(float).eps * size.max()
