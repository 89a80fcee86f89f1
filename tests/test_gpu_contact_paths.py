"""The contact kernels where their paths divide: the level-set search with and
without the candidates' bounding boxes (and with tets that make a box
unbounded), and the penalty lists in LDS, with the keys in memory, and wholly
in memory."""
import numpy as np
import pytest

import pd_inputs as P
from gpu_util import dev, host, oracle_model
from oracle import collision as ocol

pytestmark = pytest.mark.gpu


def detect(ctx, cand, phi, body, eidx, ew, pbody, rest2, x2):
    import torch
    n = pbody.size
    idx = torch.empty(8 * n, dtype=torch.int32, device="cuda")
    w = torch.empty(8 * n, dtype=torch.float64, device="cuda")
    c = torch.empty(n, dtype=torch.float64, device="cuda")
    t = torch.empty(3 * n, dtype=torch.float64, device="cuda")
    ctx.detect_levelset(dev(eidx.astype(np.int32)), dev(ew), dev(pbody.astype(np.int32)),
                        dev(cand.astype(np.int32)), dev(phi), dev(body.astype(np.int32)),
                        dev(rest2), 5.0e5, dev(x2), idx, w, c, t)
    return host(idx), host(w), host(c), host(t)


@pytest.mark.parametrize("spoil", ["none", "flat", "tiny", "nan", "far"])
def test_levelset_boxes_change_nothing(spoil):
    from paper_2008_01541_amd import PDContext
    sc = P.scene_slit(13, 12, 6, zs=3, ys_end=8)
    bd = P.slit_levelset_bodies(sc, per_cell=1.0, seed=3)
    rid = sc.region_ids()
    pos = np.full(sc.n_nodes, -1, dtype=np.int64)
    pos[rid] = np.arange(rid.size)
    cand, rest2 = pos[bd.body_tets], sc.rest[:, rid]
    assert cand.shape[1] >= 512
    rng = np.random.default_rng(4)
    eidx, ew = np.zeros((bd.proxy_body.size, 4), int), np.zeros((bd.proxy_body.size, 4))
    for b in (0, 1):
        sel = np.nonzero(bd.proxy_body == b)[0]
        _, eidx[sel], ew[sel] = ocol.embed_points(bd.proxy_points[:, sel], cand[:, bd.body_id == b],
                                                  rest2)
    x2 = rest2 + 0.02 * rng.standard_normal(rest2.shape)
    up = np.zeros(rid.size, dtype=bool)
    up[np.unique(cand[:, bd.body_id == 1])] = True
    x2[2] += np.where(up, -0.2, 0.2)
    node = cand[0, 300]
    if spoil == "flat":                      # a tet of no volume
        x2[:, cand[0, 300]] = x2[:, cand[1, 300]]
    elif spoil == "tiny":                    # nearly none, and a long sliver
        x2[:, cand[0, 300]] = x2[:, cand[1, 300]] + 1e-9
        x2[0, cand[3, 700]] += 40.0
    elif spoil == "nan":
        x2[1, node] = np.nan
    elif spoil == "far":
        x2[:, node] = 1e150
    ctx = PDContext(sc.rest, sc.tets, sc.region, sc.dirichlet, sc.mu)
    args = (eidx, ew, bd.proxy_body, rest2, x2)
    boxed = detect(ctx, cand, bd.body_phi, bd.body_id, *args)
    # unused candidates past the room for boxes: every batch is scanned
    pad = 64 * (ctx.n_beta // 64 + 2)
    scanned = detect(ctx, np.concatenate([cand, np.full((4, pad), -1)], axis=1),
                     np.concatenate([bd.body_phi, np.zeros((4, pad))], axis=1),
                     np.concatenate([bd.body_id, np.zeros(pad, int)]), *args)
    ctx.close()
    for a, b in zip(boxed, scanned):
        assert np.array_equal(a, b, equal_nan=True)
    if spoil == "none":
        ref = ocol.levelset_penalties(x2, rest2, eidx, ew, bd.proxy_body, cand, bd.body_phi,
                                      bd.body_id, 5.0e5)
        assert np.array_equal(boxed[2], ref[2]) and (ref[2] > 0).sum() > 20
        assert np.array_equal(boxed[0].reshape(-1, 8), ref[0])


@pytest.mark.parametrize("n,n_pen", [(12, 1), (20, 700), (109, 5000), (112, 3000)])
def test_penalty_lists(n, n_pen):
    """All in LDS; keys past the room in LDS; counters past it (m > 12,288)."""
    import torch
    from paper_2008_01541_amd import PDContext
    sc = P.scene_small(n, n, 1, region_top_layers=1)
    ctx = PDContext(sc.rest, sc.tets, sc.region, sc.dirichlet, sc.mu)
    m = ctx.m
    rng = np.random.default_rng(n)
    # eight distinct nodes around a seeded one each (rows are named many times), some unused
    start = rng.integers(0, m - 40, n_pen)
    idx = (start[:, None] + np.argsort(rng.random((n_pen, 40)), axis=1)[:, :8]).astype(np.int32)
    idx[rng.random(idx.shape) < 0.2] = -1
    w = rng.standard_normal(idx.shape)
    c = np.where(rng.random(n_pen) < 0.9, 1.0e3 * rng.random(n_pen), 0.0)
    t = rng.standard_normal((3, n_pen))
    x2 = rng.standard_normal((3, m))
    fcol = torch.empty(3 * m, dtype=torch.float64, device="cuda")
    ctx.collision_update(dev(idx), dev(w), dev(c), dev(t), dev(x2), fcol)
    got = host(fcol, (3, m))
    ctx.close()
    wz = np.where(idx >= 0, w, 0.0)
    ii = np.maximum(idx, 0)
    r = np.einsum("ps,dps->dp", wz, x2[:, ii]) - t
    ref = np.zeros((3, m))
    size = np.zeros((3, m))
    for d in range(3):
        np.add.at(ref[d], ii, -(c * r[d])[:, None] * wz)
        np.add.at(size[d], ii, np.abs((c * r[d])[:, None] * wz))
    # a row adds up to 8 x 40 terms of size <= `size` in total
    assert np.abs(got - ref).max() <= 400 * np.finfo(float).eps * size.max()
