"""The level-set search over candidates in no spatial order, where the boxes of
batches skip nothing, on both sides of the number from which they are formed
(1,024): the oracle's penalties."""
import numpy as np
import pytest

import pd_inputs as P
from gpu_util import dev, host
from oracle import collision as ocol

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [1, 63, 65, 1000, 1023, 1024, 1248])
def test_shuffled_candidates(count):
    import torch
    from paper_2008_01541_amd import PDContext
    sc = P.scene_slit(13, 12, 6, zs=3, ys_end=8)
    bd = P.slit_levelset_bodies(sc, per_cell=1.0, seed=3)
    rid = sc.region_ids()
    pos = np.full(sc.n_nodes, -1, dtype=np.int64)
    pos[rid] = np.arange(rid.size)
    rng = np.random.default_rng(count)
    cand, rest2 = pos[bd.body_tets], sc.rest[:, rid]
    eidx, ew = np.zeros((bd.proxy_body.size, 4), int), np.zeros((bd.proxy_body.size, 4))
    for b in (0, 1):
        sel = np.nonzero(bd.proxy_body == b)[0]
        _, eidx[sel], ew[sel] = ocol.embed_points(bd.proxy_points[:, sel], cand[:, bd.body_id == b],
                                                  rest2)
    x2 = rest2 + 0.02 * rng.standard_normal(rest2.shape)
    up = np.zeros(rid.size, dtype=bool)
    up[np.unique(cand[:, bd.body_id == 1])] = True
    x2[2] += np.where(up, -0.2, 0.2)
    order = rng.permutation(cand.shape[1])[:count]
    cand, phi, body = cand[:, order], bd.body_phi[:, order], bd.body_id[order]
    ctx = PDContext(sc.rest, sc.tets, sc.region, sc.dirichlet, sc.mu)
    n = bd.proxy_body.size
    idx = torch.empty(8 * n, dtype=torch.int32, device="cuda")
    w = torch.empty(8 * n, dtype=torch.float64, device="cuda")
    c = torch.empty(n, dtype=torch.float64, device="cuda")
    t = torch.empty(3 * n, dtype=torch.float64, device="cuda")
    ctx.detect_levelset(dev(eidx.astype(np.int32)), dev(ew), dev(bd.proxy_body.astype(np.int32)),
                        dev(cand.astype(np.int32)), dev(phi), dev(body.astype(np.int32)),
                        dev(rest2), 5.0e5, dev(x2), idx, w, c, t)
    ref = ocol.levelset_penalties(x2, rest2, eidx, ew, bd.proxy_body, cand, phi, body, 5.0e5)
    got_idx, got_w, got_c = host(idx).reshape(-1, 8), host(w).reshape(-1, 8), host(c)
    ctx.close()
    assert np.array_equal(got_c, ref[2]) and np.array_equal(got_idx, ref[0])
    # barycentric weights of tets with edges of one cell
    assert np.abs(got_w - ref[1]).max() <= 1e-9
