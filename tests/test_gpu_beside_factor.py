"""Calls of one context beside another handle's factorization that is capped to
one workgroup per compute unit, or to one and a half: they run beside it and end
in its first half (it takes about 13 ms, its first workgroups leave after 11;
the calls take less than 2), with the results that they have alone."""
import time

import numpy as np
import pytest

import pd_inputs as P
from pd_inputs.grid import kuhn_grid, layer_mask

pytestmark = pytest.mark.gpu

N = 12032


@pytest.fixture(scope="module")
def factor():
    import ctypes as C
    import torch
    from paper_2008_01541_amd import DenseCholesky
    # two streams for the whole module: they may share a hardware queue, which
    # runs in order, with others created later
    st, main = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(st):
        h = DenseCholesky(N)
        a = torch.rand(N, N, dtype=torch.float64, device="cuda") - 0.5
        a = a + a.T
        a.diagonal().add_(float(N))
        work = torch.empty_like(a)

    def run(wg):
        with torch.cuda.stream(st):
            work.copy_(a)
            torch.cuda.synchronize()
            e0 = torch.cuda.Event(enable_timing=True)
            e0.record()
            assert h._lib.pd_chol_factor(h._h, C.c_void_p(work.data_ptr()), N, N, wg, None) == 0
            e1 = torch.cuda.Event(enable_timing=True)
            e1.record()
        time.sleep(0.002)                     # the factorization is running
        return e0, e1

    yield run, main
    h.close()


def _runner(nx, ny, nz, interior):
    from paper_2008_01541_amd.driver import Alg1Runner
    rest, tets = kuhn_grid(nx, ny, nz, 1.0)
    prox = np.nonzero(layer_mask(nx, ny, nz, [nz]))[0]
    r = Alg1Runner(rest, tets, layer_mask(nx, ny, nz, [nz - 1, nz]), layer_mask(nx, ny, nz, [0]),
                   P.lame_mu(), prox, 1.0e6, interior=interior)
    r.set_spheres(np.array([[nx / 2.0], [ny / 2.0], [nz + 1.8]]), np.array([2.0]))
    r.outer_iteration()
    r.detect()
    return r


def _beside(run, wg, call, results):
    """Runs call alone and beside the factorization; the same results twice.  A
    call that waits for the factorization does so every time; one that ran late
    because the host was held up is tried again."""
    import torch
    call()
    torch.cuda.synchronize()
    alone = [t.clone() for t in results]
    torch.cuda.synchronize()
    for _ in range(3):
        f0, f1 = run(wg)
        c0, c1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        c0.record()
        call()
        c1.record()
        torch.cuda.synchronize()
        for t, s in zip(results, alone):
            assert torch.equal(t, s)
        begun, done, total = f0.elapsed_time(c0), f0.elapsed_time(c1), f0.elapsed_time(f1)
        if 0 < begun < done < 0.5 * total:
            return
    assert False, "the call waited for the factorization"


@pytest.mark.parametrize("wg", [256, 384])
@pytest.mark.parametrize("grid", [(20, 20, 6), (56, 56, 4)])
def test_solve(factor, wg, grid):
    import torch
    run, main = factor
    with torch.cuda.stream(main):
        r = _runner(*grid, "nd")
        g = torch.linspace(-1.0, 1.0, 3 * r.ctx.m, dtype=torch.float64, device="cuda")
        _beside(run, wg, lambda: r.ctx.global_solve(g, r.u), [r.u])
        r.close()


@pytest.mark.parametrize("wg", [256, 384])
def test_collision_update(factor, wg):
    import torch
    run, main = factor
    with torch.cuda.stream(main):
        r = _runner(56, 56, 4, "nd")
        _beside(run, wg,
                lambda: r.ctx.collision_update(r.idx, r.w, r.c, r.t, r.x2, r.fcol), [r.fcol])
        r.close()


# levels of 441 and 928 nodes, and one width of each instance past 1,024
@pytest.mark.parametrize("wg", [256, 384])
@pytest.mark.parametrize("grid", [(20, 20, 6), (31, 28, 6), (33, 33, 6), (38, 38, 6), (40, 41, 6),
                                  (44, 44, 6)])
def test_level_sweeps(factor, wg, grid):
    import torch
    run, main = factor
    with torch.cuda.stream(main):
        r = _runner(*grid, "levels")
        _beside(run, wg, lambda: r.ctx.condense_rhs(r.f, r.ft), [r.ft])
        d2 = torch.linspace(-1.0, 1.0, 3 * r.ctx.m, dtype=torch.float64, device="cuda")
        x = torch.empty_like(r.x)

        def backsub():
            x.zero_()
            r.ctx.backsub(d2, x)

        _beside(run, wg, backsub, [x])
        r.close()
