"""The work a program gives this framework, as cases that can be timed.

The sizes are those of the repository's own scenes, tests and benchmark: the
8^3 cube, mid-size slabs, the 56 x 56 x 32 slab (602,112 tets), the 64 x 64 x 40
slit, the standalone Cholesky up to the coupled order 19,494 and the
warm-start network of the slab.  Kinds:

  iterate     Algorithm-1 outer iterations through Alg1Runner on one stream
              (local step, condensation, contact, Cholesky, solves, update)
  pipelined   the same iterations overlapped on two streams
  factor      the dense FP64 Cholesky on a caller's own matrix
  solve       penalty update + refined low-precision solve of the region system
  sweeps      full local step, condensation and back substitution alone: the
              interior's response between two dense solves
  forces      the full local step alone, on a mesh above the cache
  contact     rest-pose level-set detection and its penalty update
  infer       one prediction of the warm-start network
  train       a run of training steps of that network; returns the weights
"""
import functools
import math

import numpy as np
import torch

import pd_inputs as P
from pd_inputs.grid import kuhn_grid, layer_mask
from paper_2008_01541_amd import DenseCholesky, MLP, PDContext
from paper_2008_01541_amd.driver import Alg1Runner

MU = P.lame_mu()
K_PEN = 1.0e6          # penalty stiffness of the sphere scenes
K_LIP = 5.0e5          # and of the slit's lips
DENSITY, DT = 1000.0, 1.0 / 30.0
RATE = 1.0e-4          # learning rate of the training run
DEV = "cuda"


def listed():
    return [
        # the smallest call: one iteration on the 8^3 cube, bound by launches
        dict(name="iterate_cube8", kind="iterate", nx=8, ny=8, nz=8, layers=1, spheres=1,
             interior="levels", inner=1, dynamics=False),
        # an ordinary time step: backward Euler, ragged grid, nested inner iterations
        dict(name="iterate_mid_dynamics", kind="iterate", nx=27, ny=22, nz=13, layers=2, spheres=4,
             interior="nd", inner=2, dynamics=True),
        # the driver's default interior factor at an ordinary size
        dict(name="iterate_levels", kind="iterate", nx=36, ny=31, nz=18, layers=2, spheres=8,
             interior="levels", inner=1, dynamics=False),
        # the benchmark: 602K tets, 6,498 region nodes, two streams
        dict(name="pipelined_slab56", kind="pipelined", nx=56, ny=56, nz=32, layers=2, spheres=16,
             interior="nd", iters=2),
        # the largest scene: self-contact of the slit, 983K tets, 12,155 region nodes
        dict(name="iterate_slit64", kind="iterate_slit", nx=64, ny=64, nz=40, zs=20, ys_end=46),
        # callers' own systems: a small odd order, and the coupled 3m x 3m order of the slab
        dict(name="factor_1001", kind="factor", n=1001),
        dict(name="factor_19494", kind="factor", n=19494),
        # the refined FP32 mode on a slab of ordinary size
        dict(name="solve_fp32", kind="solve", nx=48, ny=44, nz=10, spheres=12, prec="fp32"),
        # what runs between two dense solves, at the benchmark's size
        dict(name="sweeps_slab56", kind="sweeps", nx=56, ny=56, nz=32, interior="nd"),
        # rest-pose level sets on a mid-size slit
        dict(name="contact_levelset", kind="contact", nx=48, ny=40, nz=12, zs=6, ys_end=28),
        # one prediction per frame, and the training run that precedes it (slab network)
        dict(name="infer_slab56", kind="infer", m=6498, hidden=512, batch=1),
        dict(name="train_slab56", kind="train", m=6498, hidden=512, batch=20, steps=32),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["iterate", "iterate", "pipelined", "iterate_slit", "factor", "factor",
                       "solve", "sweeps", "forces", "contact", "infer", "train"])
    if kind == "iterate":
        nx, ny = _log(rng, 7, 56), _log(rng, 7, 56)
        return dict(kind=kind, nx=nx, ny=ny, nz=_log(rng, 5, 32), layers=rng.choice([1, 2, 2]),
                    spheres=rng.randint(1, 16), interior=rng.choice(["levels", "nd"]),
                    inner=rng.choice([1, 1, 2, 3]), dynamics=rng.choice([False, True]))
    if kind == "pipelined":
        return dict(kind=kind, nx=rng.randint(20, 56), ny=rng.randint(20, 56),
                    nz=rng.randint(8, 32), layers=2, spheres=rng.randint(2, 16), interior="nd",
                    iters=rng.randint(2, 4))
    if kind == "iterate_slit":
        nz = rng.randint(8, 40)
        ny = rng.randint(16, 64)
        return dict(kind=kind, nx=rng.randint(16, 64), ny=ny, nz=nz, zs=nz // 2,
                    ys_end=rng.randint(ny // 3, 2 * ny // 3))
    if kind == "factor":
        return dict(kind=kind, n=_log(rng, 200, 19494))
    if kind == "solve":
        return dict(kind=kind, nx=rng.randint(16, 52), ny=rng.randint(16, 52),
                    nz=rng.randint(6, 14), spheres=rng.randint(2, 16),
                    prec=rng.choice(["fp32", "bf16"]))
    if kind == "sweeps":
        return dict(kind=kind, nx=rng.randint(16, 56), ny=rng.randint(16, 56),
                    nz=rng.randint(10, 32), interior=rng.choice(["levels", "nd", "nd"]))
    if kind == "forces":
        return dict(kind=kind, nx=rng.randint(14, 28), ny=rng.randint(14, 28),
                    nz=rng.randint(100, 380))
    if kind == "contact":
        nz = rng.randint(8, 14)
        ny = rng.randint(16, 48)
        return dict(kind=kind, nx=rng.randint(16, 48), ny=ny, nz=nz, zs=nz // 2,
                    ys_end=rng.randint(ny // 2, 3 * ny // 4))
    m, hidden = _log(rng, 81, 6498), rng.choice([128, 256, 500, 512])
    if kind == "infer":
        return dict(kind=kind, m=m, hidden=hidden, batch=rng.choice([1, 1, 3, 32]))
    return dict(kind=kind, m=m, hidden=hidden, batch=rng.choice([7, 20, 32]),
                steps=rng.randint(8, 32))


# ---- inputs ------------------------------------------------------------------

@functools.lru_cache(maxsize=4)
def _grid(nx, ny, nz):
    return kuhn_grid(nx, ny, nz, 1.0)


@functools.lru_cache(maxsize=2)
def _slit(nx, ny, nz, zs, ys_end):
    return P.scene_slit(nx, ny, nz, zs=zs, ys_end=ys_end)


def _slab(case):
    """rest, tets, region, dirichlet, proxies of a slab pinned at the bottom."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    rest, tets = _grid(nx, ny, nz)
    layers = case.get("layers", 2)
    region = layer_mask(nx, ny, nz, range(nz + 1 - layers, nz + 1))
    dirichlet = layer_mask(nx, ny, nz, [0])
    proxies = np.nonzero(layer_mask(nx, ny, nz, [nz]))[0]
    return rest, tets, region, dirichlet, proxies


def _spheres(case, rng):
    """(3, ns) centres and (ns,) radii of spheres pressed into the top face."""
    ns = case["spheres"]
    r = rng.uniform(0.5, 2.0, ns)
    xy = np.stack([rng.uniform(1.0, case["nx"] - 1.0, ns), rng.uniform(1.0, case["ny"] - 1.0, ns)])
    return np.vstack([xy, case["nz"] + r - rng.uniform(0.1, 0.5, ns) * r]), r


def _deformed(rest, fixed, rng, amp=0.02):
    """rest bent smoothly with a small per-node noise; the fixed nodes stay."""
    size = rest.max(axis=1) + 1.0
    x = rest.copy()
    for d in range(3):
        a, b = rng.uniform(0.5, 1.5, 2)
        x[d] += 0.01 * size[2] * np.sin(a * rest[(d + 1) % 3] / size[(d + 1) % 3] * np.pi
                                        + b) * rest[2] / size[2]
    x += amp * rng.standard_normal(rest.shape)
    x[:, fixed] = rest[:, fixed]
    return x


def _iterate_inputs(case, seed):
    rng = np.random.default_rng(seed)
    rest, tets, region, dirichlet, proxies = _slab(case)
    cen, rad = _spheres(case, rng)
    x = _deformed(rest, dirichlet, rng)
    v = np.zeros_like(x)
    if case.get("dynamics"):
        v = 0.05 * rng.standard_normal(x.shape)
        v[:, dirichlet] = 0.0
    return rest, tets, region, dirichlet, proxies, cen, rad, x, v


def _slit_inputs(case, seed):
    sc = _slit(case["nx"], case["ny"], case["nz"], case["zs"], case["ys_end"])
    rng = np.random.default_rng(seed)
    zs = float(case["zs"])
    x = _deformed(sc.rest, sc.dirichlet, rng, amp=0.01)
    # the jaw pose fades out from the bottom to the slit, at most a quarter of
    # the lower half's height; the lips overlap towards the front
    pose = sc.jaw.positions(sc.rest, int(rng.integers(4, sc.jaw.steps + 1))) - sc.rest
    pose *= min(1.0, 0.25 * zs / np.abs(pose[:, sc.bottom]).max())
    x += pose * np.clip(1.0 - sc.rest[2] / zs, 0.0, 1.0)
    x[2, sc.pairs[0]] += rng.uniform(0.02, 0.1) * (1.0 - sc.rest[1, sc.pairs[0]] / case["ys_end"])
    return sc, x


def _contact_inputs(case, seed):
    """The slit's lips pushed into each other, and seeded proxies on both."""
    sc = _slit(case["nx"], case["ny"], case["nz"], case["zs"], case["ys_end"])
    rng = np.random.default_rng(seed)
    bd = P.slit_levelset_bodies(sc, per_cell=1.0, seed=int(rng.integers(1 << 30)))
    rid = sc.region_ids()
    pos = np.full(sc.n_nodes, -1, dtype=np.int64)
    pos[rid] = np.arange(rid.size)
    cand = pos[bd.body_tets].astype(np.int32)
    rest2 = sc.rest[:, rid]
    up = np.zeros(rid.size, dtype=bool)
    up[np.unique(cand[:, bd.body_id == 1])] = True
    x2 = rest2 + 0.01 * rng.standard_normal(rest2.shape)
    front = np.clip(1.0 - rest2[1] / sc.meta_ys_end, 0.0, 1.0)
    x2[2] += np.where(up, -1.0, 1.0) * rng.uniform(0.1, 0.25) * front
    return sc, bd, cand, rest2, x2


def _spd(n, seed):
    """Symmetric U[-0.5, 0.5] entries plus n/2 on the diagonal, as lda-padded columns."""
    lda = (n + 15) // 16 * 16
    g = torch.Generator(device=DEV).manual_seed(seed)
    a = torch.rand(n, n, dtype=torch.float64, device=DEV, generator=g) - 0.5
    a = torch.tril(a) + torch.tril(a, -1).T
    a.diagonal().add_(0.5 * n)
    out = torch.zeros(n, lda, dtype=torch.float64, device=DEV)
    out[:, :n] = a
    return out, lda


def _net_shape(case):
    return 4 * case["m"], case["hidden"], case["hidden"], 3 * case["m"]


def _net_params(case, seed):
    shape = _net_shape(case)
    g = torch.Generator(device=DEV).manual_seed(seed)
    parts = []
    for k, (o, i) in enumerate(zip(shape[1:], shape[:-1])):
        lim = math.sqrt(6.0 / i) * (0.1 if k == 2 else 1.0)
        parts.append((torch.rand(o, i, device=DEV, generator=g) * 2 - 1) * lim)
        parts.append(torch.zeros(o, device=DEV))
    return parts


def _net_data(case, seed, count):
    """Standardised increments with a sparse contact mask, and smaller targets."""
    m = case["m"]
    g = torch.Generator(device=DEV).manual_seed(seed + 77)
    du = torch.randn(count, 3 * m, device=DEV, generator=g)
    mask = (torch.rand(count, m, device=DEV, generator=g) < 0.04).float()
    y = 0.3 * du + 0.1 * torch.randn(count, 3 * m, device=DEV, generator=g)
    return torch.cat([du, mask], 1).contiguous(), y.contiguous()


@functools.lru_cache(maxsize=1)
def _streams():
    """The program's two streams for overlapped iterations."""
    return torch.cuda.Stream(), torch.cuda.Stream()


def _dev(a):
    return torch.tensor(np.ascontiguousarray(a), device=DEV).reshape(-1)


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind in ("iterate", "pipelined"):
        rest, tets, region, dirichlet, proxies, cen, rad, x, v = _iterate_inputs(case, seed)
        dyn = dict(density=DENSITY, dt=DT) if case.get("dynamics") else {}
        with torch.cuda.stream(_streams()[0] if kind == "pipelined" else None):
            r = Alg1Runner(rest, tets, region, dirichlet, MU, proxies, K_PEN,
                           interior=case["interior"], **dyn)
            r.set_spheres(cen, rad)
            if dyn:
                r.set_state(x, v)
            else:
                r.set_positions(x)
        s["run"] = r
    elif kind == "iterate_slit":
        sc, x = _slit_inputs(case, seed)
        r = Alg1Runner(sc.rest, sc.tets, sc.region, sc.dirichlet, MU, np.zeros(0, np.int64),
                       K_LIP, interior="nd")
        r.use_pairs(sc.pairs)
        r.set_positions(x)
        s["run"] = r
    elif kind == "factor":
        s["a"], s["lda"] = _spd(case["n"], seed)
        s["work"] = torch.empty_like(s["a"])
        s["chol"] = DenseCholesky(case["n"])
    elif kind == "solve":
        rest, tets, region, dirichlet, proxies, cen, rad, x, v = _iterate_inputs(case, seed)
        r = Alg1Runner(rest, tets, region, dirichlet, MU, proxies, K_PEN, interior="nd")
        r.set_spheres(cen, rad)
        r.set_positions(x)
        r.ctx.region_gather(r.x, r.x2)
        r.detect()
        # the refined modes stand in for the FP64 solve, so they are refined well
        # below the default stopping point
        r.ctx.set_refinement(max_steps=100, tol=1e-12)
        rng = np.random.default_rng(seed + 1)
        r.g.copy_(_dev(1.0e3 * rng.standard_normal((3, r.ctx.m))))
        s["run"], s["prec"] = r, 1 if case["prec"] == "fp32" else 2
    elif kind in ("sweeps", "forces"):
        rng = np.random.default_rng(seed)
        rest, tets, region, dirichlet, _ = _slab(case)
        c = PDContext(rest, tets, region, dirichlet, MU, interior=case.get("interior", "nd"))
        s["ctx"] = c
        s["x0"] = _dev(_deformed(rest, dirichlet, rng))
        s["f"] = torch.empty_like(s["x0"])
        s["x"] = torch.empty_like(s["x0"])
        s["y2"] = torch.empty(3 * c.m, dtype=torch.float64, device=DEV)
        s["d2"] = _dev(0.01 * rng.standard_normal((3, c.m)))
    elif kind == "contact":
        sc, bd, cand, rest2, x2 = _contact_inputs(case, seed)
        # interior nested dissection with the default leaf: contact uses the region only
        c = PDContext(sc.rest, sc.tets, sc.region, sc.dirichlet, MU, interior="nd")
        n, pb = bd.proxy_body.size, bd.proxy_body
        s["ctx"], s["n"] = c, n
        s["cand"], s["phi"] = _dev(cand), _dev(bd.body_phi)
        s["cbody"], s["pbody"] = _dev(bd.body_id.astype(np.int32)), _dev(pb.astype(np.int32))
        s["rest2"], s["x2"] = _dev(rest2), _dev(x2)
        i32 = dict(dtype=torch.int32, device=DEV)
        f64 = dict(dtype=torch.float64, device=DEV)
        s["eidx"], s["ew"] = torch.empty(4 * n, **i32), torch.empty(4 * n, **f64)
        for b in (0, 1):
            sel = np.nonzero(pb == b)[0]
            a, e = int(sel[0]), int(sel[-1]) + 1
            c.embed_points(_dev(bd.proxy_points[:, a:e]), _dev(cand[:, bd.body_id == b]),
                           s["rest2"], torch.empty(e - a, **i32), s["eidx"][4 * a:4 * e],
                           s["ew"][4 * a:4 * e])
        s["idx"], s["w"] = torch.empty(8 * n, **i32), torch.empty(8 * n, **f64)
        s["c"], s["t"] = torch.empty(n, **f64), torch.empty(3 * n, **f64)
        s["fcol"] = torch.empty(3 * c.m, **f64)
    else:
        p = torch.cat([q.reshape(-1) for q in _net_params(case, seed)]).cpu().numpy()
        b = case["batch"]
        s["net"] = MLP(*_net_shape(case), 32, p)
        count = b if kind == "infer" else b * min(case["steps"], 4)
        s["x"], s["y"] = _net_data(case, seed, count)
        s["out"] = torch.empty_like(s["y"])
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind in ("iterate", "iterate_slit"):
        r = s["run"]
        r.outer_iteration(n_inner=case.get("inner", 1))
        if case.get("dynamics"):
            r.advance_time_step()
            return {"x": r.x, "v": r.v}
        return {"x": r.x}
    if kind == "pipelined":
        r = s["run"]
        main, second = _streams()
        with torch.cuda.stream(main):
            r.run_pipelined(case["iters"], factor_stream=second)
        return {"x": r.x}
    if kind == "factor":
        # the matrix is the caller's and is factored in place, so it is copied first
        s["work"].copy_(s["a"])
        s["chol"].factor(s["work"].view(-1), case["n"], s["lda"], want_info=False)
        return s["work"]
    if kind == "solve":
        r = s["run"]
        r.ctx.collision_update(r.idx, r.w, r.c, r.t, r.x2, r.fcol)
        r.ctx.global_solve(r.g, r.u, s["prec"])
        return {"u": r.u, "fcol": r.fcol}
    if kind == "sweeps":
        c = s["ctx"]
        s["x"].copy_(s["x0"])
        c.local_step_full(s["x"], s["f"])
        c.condense_rhs(s["f"], s["y2"])
        c.backsub(s["d2"], s["x"])
        return {"y2": s["y2"], "x": s["x"]}
    if kind == "forces":
        s["ctx"].local_step_full(s["x0"], s["f"])
        return {"f": s["f"]}
    if kind == "contact":
        c = s["ctx"]
        c.detect_levelset(s["eidx"], s["ew"], s["pbody"], s["cand"], s["phi"], s["cbody"],
                          s["rest2"], K_LIP, s["x2"], s["idx"], s["w"], s["c"], s["t"])
        c.collision_update(s["idx"], s["w"], s["c"], s["t"], s["x2"], s["fcol"])
        return {"idx": s["idx"], "w": s["w"], "c": s["c"], "t": s["t"], "fcol": s["fcol"]}
    if kind == "infer":
        s["net"].forward(s["x"], s["out"])
        return s["out"]
    b, parts = case["batch"], s["x"].shape[0] // case["batch"]
    for k in range(case["steps"]):
        j = b * (k % parts)
        s["net"].train_step(s["x"][j:j + b], s["y"][j:j + b], RATE, want_loss=False)
    return s["net"].params()


# ---- what a pass cannot do without -------------------------------------------

def _counts(case):
    """Nodes, tets, region nodes and interior nodes of a slab or slit case."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    layer = (nx + 1) * (ny + 1)
    if "zs" in case:
        twins = (nx + 1) * case["ys_end"]
        n = layer * (nz + 1) + twins
        m = 3 * (nx + 1) * (case["ys_end"] + 1) + twins
        return n, 6 * nx * ny * nz, m, n - m - 2 * layer
    m = layer * case.get("layers", 2)
    return layer * (nz + 1), 6 * nx * ny * nz, m, layer * nz - m


def _interior_bytes(case):
    """Bytes of a sparse factor of the interior: 15 n^(4/3) values of 8 B (the
    growth of nested dissection on a regular grid; 0.54 GB for the 97,470
    interior nodes of the 56 x 56 x 32 slab)."""
    n1 = max(_counts(case)[3], 2)
    return 8.0 * n1 * (n1 ** (1.0 / 3.0)) * 15.0


def work(case):
    kind = case["kind"]
    if kind == "factor":
        n = case["n"]
        return {"bytes": 8.0 * n * n, "flops": n ** 3 / 3.0}
    if kind in ("infer", "train"):
        nin, h1, h2, nout = _net_shape(case)
        nw, b = nin * h1 + h1 * h2 + h2 * nout, case["batch"]
        if kind == "infer":
            return {"bytes": 2.0 * nw + 4.0 * b * (nin + nout), "flops": 2.0 * nw * b}
        # per step: master weights and both moments read and written, BF16 weights
        # read by the forward and backward pass and written once
        return {"bytes": case["steps"] * (24.0 + 6.0) * nw + 4.0 * nw,
                "flops": case["steps"] * 6.0 * nw * b}
    n, tets, m, n1 = _counts(case)
    local = tets * (16.0 + 72.0 + 8.0) + n * 48.0
    if kind == "forces":
        return {"bytes": local, "flops": tets * 600.0}
    if kind == "contact":
        npx = 2.0 * case["nx"] * case["ys_end"]
        cand = 6.0 * 2.0 * case["nx"] * case["ys_end"]
        return {"bytes": npx * (16 + 32 + 4 + 32 + 64 + 8 + 24) + cand * (16 + 32 + 4) + m * 72.0,
                "flops": npx * 2000.0}
    inner = case.get("inner", 1) * case.get("iters", 1)
    outer = case.get("iters", 1)
    dense = {"bytes": 8.0 * m * m, "flops": m ** 3 / 3.0 + 6.0 * m * m + 6.0 * m * m}
    sweeps = {"bytes": 2.0 * _interior_bytes(case) + local,
              "flops": 4.0 * 3.0 * _interior_bytes(case) / 8.0 + tets * 600.0}
    if kind == "sweeps":
        return sweeps
    if kind == "solve":
        return dense
    return {k: inner * dense[k] + outer * sweeps[k] for k in ("bytes", "flops")}


# ---- the same results in 64 bits, by plain torch -----------------------------

class _Elastic:
    """Full-space model: stiffness, forces and conjugate-gradient solves."""

    def __init__(self, rest, tets, region, dirichlet, dynamics=False):
        f64 = dict(dtype=torch.float64, device=DEV)
        self.n = n = rest.shape[1]
        X = torch.tensor(np.ascontiguousarray(rest.T), **f64)
        self.T = torch.tensor(np.ascontiguousarray(tets.T), device=DEV).long()
        D = (X[self.T[:, 1:]] - X[self.T[:, :1]]).transpose(1, 2)       # columns: edges
        inv, det = _inv3(D)
        self.vol = det / 6.0
        self.B = torch.cat([-inv.sum(1, keepdim=True), inv], 1)         # (T, 4, 3) gradients
        self.free = torch.tensor(~dirichlet, device=DEV)
        reg = torch.tensor(region & ~dirichlet, device=DEV)
        self.region = reg.nonzero()[:, 0]
        beta = reg[self.T].all(1)
        self.alpha, self.beta = (~beta).nonzero()[:, 0], beta.nonzero()[:, 0]
        self.D = torch.zeros(n, **f64)
        if dynamics:
            mass = torch.zeros(n, **f64).index_add_(
                0, self.T.reshape(-1), (0.25 * DENSITY * self.vol)[:, None].expand(-1, 4).reshape(-1))
            self.D = mass / DT ** 2
        self.Kfull = self._matrix(torch.arange(self.T.shape[0], device=DEV), self.D)
        self.Kalpha = self._matrix(self.alpha, self.D)
        diag = torch.zeros(n, **f64)
        ke = (self.B * self.B).sum(2) * (2.0 * MU * self.vol)[:, None]
        self.diag = diag.index_add_(0, self.T.reshape(-1), ke.reshape(-1)) + self.D

    def _matrix(self, sel, extra):
        t, b = self.T[sel], self.B[sel]
        ke = (2.0 * MU * self.vol[sel])[:, None, None] * (b @ b.transpose(1, 2))
        i = t[:, :, None].expand(-1, -1, 4).reshape(-1)
        j = t[:, None, :].expand(-1, 4, -1).reshape(-1)
        a = torch.arange(self.n, device=DEV)
        m = torch.sparse_coo_tensor(torch.stack([torch.cat([i, a]), torch.cat([j, a])]),
                                    torch.cat([ke.reshape(-1), extra]), (self.n, self.n))
        return m.coalesce().to_sparse_csr()

    def forces(self, x, sel):
        """Elastic forces of the tets sel at x (n, 3): -vol 2 mu (F - polar F) B."""
        t, b = self.T[sel], self.B[sel]
        F = x[t].transpose(1, 2) @ b
        f = -(2.0 * MU * self.vol[sel])[:, None, None] * (b @ (F - _polar(F)).transpose(1, 2))
        return torch.zeros_like(x).index_add_(0, t.reshape(-1), f.reshape(-1, 3))

    def solve(self, rhs, pen):
        """(K + W^T C W) d = rhs on the free nodes; pen = (idx (p, s), w (p, s), c (p,))."""
        idx, w, c = pen
        free = self.free[:, None].to(rhs.dtype)
        dg = self.diag.clone().index_add_(0, idx.reshape(-1), (c[:, None] * w * w).reshape(-1))
        minv = free / dg[:, None]

        def apply(v):
            y = self.Kfull @ v
            q = (w[:, :, None] * v[idx]).sum(1) * c[:, None]
            return y.index_add_(0, idx.reshape(-1), (w[:, :, None] * q[:, None, :]).reshape(-1, 3)) * free

        b = rhs * free
        d = torch.zeros_like(b)
        for _ in range(2):                                   # restarted from the true residual
            r = b - apply(d)
            z = minv * r
            p, rz = z.clone(), (r * z).sum(0)
            goal = 1e-15 * b.norm()
            for it in range(6000):
                q = apply(p)
                a = rz / (p * q).sum(0).clamp_min(1e-300)
                d = d + a * p
                r = r - a * q
                z = minv * r
                new = (r * z).sum(0)
                p = z + (new / rz.clamp_min(1e-300)) * p
                rz = new
                if it % 50 == 49 and float(r.norm()) <= float(goal):
                    break
        return d

    def sphere_penalties(self, x, proxies, cen, rad):
        px = torch.tensor(np.asarray(proxies), device=DEV).long()
        c = torch.tensor(cen.T.copy(), device=DEV)
        r = torch.tensor(rad, device=DEV)
        v = x[px][:, None, :] - c[None]
        dist = v.norm(dim=2)
        depth = torch.where(dist < r, r - dist, torch.full_like(dist, -1.0))
        best, s = depth.max(1)
        hit = (best > 0).nonzero()[:, 0]
        s = s[hit]
        vv, dd = v[hit, s], dist[hit, s]
        target = c[s] + r[s][:, None] * vv / dd[:, None]
        idx = px[hit][:, None]
        one = torch.ones(hit.numel(), 1, dtype=torch.float64, device=DEV)
        return idx, one, torch.full((hit.numel(),), K_PEN, dtype=torch.float64, device=DEV), target


def _inv3(A):
    c = torch.stack([torch.linalg.cross(A[:, :, 1], A[:, :, 2]),
                     torch.linalg.cross(A[:, :, 2], A[:, :, 0]),
                     torch.linalg.cross(A[:, :, 0], A[:, :, 1])], 1)
    det = (c[:, 0] * A[:, :, 0]).sum(1)
    return c / det[:, None, None], det


def _polar(F):
    """The rotation of F = R S by Newton's iteration (det F > 0 here)."""
    R = F
    for _ in range(14):
        R = 0.5 * (R + _inv3(R)[0].transpose(1, 2))
    return R


def _contact_force(pen, target, x):
    idx, w, c = pen
    q = ((w[:, :, None] * x[idx]).sum(1) - target) * c[:, None]
    return torch.zeros_like(x).index_add_(0, idx.reshape(-1),
                                          -(w[:, :, None] * q[:, None, :]).reshape(-1, 3))


def _pair_penalties(x, pairs):
    a, b = (torch.tensor(p, device=DEV).long() for p in pairs)
    hit = (x[b, 2] < x[a, 2]).nonzero()[:, 0]
    idx = torch.stack([a[hit], b[hit]], 1)
    w = torch.tensor([[1.0, -1.0]], dtype=torch.float64, device=DEV).expand(hit.numel(), 2)
    return (idx, w, torch.full((hit.numel(),), K_LIP, dtype=torch.float64, device=DEV),
            torch.zeros(hit.numel(), 3, dtype=torch.float64, device=DEV))


def _flat(x):
    return x.T.contiguous().reshape(-1)


def _exact_iterations(model, x, penalties, inner, outer, y=None):
    """Algorithm 1 in the full space: outer forces linear in the correction, region
    forces and contacts renewed in every inner iteration."""
    reg = torch.zeros(model.n, 1, dtype=torch.float64, device=DEV)
    reg[model.region] = 1.0
    for _ in range(outer):
        fa = model.forces(x, model.alpha)
        if y is not None:
            fa = fa - model.D[:, None] * (x - y)
        d = torch.zeros_like(x)
        for _ in range(inner):
            xc = x + d
            *pen, target = penalties(xc)
            r = fa - model.Kalpha @ d + reg * (model.forces(xc, model.beta)
                                               + _contact_force(pen, target, xc))
            d = d + model.solve(r, pen)
        x = x + d
    return x


def exact(case, seed):
    kind = case["kind"]
    to = lambda a: torch.tensor(np.ascontiguousarray(a.T), device=DEV)  # noqa: E731
    if kind in ("iterate", "pipelined", "solve"):
        rest, tets, region, dirichlet, proxies, cen, rad, x, v = _iterate_inputs(case, seed)
        model = _Elastic(rest, tets, region, dirichlet, bool(case.get("dynamics")))
        X, V = to(x), to(v)
        pens = lambda z: model.sphere_penalties(z, proxies, cen, rad)  # noqa: E731
        if kind == "solve":
            *pen, target = pens(X)
            rng = np.random.default_rng(seed + 1)
            g = torch.zeros_like(X)
            g[model.region] = to(1.0e3 * rng.standard_normal((3, model.region.numel())))
            return {"u": _flat(model.solve(g, pen)[model.region]),
                    "fcol": _flat(_contact_force(pen, target, X)[model.region])}
        y = X + DT * V if case.get("dynamics") else None
        x1 = _exact_iterations(model, X, pens, case.get("inner", 1), case.get("iters", 1), y)
        if case.get("dynamics"):
            return {"x": _flat(x1), "v": _flat((x1 - X) / DT)}
        return {"x": _flat(x1)}
    if kind == "iterate_slit":
        sc, x = _slit_inputs(case, seed)
        model = _Elastic(sc.rest, sc.tets, sc.region, sc.dirichlet)
        pens = lambda z: _pair_penalties(z, sc.pairs)  # noqa: E731
        return {"x": _flat(_exact_iterations(model, to(x), pens, 1, 1))}
    if kind == "factor":
        a, lda = _spd(case["n"], seed)
        low = torch.linalg.cholesky(a[:, :case["n"]])
        a[:, :case["n"]] = low + torch.tril(low, -1).T
        return a
    if kind in ("sweeps", "forces"):
        rng = np.random.default_rng(seed)
        rest, tets, region, dirichlet, _ = _slab(case)
        model = _Elastic(rest, tets, region, dirichlet)
        X = to(_deformed(rest, dirichlet, rng))
        f = model.forces(X, model.alpha)
        if kind == "forces":
            return {"f": _flat(f)}
        d2 = torch.zeros_like(X)
        d2[model.region] = to(0.01 * rng.standard_normal((3, model.region.numel())))
        none = (torch.zeros(0, 1, dtype=torch.long, device=DEV),
                torch.zeros(0, 1, dtype=torch.float64, device=DEV),
                torch.zeros(0, dtype=torch.float64, device=DEV))
        model.free[model.region] = False                     # solves with the interior block
        w = model.solve(f, none)
        y2 = (f - model.Kfull @ w)[model.region]
        w = model.solve(f - model.Kfull @ d2, none)
        return {"y2": _flat(y2), "x": _flat(X + w + d2)}
    if kind == "contact":
        return _exact_contact(case, seed)
    # the network in float64 on the same parameters
    p = [q.double() for q in _net_params(case, seed)]
    X, Y = (t.double() for t in _net_data(
        case, seed, case["batch"] * (1 if kind == "infer" else min(case["steps"], 4))))
    if kind == "infer":
        return _net(p, X)[2]
    b, parts = case["batch"], X.shape[0] // case["batch"]
    m1, m2 = [torch.zeros_like(q) for q in p], [torch.zeros_like(q) for q in p]
    for k in range(case["steps"]):
        j = b * (k % parts)
        g = _net_gradients(p, X[j:j + b], Y[j:j + b])
        for q, gq, a, v in zip(p, g, m1, m2):
            a.mul_(0.9).add_(gq, alpha=0.1)
            v.mul_(0.999).addcmul_(gq, gq, value=0.001)
            q.sub_(RATE * (a / (1 - 0.9 ** (k + 1)))
                   / ((v / (1 - 0.999 ** (k + 1))).sqrt() + 1e-8))
    return torch.cat([q.reshape(-1) for q in p])


def _net(p, X):
    h1 = torch.relu(X @ p[0].T + p[1])
    h2 = torch.relu(h1 @ p[2].T + p[3])
    return h1, h2, h2 @ p[4].T + p[5]


def _net_gradients(p, X, Y):
    h1, h2, out = _net(p, X)
    dy = (out - Y) / Y.numel()
    d2 = (dy @ p[4]) * (h2 > 0)
    d1 = (d2 @ p[2]) * (h1 > 0)
    return [d1.T @ X, d1.sum(0), d2.T @ h1, d2.sum(0), dy.T @ h2, dy.sum(0)]


def _exact_contact(case, seed):
    """Which proxies are in contact and the contact forces, by scanning every
    candidate; the row layout (which of several equal tets names a point) has
    no value of its own."""
    sc, bd, cand, rest2, x2 = _contact_inputs(case, seed)
    R, X = torch.tensor(rest2.T.copy(), device=DEV), torch.tensor(x2.T.copy(), device=DEV)
    tets = torch.tensor(cand.T.copy(), device=DEV).long()
    body = torch.tensor(bd.body_id, device=DEV)
    phi = torch.tensor(bd.body_phi.T.copy(), device=DEV)
    pts = torch.tensor(bd.proxy_points.T.copy(), device=DEV)
    pbody = torch.tensor(bd.proxy_body, device=DEV)

    def locate(pos, p, sel, skip=None):
        """Lowest of the candidates sel that holds each point (-1: none), weights."""
        v = pos[tets[sel]]
        inv = _inv3((v[:, 1:] - v[:, :1]).transpose(1, 2))[0]
        found = torch.full((p.shape[0],), -1, dtype=torch.long, device=DEV)
        wt = torch.zeros(p.shape[0], 4, dtype=torch.float64, device=DEV)
        for a in range(0, p.shape[0], 512):
            l = torch.einsum("tij,ptj->pti", inv, p[a:a + 512, None, :] - v[None, :, 0])
            lam = torch.cat([1.0 - l.sum(2, keepdim=True), l], 2)
            ok = (lam >= -1e-12).all(2)
            if skip is not None:
                own = skip[a:a + 512]
                ok &= ~(tets[sel][None, :, :, None] == own[:, None, None, :]).any(3).any(2)
            last = ok.shape[1]
            first = torch.where(ok, torch.arange(last, device=DEV), last).amin(1)
            found[a:a + 512] = torch.where(first < last, first, -1)
            wt[a:a + 512] = lam[torch.arange(lam.shape[0], device=DEV), first.clamp_max(last - 1)]
        return found, wt

    c = torch.zeros(pts.shape[0], dtype=torch.float64, device=DEV)
    f = torch.zeros_like(X)
    for b in (0, 1):
        mine, other = (body == b).nonzero()[:, 0], (body == 1 - b).nonzero()[:, 0]
        who = (pbody == b).nonzero()[:, 0]
        e, we = locate(R, pts[who], mine)
        pn = tets[mine[e]]
        p = (we[:, :, None] * X[pn]).sum(1)
        t, wt = locate(X, p, other, pn)
        inside = t >= 0
        who, pn, we, t, wt = who[inside], pn[inside], we[inside], other[t[inside]], wt[inside]
        val = (wt * phi[t]).sum(1)
        v = R[tets[t]]
        inv = _inv3((v[:, 1:] - v[:, :1]).transpose(1, 2))[0]
        grad = ((phi[t][:, 1:] - phi[t][:, :1])[:, :, None] * inv).sum(1)
        surf = (wt[:, :, None] * v).sum(1) - val[:, None] * grad / (grad * grad).sum(1, keepdim=True)
        u, wu = locate(R, surf, other, pn)
        hit = (val < 0) & (u >= 0)
        who, pn, we, wu = who[hit], pn[hit], we[hit], wu[hit]
        un = tets[other[u[hit]]]
        c[who] = K_LIP
        q = K_LIP * ((we[:, :, None] * X[pn]).sum(1) - (wu[:, :, None] * X[un]).sum(1))
        f.index_add_(0, pn.reshape(-1), -(we[:, :, None] * q[:, None, :]).reshape(-1, 3))
        f.index_add_(0, un.reshape(-1), (wu[:, :, None] * q[:, None, :]).reshape(-1, 3))
    return {"c": c, "fcol": _flat(f)}
