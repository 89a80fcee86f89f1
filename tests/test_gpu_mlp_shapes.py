"""The warm-start network's kernels at the edges of their tiles (16 rows of a
batch, 16 outputs, 32 inputs, splits of 256 inputs and more than four of them)
against the oracle with the same BF16 rounding points."""
import numpy as np
import pytest

from oracle import mlp as omlp
from pd_inputs.mlp_init import mlp_init_params, pack, unpack
from gpu_util import dev, host

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return np.linalg.norm(np.asarray(a) - np.asarray(b)) / max(np.linalg.norm(b), 1e-300)


@pytest.mark.parametrize("shape,B", [((41, 17, 50, 29), 1), ((33, 16, 15, 3), 16),
                                     ((1500, 64, 129, 1400), 17), ((520, 500, 500, 61), 33),
                                     ((3001, 31, 33, 65), 32)])
def test_forward_gradients_and_step(shape, B):
    import torch
    from paper_2008_01541_amd import MLP
    p = mlp_init_params(*shape, seed=B)
    rng = np.random.default_rng(B + 1)
    for k in ["b1", "b2", "b3"]:
        p[k] = 0.05 * rng.normal(size=p[k].shape)
    flat = pack(p)
    p_or = unpack(flat, *shape)
    X = rng.normal(size=(B, shape[0])).astype(np.float32)
    T = rng.normal(size=(B, shape[3])).astype(np.float32)
    net = MLP(*shape, max_batch=40, params_flat=flat)
    y = torch.empty(B * shape[3], dtype=torch.float32, device="cuda")
    net.forward(dev(X), y)
    Y, cache = omlp.forward(p_or, X.astype(np.float64))
    # FP32 sums against FP64 ones, with the odd BF16 rounding that goes the other way
    assert _rel(host(y, (B, shape[3])), Y) <= 1e-3
    g, _ = net.gradients(dev(X), dev(T))
    gd, g_or = unpack(g, *shape), omlp.backward(p_or, cache, Y, T.astype(np.float64))
    for k in g_or:
        assert _rel(gd[k], g_or[k]) <= 5e-3, k
    # the fused update from the gradients that the library itself reports: one
    # Adam step is lr g / (|g| + eps) for the first step
    net.train_step(dev(X), dev(T), lr=1e-3, want_loss=False)
    got = net.params().astype(np.float64)
    g64 = g.astype(np.float64)
    upd = 1e-3 * g64 / (np.abs(g64) + 1e-8)
    ref = flat.astype(np.float64) - upd
    # FP32 rounding of the weight (1 ulp) and of the normalised step (a few ulp)
    assert np.abs(got - ref).max() <= 2.0 ** -23 * np.abs(ref).max() + 1e-3 * 2.0 ** -18
