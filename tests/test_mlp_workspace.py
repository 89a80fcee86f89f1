"""Large batches of the warm-start network: the split sums of its products
stay inside the workspace (host only); a wide layer with more than 64 splits,
and more blocks of rows than a grid's y or z holds, against the oracle (GPU)."""
import ctypes as C

import numpy as np
import pytest

TILE, SPLIT_MIN, CHUNK = 64, 256, 32


def _workspace(shape, max_batch, batch):
    from paper_2008_01541_amd import load_library
    used, held = C.c_int64(), C.c_int64()
    assert load_library().pd_mlp_workspace(*shape, max_batch, batch, C.byref(used),
                                           C.byref(held)) == 0
    return used.value, held.value


def _splits(M, N, K):
    """Splits of an M x N product over K: at least 256 inner values each, and
    about two workgroups of a 64 x 64 tile per compute unit."""
    tiles = -(-M // TILE) * -(-N // TILE)
    s = min(max(1, 512 // tiles), max(1, K // SPLIT_MIN))
    ks = -(-(-(-K // s)) // CHUNK) * CHUNK
    return -(-K // ks)


def _written(shape, B):
    """Most floats a call with B rows writes: layers, backward products, gradients."""
    most = 0
    for i in range(3):
        k, n = shape[i], shape[i + 1]
        prods = [(B, n, k), (n, k, B)] + ([(B, k, n)] if i else [])
        most = max([most] + [_splits(*p) * p[0] * p[1] for p in prods])
    return most


SHAPES = [(26000, 16, 16, 3), (25992, 512, 512, 19494), (324, 128, 128, 243), (1, 1, 1, 1),
          (3, 2, 40000, 16), (16384, 1, 1, 1), (64, 64, 64, 64), (70000, 3, 130, 60000)]


@pytest.mark.parametrize("shape", SHAPES)
def test_split_sums_fit_the_workspace(shape):
    for max_batch in (1, 32, 64, 320, 700, 5000, 20000):
        batches = {b for b in (1, 16, 17, 32, 33, 63, 64, 65, 128, 320, 512, 513, 700, 1800, 4999,
                               5000, 16448, 20000) if b <= max_batch} | {max_batch}
        for b in sorted(batches):
            used, held = _workspace(shape, max_batch, b)
            assert used == _written(shape, b)
            assert used <= held, (shape, max_batch, b)


def test_workspace_rejects_bad_arguments():
    from paper_2008_01541_amd import load_library
    lib = load_library()
    u, h = C.c_int64(), C.c_int64()
    assert lib.pd_mlp_workspace(0, 1, 1, 1, 1, 1, C.byref(u), C.byref(h)) == -1
    assert lib.pd_mlp_workspace(1, 1, 1, 1, 4, 5, C.byref(u), C.byref(h)) == -1
    assert lib.pd_mlp_workspace(1, 1, 1, 1, 4, 4, None, C.byref(h)) == -1


@pytest.mark.gpu
def test_wide_input_of_many_splits():
    import torch
    from oracle import mlp as omlp
    from paper_2008_01541_amd import MLP
    from pd_inputs.mlp_init import mlp_init_params, pack, unpack
    shape, B = (26000, 16, 16, 3), 320
    assert _splits(B, 16, 26000) > 64
    flat = pack(mlp_init_params(*shape, seed=5))
    rng = np.random.default_rng(6)
    X = rng.normal(size=(B, shape[0])).astype(np.float32)
    net = MLP(*shape, max_batch=B, params_flat=flat)
    y = torch.empty(B * shape[3], dtype=torch.float32, device="cuda")
    net.forward(torch.tensor(X.reshape(-1), device="cuda"), y)
    Y, _ = omlp.forward(unpack(flat, *shape), X.astype(np.float64))
    got = y.cpu().numpy().reshape(B, shape[3])
    # FP32 sums against FP64 ones, with the odd BF16 rounding that goes the other way
    assert np.linalg.norm(got - Y) <= 1e-3 * np.linalg.norm(Y)
    net.close()


@pytest.mark.gpu
def test_more_row_blocks_than_a_grid_dimension_holds():
    import torch
    from oracle import mlp as omlp
    from paper_2008_01541_amd import MLP
    from pd_inputs.mlp_init import mlp_init_params, pack, unpack
    shape, B = (3, 2, 2, 3), 65535 * 32 + 33
    flat = pack(mlp_init_params(*shape, seed=7))
    rng = np.random.default_rng(8)
    X = rng.normal(size=(B, 3)).astype(np.float32)
    T = rng.normal(size=(B, 3)).astype(np.float32)
    net = MLP(*shape, max_batch=B, params_flat=flat)
    x, y = torch.tensor(X.reshape(-1), device="cuda"), torch.empty(3 * B, device="cuda")
    net.forward(x, y)
    p = unpack(flat, *shape)
    Y, cache = omlp.forward(p, X.astype(np.float64))
    got = y.cpu().numpy().reshape(B, 3)
    assert np.linalg.norm(got - Y) <= 1e-3 * np.linalg.norm(Y)
    assert np.linalg.norm(got[-33:] - Y[-33:]) <= 1e-2 * np.linalg.norm(Y[-33:])
    # the backward products take the same grid
    g, _ = net.gradients(x, torch.tensor(T.reshape(-1), device="cuda"))
    gd, ref = unpack(g, *shape), omlp.backward(p, cache, Y, T.astype(np.float64))
    for k in ref:
        assert np.linalg.norm(gd[k] - ref[k]) <= 5e-3 * np.linalg.norm(ref[k]), k
    net.close()
