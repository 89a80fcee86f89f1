"""The FP64 Cholesky at the places where its 16 x 16 diagonal blocks and its
64 x 64 tiles meet: pivots that are not positive in every block of a tile, and
orders around the block, tile and tile-pair edges (pd_chol_factor), against an
elimination pivot by pivot on the CPU."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def eliminate(a):
    """Column by column L with the reciprocal square root of a non-positive
    pivot taken as 1, and the 1-based index of the first such pivot (0: none)."""
    a = np.tril(a).copy()
    n, bad = a.shape[0], 0
    for c in range(n):
        d = a[c, c]
        if not d > 0.0 and bad == 0:
            bad = c + 1
        a[c:, c] *= 1.0 / np.sqrt(d) if d > 0.0 else 1.0
        a[c + 1:, c + 1:] -= np.tril(np.outer(a[c + 1:, c], a[c + 1:, c]))
    return a, bad


def factor(a, lda):
    import torch
    from paper_2008_01541_amd import DenseCholesky
    n = a.shape[0]
    buf = np.full((n, lda), np.nan)
    buf[:, :n] = a.T
    dA = torch.tensor(buf.reshape(-1), device="cuda")
    chol = DenseCholesky(n)
    info = chol.factor(dA, n, lda)
    chol.close()
    out = dA.cpu().numpy().reshape(n, lda)
    assert np.isnan(out[:, n:]).all()
    lo, up = np.tril(out[:, :n].T), np.triu(out[:, :n].T, 1)
    assert np.array_equal(up, np.triu(lo.T, 1))
    return lo, info


# rounding: n products per element of a matrix with entries of order 1
def close(lo, ref, n):
    return np.abs(lo - ref).max() <= 64 * n * np.finfo(float).eps * max(1.0, np.abs(ref).max())


@pytest.mark.parametrize("bad", [0, 15, 16, 30, 33, 47, 48, 63, 64, 79, 127, 130, 149])
@pytest.mark.parametrize("value", [-1.0, 0.0])
def test_bad_pivot_in_every_block(bad, value):
    n, lda = 150, 160
    rng = np.random.default_rng(bad)
    a = 0.02 * rng.uniform(-1.0, 1.0, (n, n))
    a = np.tril(a) + np.tril(a, -1).T + 4.0 * np.eye(n)
    a[bad, bad] = value                # later pivots keep their sign
    a[bad, :bad] *= 1e-3
    a[:bad, bad] = a[bad, :bad]
    ref, first = eliminate(a)
    assert first == bad + 1
    lo, info = factor(a, lda)
    assert info == bad + 1
    assert close(lo, ref, n)


@pytest.mark.parametrize("n", [2, 15, 16, 17, 31, 49, 127, 128, 129, 191, 193, 257, 321, 385, 449])
def test_orders_around_the_edges(n):
    rng = np.random.default_rng(n)
    g = rng.uniform(-1.0, 1.0, (n, n))
    a = np.tril(g) + np.tril(g, -1).T + n * np.eye(n)
    lo, info = factor(a, (n + 15) // 16 * 16)
    assert info == 0
    assert close(lo, np.linalg.cholesky(a), n)


@pytest.mark.parametrize("n", [10177, 10240, 10300])
def test_two_tile_tasks(n):
    """Orders from which a task holds two tiles of a row (160 tile columns on;
    even and odd counts, ragged last tile) against torch on the device."""
    import torch
    from paper_2008_01541_amd import DenseCholesky
    lda = (n + 15) // 16 * 16
    g = torch.Generator(device="cuda").manual_seed(n)
    a = torch.rand(n, n, dtype=torch.float64, device="cuda", generator=g) - 0.5
    a = torch.tril(a) + torch.tril(a, -1).T
    a.diagonal().add_(0.5 * n)
    buf = torch.full((n, lda), float("nan"), dtype=torch.float64, device="cuda")
    buf[:, :n] = a
    chol = DenseCholesky(n)
    assert chol.factor(buf.view(-1), n, lda) == 0
    chol.close()
    ref = torch.linalg.cholesky(a)
    lo = torch.tril(buf[:, :n].T)
    assert torch.equal(torch.triu(buf[:, :n].T, 1), torch.tril(lo, -1).T)
    eps = torch.finfo(torch.float64).eps
    assert float((lo - ref).abs().max()) <= 64 * n * eps * float(ref.abs().max())
