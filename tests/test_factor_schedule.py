"""Ticket order of the FP64 factorization where a task may hold two tiles of a
row (from 160 tile columns on): every tile once, and every tile's operands
given out before it, so that a persistent launch cannot deadlock (host only)."""
import numpy as np
import pytest

from test_kernel_bounds import schedule


@pytest.mark.parametrize("nt", [159, 160, 161])
@pytest.mark.parametrize("rhs", [0, 1])
def test_two_tile_order_respects_dependencies(nt, rhs):
    sched = schedule(64 * nt - 5, rhs)
    pos = np.full((nt + 1, nt), -1)
    for q, (i, j, _) in enumerate(sched):
        assert pos[i, j] < 0
        pos[i, j] = q
    assert (pos >= 0).sum() == len(sched) == nt * (nt + 1) // 2 + rhs * nt
    # the two tiles left of a diagonal are published by the diagonal's task
    made = pos.copy()
    for j in range(nt):
        for c in range(max(j - 2, 0), j):
            made[j, c] = pos[j, j]
    for q, (i, j, kend) in enumerate(sched):
        part = i != nt and i in (j + 1, j + 2)
        steps = kend if i != j and not part else max(min(kend, i - 2), 0)
        first = pos[i, j - 1] if j % 2 and not part and i != j and pos[i, j] == pos[i, j - 1] + 1 else q
        assert (made[i, :steps] < q).all()
        assert i == j or (made[j, :steps] < max(q, first)).all()
        assert part or i == j or pos[j, j] < q
        if i == j and j > 0:
            assert pos[j - 1, j - 1] < q and (pos[j, max(j - 2, 0):j] < q).all()
