"""The tasks that the factorization kernels run (pd_factor_schedule, the code
the kernels decode their tickets with) against the workspace the library
allocates: every tile once, every step of every tile summed by somebody, flags
and partial sums in slots of their own, every address inside its array, and
nothing awaited that a later ticket publishes.  FP64 with one and two tiles per
task, and the low-precision kernel (host only)."""
import ctypes as C

import numpy as np
import pytest

NB = 64
FIELDS = ("i", "j", "tiles", "steps", "slot", "flag")


def _schedule(n, lp, rhs):
    from paper_2008_01541_amd import load_library
    lib = load_library()
    sizes, task = (C.c_int64 * 3)(), (C.c_int32 * 6)()
    assert lib.pd_factor_schedule(n, lp, rhs, -1, None, sizes) == 0
    out = np.empty((sizes[0], 6), dtype=np.int64)
    for q in range(sizes[0]):
        assert lib.pd_factor_schedule(n, lp, rhs, q, task, sizes) == 0
        out[q] = task[:]
    return out, sizes[1], sizes[2]


NS = [1, 17, 64, 65, 128, 129, 200, 257, 3249, 6498, 64 * 159, 64 * 160 - 5, 64 * 161 + 3]


@pytest.mark.parametrize("lp,rhs", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("n", NS)
def test_tasks_cover_the_matrix_and_fit_the_workspace(n, lp, rhs):
    nt, lda = -(-n // NB), -(-n // 16) * 16
    tasks, nflags, nslots = _schedule(n, lp, rhs)
    count = np.zeros((nt + 1, nt), dtype=int)
    flags, slots = [], []
    left = 1 if lp else 2                     # tiles left of a diagonal that its task finishes
    for i, j, tiles, steps, slot, flag in tasks:
        count[i, j:j + tiles] += 1
        flags += [i * nt + j + u for u in range(tiles)]
        assert tiles == 1 or (not lp and i < nt and j + 1 < i - 2)
        # steps: all earlier columns, less those that the diagonal task adds itself
        own = min(j, left) if i == j else min(j, left - (i - j)) if slot >= 0 else 0
        assert steps == j - own
        assert (slot >= 0) == (i < nt and 0 < i - j <= left)
        if slot >= 0:
            slots.append(slot)
            flags.append(flag)
        # addresses: a task's own tiles, the steps' operands (pairs of rows, the
        # last one past an odd edge), the transposed copies
        size, ld = (NB * n, NB) if i == nt else (lda * n, lda)
        r0, mr = (0, 3) if i == nt else (i * NB, min(NB, n - i * NB))
        c0, mc = j * NB, min(NB, n - j * NB)
        assert r0 + mr - 1 + (c0 + tiles * NB - NB + mc - 1) * ld < size
        if steps:
            pair = (mr - 1) // 2 * 2 + 1
            assert r0 + pair < ld and r0 + pair + (steps * NB - 1) * ld < size
            pair = (mc - 1) // 2 * 2 + 1
            assert c0 + pair < lda and c0 + pair + (steps * NB - 1) * lda < lda * n
        if i == j:
            for cj in range(max(j - left, 0), j):
                assert n - cj * NB >= NB       # a column block left of another is full
                assert cj * NB + NB - 1 + (r0 + mr - 1) * lda < lda * n
    assert (count[:nt] == np.tril(np.ones((nt, nt), dtype=int))).all()
    assert (count[nt] == rhs).all()
    assert len(set(flags)) == len(flags) and min(flags) >= 0 and max(flags) < nflags
    assert len(set(slots)) == len(slots) and max(slots, default=0) < nslots


@pytest.mark.parametrize("lp,rhs", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("n", NS)
def test_tasks_wait_for_smaller_tickets_only(n, lp, rhs):
    nt = -(-n // NB)
    tasks, _, _ = _schedule(n, lp, rhs)
    left = 1 if lp else 2
    made = np.full((nt + 1, nt), -1)           # the ticket that publishes a tile
    part = np.full((nt + 1, nt), -1)           # the ticket that leaves its partial sum
    for q, (i, j, tiles, steps, slot, flag) in enumerate(tasks):
        if slot >= 0:
            part[i, j] = q
        else:
            made[i, j:j + tiles] = q
        if i == j:
            made[i, max(j - left, 0):j] = q
    for q, (i, j, tiles, steps, slot, flag) in enumerate(tasks):
        assert (made[i, :steps] < q).all() and (made[j:j + tiles, :steps] < q).all()
        if i == j:
            for cj in range(max(j - left, 0), j):
                assert made[cj, cj] < q and part[j, cj] < q
            assert j < 2 or made[j - 1, j - 2] < q
        elif slot < 0:
            assert (np.diag(made)[j:j + tiles] < q).all()
            assert tiles == 1 or made[j + 1, j] < q


def test_schedule_rejects_bad_arguments():
    from paper_2008_01541_amd import load_library
    lib = load_library()
    sizes, task = (C.c_int64 * 3)(), (C.c_int32 * 6)()
    assert lib.pd_factor_schedule(0, 0, 0, 0, task, sizes) == -1
    assert lib.pd_factor_schedule(100, 2, 0, 0, task, sizes) == -1
    assert lib.pd_factor_schedule(100, 1, 1, 0, task, sizes) == -1
    assert lib.pd_factor_schedule(100, 0, 0, 3, task, sizes) == -1     # 2 tiles: 3 tickets
    assert lib.pd_factor_schedule(100, 0, 0, 0, task, None) == -1
    assert lib.pd_factor_schedule(100, 0, 0, 2, task, sizes) == 0
    assert dict(zip(FIELDS, task[:])) == dict(i=1, j=1, tiles=1, steps=0, slot=-1, flag=-1)
