// Task schedules of the single-launch dataflow Cholesky: the ticket -> tile
// mappings (one tile per task in the low-precision kernel, one or two in the FP64
// kernel), the accumulation depth of a task, and where its flags and partial
// sums lie.  Host and device: the kernels decode their tickets with it, the
// workspaces are sized by it, and the library exports it (pd_factor_schedule,
// pd_dataflow_task) so that the host can check every task against the buffers.
#pragma once
#include <hip/hip_runtime.h>

namespace pdk {

// Ticket q -> tile (i, j), 0 <= j <= i < nt, i == nt for the right-hand-side
// row.  Tickets go column by column; in column j the diagonal tile first,
// then the tiles below it in order, then (rhs = 1) the right-hand-side row.
__host__ __device__ inline void df_task_of_ticket(int q, int nt, int rhs, int& i, int& j) {
  int jj = 0, start = 0;
  while (start + (nt - jj + rhs) <= q) start += nt - jj++ + rhs;
  j = jj;
  i = jj + (q - start);
}

// Number of tasks: nt (nt + 1) / 2 tiles, plus nt with a right-hand side.
__host__ __device__ inline int df_task_count(int nt, int rhs) { return nt * (nt + 1) / 2 + rhs * nt; }

// 64-column steps summed for tile (i, j) before its own last step: k < j, and
// k < j - 1 for the diagonal tile (its last step, with the tile left of it, is
// part of the tile factor).
__host__ __device__ inline int df_task_kend(int i, int j) {
  return i == j ? (j > 0 ? j - 1 : 0) : j;
}

// Of these, the steps that the FP64 kernel's task (i, j) accumulates from
// published tiles (nt: the right-hand-side row): k < j - 2 for the diagonal
// task and the partial sum left of it, k < j for every other one (the diagonal
// task adds the step k = j - 2 from its own registers).
__host__ __device__ inline int df_acc_steps(int i, int j, int nt) {
  const int steps = i == nt || i > j + 1 ? j : (i == j + 1 ? j - 1 : j - 2);
  return steps > 0 ? steps : 0;
}

// Partial sums: tile (j + 1, j) in slot j + 1, tile (j + 2, j) in slot nt + j + 2
// (-1: the task leaves none).  The low-precision kernel has the first kind only.
// Flags: nt x nt for the tiles, nt for the right-hand-side row's, then one per slot.
__host__ __device__ constexpr int df_part_slot(int i, int j, int nt) {
  return i == nt ? -1 : i == j + 1 ? i : i == j + 2 ? nt + i : -1;
}
__host__ __device__ constexpr int df_part_flag(int slot, int nt) { return (nt + 1) * nt + slot; }
__host__ __device__ constexpr int64_t df_slots(int64_t nt) { return 2 * nt; }
__host__ __device__ constexpr int64_t df_flags(int64_t nt) { return (nt + 1) * nt + df_slots(nt); }

// Tickets of the FP64 kernel.  With wide = 0, those above.  With wide = 1 they
// go by pairs of tile columns (j0, j0 + 1), j0 even: the diagonal task
// (j0, j0), (j0 + 1 .. j0 + 3, j0), the diagonal task (j0 + 1, j0 + 1),
// (j0 + 2 and j0 + 3, j0 + 1), then every row below as one task of the two
// tiles (i, j0) and (i, j0 + 1), then (rhs = 1) the right-hand-side row's two
// tiles, one task each.  cols: tiles of the task, (i, j) the first.
struct DfTask {
  int i, j, cols;
};
struct DfPair {
  int h0, h1, nw, nr;                // tasks of each kind, in this order
  __host__ __device__ DfPair(int j0, int nt, int rhs) {
    const int below = nt - j0;
    h0 = below < 4 ? below : 4;
    h1 = below - 1 < 3 ? (below > 1 ? below - 1 : 0) : 3;
    nw = below > 4 ? below - 4 : 0;
    nr = rhs * (below > 1 ? 2 : 1);
  }
  __host__ __device__ int count() const { return h0 + h1 + nw + nr; }
};
__host__ __device__ inline int df64_task_count(int nt, int wide, int rhs) {
  if (!wide) return df_task_count(nt, rhs);
  int n = 0;
  for (int j0 = 0; j0 < nt; j0 += 2) n += DfPair(j0, nt, rhs).count();
  return n;
}
__host__ __device__ inline DfTask df64_task(int q, int nt, int wide, int rhs) {
  if (!wide) {
    DfTask t{0, 0, 1};
    df_task_of_ticket(q, nt, rhs, t.i, t.j);
    return t;
  }
  int j0 = 0;
  DfPair p(0, nt, rhs);
  while (q >= p.count()) {
    q -= p.count();
    j0 += 2;
    p = DfPair(j0, nt, rhs);
  }
  if (q < p.h0) return {j0 + q, j0, 1};
  q -= p.h0;
  if (q < p.h1) return {j0 + 1 + q, j0 + 1, 1};
  q -= p.h1;
  if (q < p.nw) return {j0 + 4 + q, j0, 2};
  return {nt, j0 + q - p.nw, 1};
}
// The q-th tile in ticket order (a ticket of two tiles counts twice).
__host__ __device__ inline void df64_tile(int64_t q, int nt, int wide, int rhs, int& i, int& j) {
  int ticket = 0;
  if (!wide) {
    df_task_of_ticket((int)q, nt, rhs, i, j);
    return;
  }
  for (int j0 = 0;; j0 += 2) {
    const DfPair p(j0, nt, rhs);
    const int single = p.h0 + p.h1;
    if (q < p.count() + p.nw) {
      const bool two = q >= single && q < single + 2 * p.nw;
      const int64_t r = two ? single + (q - single) / 2 : (q < single ? q : q - p.nw);
      const DfTask t = df64_task(ticket + (int)r, nt, wide, rhs);
      i = t.i;
      j = t.j + (two ? (int)((q - single) % 2) : 0);
      return;
    }
    q -= p.count() + p.nw;
    ticket += p.count();
  }
}
// Two tiles per task from 160 tile columns on: the products then run at 58
// instead of 53 TFLOP/s, and there are enough tasks that the longer ones do not
// leave workgroups idle at the end.  Measured, one tile / two tiles:
// n = 6,498 2.28 / 2.36 ms, 9,728 6.40 / 6.46 ms, 12,155 12.5 / 12.1 ms,
// 19,494 54.6 / 48.5 ms.
__host__ __device__ inline int df64_wide(int nt) { return nt >= 160; }

}  // namespace pdk
