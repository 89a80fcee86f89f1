// Device-side building blocks shared by the dataflow Cholesky kernels: the
// factor and inverse of a 64 x 64 diagonal tile held in LDS (FP64, matrix
// cores for the blocked updates, DPP row broadcasts for the 16 x 16 diagonal
// blocks), and the per-compute-unit marks by which tasks off the critical
// path yield to the diagonal task.  Header-only: included by each kernel file.
#pragma once
#include "common.h"
#include "publish.h"

namespace pdk {

constexpr int LDS_LD = NB + 4;   // padded LDS row (doubles)

// chol16_eliminate(a, x): the scheduled elimination of a 16 x 16 block.
#include "chol16_steps.inc"

// 1/sqrt(d): the hardware estimate (relative error up to about 5e-8 on this
// chip) refined by one third-order step, y <- y (1 + e/2 + 3 e^2/8) with
// e = 1 - d y^2: four dependent operations for an error of about 2.4 ulp (two
// Newton steps reach the same accuracy in six).
__device__ __forceinline__ double rsqrt_newton(double d) {
  const double y = __builtin_amdgcn_rsq(d);
  const double e = fma(-(d * y), y, 1.0);
  return fma(y * e, fma(0.375, e, 0.5), y);
}

// One block column of the tile factor, by one wave: the 16 x 16 diagonal block
// at (b0, b0), b0 = 16 KB, is factored and 64 further rows are solved against
// it, one per lane of the four rows of 16 lanes:
//   lanes 0-15            the rows of dinv, which hold the identity and become
//                         the block's inverse;
//   the next 3 - KB rows  the panel blocks below (rows b0 + lane), which become
//                         P L_kk^-T;
//   the last KB rows      the columns of the staged -Y_kj, j < KB, which become
//                         X_kj = -L_kk^-1 Y_kj.
// All rows of 16 lanes hold the block itself (lane r row r), since the
// multipliers are broadcast within a row of 16 lanes; the riding rows use the
// issue slots that the block's own pivot chain leaves.  Instruction issue
// bounds it (386 FP64 instructions of 4 cycles and 16 square roots of 16; the
// chain of square root, scaling, update and broadcast is 92 cycles a pivot):
// 1,950 cycles measured for the elimination, 2,700 with the loads and stores
// (3,580 before the steps were scheduled across pivots, and the panel below
// and the inverse's off-diagonal blocks then took products of their own).
// dinv: rows of the block's inverse (dinv[c][b0 + r] = inverse(r, c)).
__device__ __forceinline__ double* chol16_row(double (*T)[LDS_LD], double (*X)[LDS_LD], int kb,
                                              double (*dinv)[LDS_LD], int& ld) {
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4, b0 = 16 * kb;
  const bool panel = g >= 1 && g <= 3 - kb;
  const int col = 16 * (g - 4 + kb) + r;           // column of the inverse, g > 3 - kb
  ld = panel ? LDS_LD : 1;
  return g == 0 ? &dinv[r][b0] : (panel ? &T[b0][b0 + lane] : &X[col][b0]);
}

// The same elimination step by step in LDS, for a block with a pivot that is
// not positive (never on the path of a positive definite matrix): the pivot's
// reciprocal square root is taken as 1 and the first one, if inside the first
// mr rows, is reported in *info as gbase + its index + 1.
__device__ __forceinline__ void chol16_bad_block(double (*T)[LDS_LD], double (*X)[LDS_LD], int kb,
                                                 double (*dinv)[LDS_LD], int mr, int gbase,
                                                 int* info) {
  const int lane = threadIdx.x & 63, r = lane & 15, b0 = 16 * kb;
  int ld, bad = 0;
  double* p = chol16_row(T, X, kb, dinv, ld);
#pragma unroll 1
  for (int c = 0; c < 16; ++c) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const double d = T[b0 + c][b0 + c];
    const bool ok = d > 0.0;
    if (!ok && bad == 0) bad = c + 1;
    const double y = ok ? rsqrt_newton(d) : 1.0;
    __builtin_amdgcn_wave_barrier();
    if (lane < 16) T[b0 + c][b0 + r] *= y;
    p[c * ld] *= y;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll 1
    for (int s = c + 1; s < 16; ++s) {
      const double l = T[b0 + c][b0 + s];
      if (lane < 16) T[b0 + s][b0 + r] -= l * T[b0 + c][b0 + r];
      p[s * ld] -= l * p[c * ld];
    }
    __builtin_amdgcn_wave_barrier();
  }
  if (lane == 0 && bad > 0 && b0 + bad - 1 < mr) atomicCAS(info, 0, gbase + b0 + bad);
}

__device__ __forceinline__ void chol16_block(double (*T)[LDS_LD], double (*X)[LDS_LD], int kb,
                                             double (*dinv)[LDS_LD], int mr, int gbase,
                                             int* info) {
  const int lane = threadIdx.x & 63, r = lane & 15, b0 = 16 * kb;
  int ld;
  double* p = chol16_row(T, X, kb, dinv, ld);
  double a[16], x[16];
#pragma unroll
  for (int c = 0; c < 16; ++c) a[c] = T[b0 + c][b0 + r];
#pragma unroll
  for (int c = 0; c < 16; ++c) x[c] = p[c * ld];
  const double last = chol16_eliminate(a, x);
  // a pivot that is not positive makes every later one a NaN
  if (!(__builtin_amdgcn_readfirstlane((int)(last > 0.0)))) {
    chol16_bad_block(T, X, kb, dinv, mr, gbase, info);
    return;
  }
  // (above its diagonal the block keeps values that nothing reads)
  if (lane < 16) {
#pragma unroll
    for (int c = 0; c < 16; ++c) T[b0 + c][b0 + r] = a[c];
  }
#pragma unroll
  for (int c = 0; c < 16; ++c) p[c * ld] = x[c];
}

// C(m, n) += sum_k A(m, k) B(n, k) over one 16-deep block, m, n, k < 16, for
// operands in LDS tiles (Ts[c][r] = tile(r, c)): A(m, k) = As[ak + k][am + m],
// B(n, k) = Bs[bk + k][bn + n] (BT = false) or Bs[bn + n][bk + k] (BT = true).
// Result: lane l, register q holds C(l % 16, l / 16 + 4 q).
template <bool BT>
__device__ inline void mma16(double4_t& acc, double (*As)[LDS_LD], int am, int ak,
                             double (*Bs)[LDS_LD], int bn, int bk) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int k = 4 * s + (lane >> 4);
    const double av = As[ak + k][am + (lane & 15)];
    const double bv = BT ? Bs[bn + (lane & 15)][bk + k] : Bs[bk + k][bn + (lane & 15)];
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(bv, av, acc, 0, 0, 0);
  }
}

// Cholesky of a 64 x 64 tile held in LDS (T[c][r] = tile(r, c), lower part
// valid, rows/cols >= mr padded with the identity) and the inverse of the
// factor into X (X[c][r] = inverse(r, c), zero above the diagonal).  Right-
// looking over 16-wide block columns.  In step kb wave 0 factors the diagonal
// block together with its inverse, the panel blocks below it and the finished
// part of the inverse's block row kb (chol16_block); then the four waves form,
// one block each on the matrix cores, what the next step reads: the trailing
// blocks (i, kb + 1) and the staged blocks -Y_{kb+1,j} -= L_{kb+1,kb} X_kj,
// j <= kb (-Y_ij, Y_ij = sum_{p=j}^{i-1} L_ip X_pj, waits in the X_ij slot).  The
// blocks that later steps read are updated by waves 1-3 while wave 0 is in
// its next step.  6.1 us per tile, 6.9 us with the update by B below (8.7 and
// 9.3 us when the panels and the inverse's rows were products between the
// blocks).  A non-positive pivot stores its 1-based global index
// gbase + j + 1 in *info (first one wins) and its reciprocal square root is
// taken as 1 so that the factorization stays finite.  Only the lower triangle
// of T is meaningful on return.
//
// With lflag != NULL, X enters holding a 64 x 64 tile B (X[k][r] = B(r, k))
// and the tile factored is T - B B^T: the waves subtract B B^T from the first
// block column, one block each, and while wave 0 factors it waves 1-3 update
// the six other lower blocks; once B has been read by every wave,
// *lflag = epoch is published (after this workgroup's earlier global stores
// have drained) and X is reused for the inverse.
__device__ __forceinline__ void factor_tile_blocked(double (*T)[LDS_LD], double (*X)[LDS_LD], int mr, int gbase,
                                    int* info, int* lflag = nullptr, int epoch = 0) {
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  // zero the six strictly upper 16 x 16 blocks of X, X[16 jb + c][16 ib + r],
  // ib < jb, and put the identity into the diagonal blocks from kb0 on
  const auto clear_x = [&](int kb0) {
    for (int kb = kb0; kb < 4; ++kb)
      X[16 * kb + (t >> 4)][16 * kb + (t & 15)] = (t >> 4) == (t & 15) ? 1.0 : 0.0;
    for (int e = t; e < 6 * 256; e += 256) {
      const int blk = e >> 8, r = e & 15, c = (e >> 4) & 15;
      const int ib = blk < 3 ? 0 : (blk < 5 ? 1 : 2);
      const int jb = blk < 3 ? blk + 1 : (blk < 5 ? blk - 1 : 3);
      X[16 * jb + c][16 * ib + r] = 0.0;
    }
  };
  // block (i, j) of D, D[16 j + c][16 i + r], minus the product acc
  const auto subtract = [&](double (*D)[LDS_LD], int i, int j, auto product) {
    double v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = D[16 * j + (lane >> 4) + 4 * q][16 * i + (lane & 15)];
    double4_t acc = {0.0, 0.0, 0.0, 0.0};
    product(acc);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      D[16 * j + (lane >> 4) + 4 * q][16 * i + (lane & 15)] = v[q] - acc[q];
  };
  // T block (i, j) -= L_ik L_jk^T
  const auto trail = [&](int i, int j, int k) {
    subtract(T, i, j, [&](double4_t& acc) { mma16<false>(acc, T, 16 * i, 16 * k, T, 16 * j, 16 * k); });
  };
  // -Y_ij -= L_ik X_kj for j < k, and -Y_ik = -L_ik X_kk (X_kk read from dinv)
  const auto stage = [&](int i, int j, int k, double (*dinv)[LDS_LD]) {
    if (j < k) {
      subtract(X, i, j, [&](double4_t& acc) { mma16<true>(acc, T, 16 * i, 16 * k, X, 16 * j, 16 * k); });
    } else {
      double4_t acc = {0.0, 0.0, 0.0, 0.0};
      mma16<true>(acc, T, 16 * i, 16 * k, dinv, 0, 16 * k);
#pragma unroll
      for (int q = 0; q < 4; ++q) X[16 * j + (lane >> 4) + 4 * q][16 * i + (lane & 15)] = -acc[q];
    }
  };
  // what step kb + 1 reads, one block per wave
  const auto next_column = [&](int kb, double (*dinv)[LDS_LD]) {
    if (w < 3 - kb) trail(kb + 1 + w, kb + 1, kb);
    else stage(kb + 1, w - (3 - kb), kb, dinv);
  };
  // T block (ib, jb) -= sum_{k < 64} B(16 ib + m, k) B(16 jb + n, k)
  const auto b_update = [&](int ib, int jb) {
    subtract(T, ib, jb, [&](double4_t& acc) {
#pragma unroll
      for (int s = 0; s < 4; ++s) mma16<false>(acc, X, 16 * ib, 16 * s, X, 16 * jb, 16 * s);
    });
  };
  // while X holds B, the first inverse block takes the unused upper block
  // (0, 1) of T, in the layout of X (T[16 + c][r] = inverse(r, c))
  double (*dinv)[LDS_LD] = lflag ? T + 16 : X;
  if (lflag) {
    T[16 + (t >> 4)][t & 15] = (t >> 4) == (t & 15) ? 1.0 : 0.0;
    b_update(w, 0);
  } else {
    clear_x(0);
  }
  __syncthreads();
  // unrolled: with kb a run-time value the block addresses cost 1 us per tile,
  // more than the fetch of the longer code when it is not cached
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) {
    if (w == 0) {
      chol16_block(T, X, kb, dinv, mr, gbase, info);
    } else if (kb == 0) {
      if (lflag) {
        // (1,1) (2,1) | (3,1) (2,2) | (3,2) (3,3)
        for (int u = 0; u < 2; ++u)
          b_update(u == 0 ? (w == 1 ? 1 : 3) : (w == 3 ? 3 : 2), u == 0 ? (w == 3 ? 2 : 1) : w);
      }
    } else if (kb == 1) {
      trail(w < 3 ? 1 + w : 3, w < 3 ? 2 : 3, 0);
      if (w < 3) stage(1 + w, 0, 0, X);
    } else if (kb == 2) {
      if (w == 1) trail(3, 3, 1);
      else stage(3, w - 2, 1, X + 16);
    }
    if (kb == 0 && lflag) {
      publish_flag(lflag, epoch);           // B read by every wave: X is free
      clear_x(1);
      X[t >> 4][t & 15] = T[16 + (t >> 4)][t & 15];   // X_00 (256 threads, one element each)
    } else {
      __syncthreads();
    }
    if (kb == 3) break;
    next_column(kb, dinv);
    __syncthreads();
    dinv = X + 16 * (kb + 1);
  }
}

// Compute-unit courtesy.  The diagonal tasks form the critical path of the
// factorization; their local phase (finishing the sub-diagonal tile, the tile
// factor, the inverse) runs on one compute unit and, with two workgroups per
// unit, shares its FP64 pipes with the other one's products.  A diagonal task
// marks its unit busy (slot cu_slot(), value = launch epoch) for that phase;
// tasks off the critical path that find their unit marked sleep at their next
// k-step until the mark is cleared.  The diagonal task waits for nothing while
// marked, so the pause is short; it is bounded anyway, and the marks only
// steer timing, never results.
constexpr int CU_SLOTS = 2048;
__device__ inline int cu_slot() {
  const unsigned hw = __builtin_amdgcn_s_getreg((31 << 11) | 4);    // HW_ID: SE, SH, CU in bits 15:8
  const unsigned xcc = __builtin_amdgcn_s_getreg((31 << 11) | 20);  // XCC_ID
  return (int)(((xcc & 7u) << 8) | ((hw >> 8) & 0xffu));
}
__device__ inline void cu_pause(const int* mark, int epoch) {
  for (int s = 0; s < 4096; ++s) {                                   // at most ~0.5 ms
    __builtin_amdgcn_s_sleep(8);
    if (__hip_atomic_load(mark, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != epoch) return;
  }
}

}  // namespace pdk
