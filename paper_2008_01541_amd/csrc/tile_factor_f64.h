// Device-side building blocks shared by the dataflow Cholesky kernels: the
// factor and inverse of a 64 x 64 diagonal tile held in LDS (FP64, matrix
// cores for the blocked updates, DPP row broadcasts for the 16 x 16 diagonal
// blocks), and the per-compute-unit marks by which tasks off the critical
// path yield to the diagonal task.  Header-only: included by each kernel file.
#pragma once
#include <type_traits>
#include "common.h"
#include "publish.h"

namespace pdk {

constexpr int LDS_LD = NB + 4;   // padded LDS row (doubles)
// offset of element (row r, column c) of an LDS tile Ts[c][r]
__device__ constexpr int lds_at(int c, int r) { return c * LDS_LD + r; }

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
                                              double (*dinv)[LDS_LD], int lane, int& ld) {
  const int r = lane & 15, g = lane >> 4, b0 = 16 * kb;
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
                                                 double (*dinv)[LDS_LD], int lane, int mr,
                                                 int gbase, int* info) {
  const int r = lane & 15, b0 = 16 * kb;
  int ld, bad = 0;
  double* p = chol16_row(T, X, kb, dinv, lane, ld);
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
                                             double (*dinv)[LDS_LD], int lane, int mr, int gbase,
                                             int* info) {
  const int b0 = 16 * kb;
  double* const d = &T[0][lane & 15];
  int ld;
  double* p = chol16_row(T, X, kb, dinv, lane, ld);
  double a[16], x[16];
#pragma unroll
  for (int c = 0; c < 16; ++c) a[c] = d[lds_at(b0 + c, b0)];
#pragma unroll
  for (int c = 0; c < 16; ++c) x[c] = p[c * ld];
  const double last = chol16_eliminate(a, x);
  // a pivot that is not positive makes every later one a NaN
  if (!(__builtin_amdgcn_readfirstlane((int)(last > 0.0)))) {
    chol16_bad_block(T, X, kb, dinv, lane, mr, gbase, info);
    return;
  }
  // (above its diagonal the block keeps values that nothing reads)
  if (lane < 16) {
#pragma unroll
    for (int c = 0; c < 16; ++c) d[lds_at(b0 + c, b0)] = a[c];
  }
#pragma unroll
  for (int c = 0; c < 16; ++c) p[c * ld] = x[c];
}

// C(m, n) += sum_k A(m, k) B(n, k) over one 16-deep block, m, n, k < 16, for
// operands in LDS tiles (Ts[c][r] = tile(r, c)): A(m, k) = As[ak + k][am + m],
// B(n, k) = Bs[bk + k][bn + n] (BT = false) or Bs[bn + n][bk + k] (BT = true).
// The lane's addresses are one base per tile and constants: a = lane_kn(As),
// b = lane_kn(Bs) or lane_nk(Bs), and the offsets lds_at(ak, am), lds_at(bk, bn)
// or lds_at(bn, bk).  Result: lane l, register q holds C(l % 16, l / 16 + 4 q),
// the address lane_kn(D) + lds_at(column0 + 4 q, row0) of a tile D.
__device__ __forceinline__ double* lane_kn(double (*S)[LDS_LD], int lane) {
  return &S[lane >> 4][lane & 15];
}
__device__ __forceinline__ double* lane_nk(double (*S)[LDS_LD], int lane) {
  return &S[lane & 15][lane >> 4];
}
template <bool BT>
__device__ __forceinline__ void mma16(double4_t& acc, const double* a, const double* b) {
#pragma unroll
  for (int s = 0; s < 4; ++s)
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(b[BT ? 4 * s : lds_at(4 * s, 0)], a[lds_at(4 * s, 0)],
                                               acc, 0, 0, 0);
}

// Cholesky of a 64 x 64 tile held in LDS (T[c][r] = tile(r, c), lower part
// valid, rows/cols >= mr padded with the identity) and the inverse of the
// factor into X (X[c][r] = inverse(r, c), zero above the diagonal unless it
// goes to pub.inv).  Right-
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
// With pub.lflag != NULL, X enters holding a 64 x 64 tile B (X[k][r] = B(r, k))
// and the tile factored is T - B B^T: the waves subtract B B^T from the first
// block column, one block each, and while wave 0 factors it waves 1-3 update
// the six other lower blocks and write the first lrows rows of B to pub.l;
// then X is reused for the inverse, and *lflag = epoch is published once those
// stores have drained (*pub.drained, in LDS and 0 on entry, counts the waves).  With
// pub.inv != NULL the inverse is written there (inv[64 c + r] = inverse(r, c)),
// a block row at a time while the next one is computed; its flag is the
// caller's to publish.
struct TilePublish {
  int* lflag = nullptr;
  int epoch = 0;
  double* l = nullptr;
  long ldl = 0;
  int lrows = 0;
  int* drained = nullptr;
  double* inv = nullptr;
};
__device__ __forceinline__ void factor_tile_blocked(double (*T)[LDS_LD], double (*X)[LDS_LD], int mr, int gbase,
                                    int* info, const TilePublish& pub) {
  const int t = task_tid(), lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  // the identity into the diagonal block kb of X, by all 256 threads or (tt =
  // t - 64) by the last 192
  const auto ident = [&](int kb, int tt, int nthr) {
    for (int e = tt; e < 256; e += nthr)
      X[16 * kb + (e >> 4)][16 * kb + (e & 15)] = (e >> 4) == (e & 15) ? 1.0 : 0.0;
  };
  double* const tk = lane_kn(T, lane);
  double* const xk = lane_kn(X, lane);
  double* const xn = lane_nk(X, lane);
  // block (i, j) of a tile, at d = lane_kn(D) + lds_at(16 j, 16 i), minus the product acc
  const auto subtract = [&](double* d, auto product) {
    double v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = d[lds_at(4 * q, 0)];
    double4_t acc = {0.0, 0.0, 0.0, 0.0};
    product(acc);
#pragma unroll
    for (int q = 0; q < 4; ++q) d[lds_at(4 * q, 0)] = v[q] - acc[q];
  };
  // T block (i, j) -= L_ik L_jk^T
  const auto trail = [&](int i, int j, int k) {
    subtract(tk + lds_at(16 * j, 16 * i), [&](double4_t& acc) {
      mma16<false>(acc, tk + lds_at(16 * k, 16 * i), tk + lds_at(16 * k, 16 * j));
    });
  };
  // -Y_ij -= L_ik X_kj for j < k, and -Y_ik = -L_ik X_kk (dn = lane_nk of X_kk's rows)
  const auto stage = [&](int i, int j, int k, const double* dn) {
    if (j < k) {
      subtract(xk + lds_at(16 * j, 16 * i), [&](double4_t& acc) {
        mma16<true>(acc, tk + lds_at(16 * k, 16 * i), xn + lds_at(16 * j, 16 * k));
      });
    } else {
      double4_t acc = {0.0, 0.0, 0.0, 0.0};
      mma16<true>(acc, tk + lds_at(16 * k, 16 * i), dn + 16 * k);
#pragma unroll
      for (int q = 0; q < 4; ++q) xk[lds_at(16 * j + 4 * q, 16 * i)] = -acc[q];
    }
  };
  // what step kb + 1 reads, one block per wave
  const auto next_column = [&](int kb, const double* dn) {
    if (w < 3 - kb) trail(kb + 1 + w, kb + 1, kb);
    else stage(kb + 1, w - (3 - kb), kb, dn);
  };
  // T block (i, 0) -= sum_{k < 64} B(16 i + m, k) B(n, k)
  const auto b_update = [&](int i) {
    subtract(tk + lds_at(0, 16 * i), [&](double4_t& acc) {
#pragma unroll
      for (int s = 0; s < 4; ++s)
        mma16<false>(acc, xk + lds_at(16 * s, 16 * i), xk + lds_at(16 * s, 0));
    });
  };
  // the same for the blocks (i0, j0) and (i1, j1) together, whose operands are
  // block rows p, q and r of B: two independent sums, each operand read once
  const auto b_update2 = [&](auto p_, auto q_, auto r_, auto i0_, auto j0_, auto i1_, auto j1_) {
    constexpr int p = decltype(p_)::value, q = decltype(q_)::value, r = decltype(r_)::value;
    constexpr int i0 = decltype(i0_)::value, j0 = decltype(j0_)::value;
    constexpr int i1 = decltype(i1_)::value, j1 = decltype(j1_)::value;
    double v[2][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      v[0][u] = tk[lds_at(16 * j0 + 4 * u, 16 * i0)];
      v[1][u] = tk[lds_at(16 * j1 + 4 * u, 16 * i1)];
    }
    double4_t a0 = {0.0, 0.0, 0.0, 0.0}, a1 = a0;
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      const double bp = xk[lds_at(4 * s, 16 * p)], bq = xk[lds_at(4 * s, 16 * q)];
      const double br = r == q ? bq : xk[lds_at(4 * s, 16 * r)];
      const auto of = [&](int i) { return i == p ? bp : (i == q ? bq : br); };
      a0 = __builtin_amdgcn_mfma_f64_16x16x4f64(of(j0), of(i0), a0, 0, 0, 0);
      a1 = __builtin_amdgcn_mfma_f64_16x16x4f64(of(j1), of(i1), a1, 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      tk[lds_at(16 * j0 + 4 * u, 16 * i0)] = v[0][u] - a0[u];
      tk[lds_at(16 * j1 + 4 * u, 16 * i1)] = v[1][u] - a1[u];
    }
  };
  // block row kb of the inverse to memory, by nthr threads (this one is tt),
  // zero above the diagonal (all LDS reads of a thread before its stores)
  const auto put_rows = [&](int kb, int tt, auto threads) {
    constexpr int nthr = decltype(threads)::value, per = (16 * NB + nthr - 1) / nthr;
    double v[per];
#pragma unroll
    for (int u = 0; u < per; ++u) {
      const int e = min(tt + u * nthr, 16 * NB - 1);
      v[u] = X[e >> 4][16 * kb + (e & 15)];
    }
#pragma unroll
    for (int u = 0; u < per; ++u) {
      const int e = tt + u * nthr;
      if (e < 16 * NB)
        coherent_store(&pub.inv[NB * (e >> 4) + 16 * kb + (e & 15)], (e >> 8) > kb ? 0.0 : v[u]);
    }
  };
  const std::integral_constant<int, 192> others{};
  const std::integral_constant<int, 256> all{};
  // while X holds B, the first inverse block takes the unused upper block
  // (0, 1) of T, in the layout of X (T[16 + c][r] = inverse(r, c))
  double (*const dinv0)[LDS_LD] = pub.lflag ? T + 16 : X;
  if (pub.lflag) {
    T[16 + (t >> 4)][t & 15] = (t >> 4) == (t & 15) ? 1.0 : 0.0;
    b_update(w);
  } else {
    ident(0, t, 256);
  }
  __syncthreads();
  double lv[22];                            // 22 columns of B per wave, on their way to pub.l
  // unrolled: with kb a run-time value the block addresses cost 1 us per tile,
  // more than the fetch of the longer code when it is not cached
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) {
    if (w == 0) {
      chol16_block(T, X, kb, kb == 0 ? dinv0 : X + 16 * kb, lane, mr, gbase, info);
    } else if (kb == 0) {
      if (pub.lflag) {
        using std::integral_constant;
        const integral_constant<int, 1> c1;
        const integral_constant<int, 2> c2;
        const integral_constant<int, 3> c3;
        if (w == 1) b_update2(c1, c2, c2, c1, c1, c2, c1);
        else if (w == 2) b_update2(c1, c2, c3, c3, c1, c3, c2);
        else b_update2(c2, c3, c3, c2, c2, c3, c3);
#pragma unroll
        for (int u = 0; u < 22; ++u) lv[u] = X[min(22 * (w - 1) + u, NB - 1)][lane];
      }
    } else if (kb == 1) {
      if (pub.lflag) {
#pragma unroll
        for (int u = 0; u < 22; ++u) {
          const int c = 22 * (w - 1) + u;
          if (c < NB && lane < pub.lrows) coherent_store(&pub.l[lane + (long)c * pub.ldl], lv[u]);
        }
        for (int e = t - 64; e < 256; e += 192) X[e >> 4][e & 15] = T[16 + (e >> 4)][e & 15];   // X_00
      }
      ident(2, t - 64, 192);
      ident(3, t - 64, 192);
      trail(w < 3 ? 1 + w : 3, w < 3 ? 2 : 3, 0);
      if (w < 3) stage(1 + w, 0, 0, lane_nk(dinv0, lane));
      // the last of the three waves to see its stores drained publishes the flag
      if (pub.lflag) {
        wait_stores();
        if (lane == 0 && atomicAdd(pub.drained, 1) == 2)
          __hip_atomic_store(pub.lflag, pub.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    } else if (kb == 2) {
      if (w == 1) trail(3, 3, 1);
      else stage(3, w - 2, 1, xn + lds_at(16, 0));
      if (pub.inv) {
        put_rows(0, t - 64, others);
        put_rows(1, t - 64, others);
      }
    } else if (pub.inv) {
      put_rows(2, t - 64, others);
    }
    __syncthreads();                        // (kb = 0: B read by every wave, X is free)
    if (kb == 3) break;
    if (kb == 0) ident(1, t, 256);
    next_column(kb, lane_nk(kb == 0 ? dinv0 : X + 16 * kb, lane));
    __syncthreads();
  }
  if (pub.inv) {
    put_rows(3, t, all);
  } else {
    // strictly upper 16 x 16 blocks of X, X[16 jb + c][16 ib + r], ib < jb
    for (int e = t; e < 6 * 256; e += 256) {
      const int blk = e >> 8, r = e & 15, c = (e >> 4) & 15;
      const int ib = blk < 3 ? 0 : (blk < 5 ? 1 : 2);
      const int jb = blk < 3 ? blk + 1 : (blk < 5 ? blk - 1 : 3);
      X[16 * jb + c][16 * ib + r] = 0.0;
    }
    __syncthreads();
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
