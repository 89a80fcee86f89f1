// Dense FP64 kernels for gfx950: tiled Cholesky of the Schur system and of the
// interior level blocks, triangular inverse, symmetric inverse assembly,
// three-right-hand-side triangular solves and the symmetric matrix-vector
// product.  Tiles are NB x NB (NB = 64), column-major.  Products run on the
// FP64 matrix cores (v_mfma_f64_16x16x4f64) with operands staged through LDS.
#include <algorithm>
#include <climits>
#include "common.h"
#include "tile_factor_f64.h"
#include "publish.h"
#include "df_schedule.h"

namespace pdk {

constexpr int KC = 16;           // K-chunk staged through LDS per step

struct Acc {                     // one wave's 32 x 32 share of a 64 x 64 tile
  double4_t c[2][2];
};
typedef double double2_t __attribute__((ext_vector_type(2)));

__device__ inline void acc_zero(Acc& a) {
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) a.c[i][j] = double4_t{0.0, 0.0, 0.0, 0.0};
}

// Tile-local coordinates of accumulator element (mb, nb, q) of this lane.
// The product is issued with the column operand in the MFMA "A" slot, so the
// 16x16 result block D[i][j] (lane l, register q: i = l/16 + 4q, j = l%16)
// holds C(row = j, col = i): consecutive lanes walk down a column of C, which
// makes loads and stores of C coalesced.
__device__ inline int acc_row(int mb) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  return (w >> 1) * 32 + mb * 16 + (lane & 15);
}
__device__ inline int acc_col(int nb, int q) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  return (w & 1) * 32 + nb * 16 + (lane >> 4) + 4 * q;
}

// Ls[k][r] = op(G)(r0 + r, k0 + k) for r < NB, k < KC; zero outside (mr, kr).
// TRANS = false: element (r, k) at G[r + k*ld]; TRANS = true: at G[k + r*ld].
template <bool TRANS>
__device__ inline void load_chunk(double (*Ls)[LDS_LD], const double* __restrict__ G, long ld,
                                  int r0, int k0, int mr, int kr) {
  const int t = threadIdx.x;
  if (!TRANS) {
    const int r = t & 63;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = (t >> 6) + 4 * q;
      double v = 0.0;
      if (r < mr && k < kr) v = G[(long)(r0 + r) + (long)(k0 + k) * ld];
      Ls[k][r] = v;
    }
  } else {
    const int k = t & 15;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = (t >> 4) + 16 * q;
      double v = 0.0;
      if (r < mr && k < kr) v = G[(long)(k0 + k) + (long)(r0 + r) * ld];
      Ls[k][r] = v;
    }
  }
}

// acc(r, c) += sum_{kk < K} Ahat(r, kk) * Bhat(c, kk) where
// Ahat(r, kk) = opA(A)(ar0 + r, ak0 + kk) and Bhat(c, kk) = opB(B)(br0 + c, bk0 + kk);
// rows r >= amr and cols c >= bmr read as zero.
template <bool TA, bool TB>
__device__ void gemm_acc(Acc& acc, double (*As)[LDS_LD], double (*Bs)[LDS_LD],
                         const double* __restrict__ A, long lda, int ar0, int amr, int ak0,
                         const double* __restrict__ B, long ldb, int br0, int bmr, int bk0,
                         int K) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int wr = w >> 1, wc = w & 1;
  for (int kk = 0; kk < K; kk += KC) {
    __syncthreads();
    load_chunk<TA>(As, A, lda, ar0, ak0 + kk, amr, K - kk);
    load_chunk<TB>(Bs, B, ldb, br0, bk0 + kk, bmr, K - kk);
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < KC / 4; ++ks) {
      const int k = ks * 4 + (lane >> 4);
      const double a0 = As[k][wr * 32 + (lane & 15)];
      const double a1 = As[k][wr * 32 + 16 + (lane & 15)];
      const double b0 = Bs[k][wc * 32 + (lane & 15)];
      const double b1 = Bs[k][wc * 32 + 16 + (lane & 15)];
      acc.c[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(b0, a0, acc.c[0][0], 0, 0, 0);
      acc.c[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(b1, a0, acc.c[0][1], 0, 0, 0);
      acc.c[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(b0, a1, acc.c[1][0], 0, 0, 0);
      acc.c[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(b1, a1, acc.c[1][1], 0, 0, 0);
    }
  }
}

__device__ inline void tri_index(int b, int& i, int& j) {
  // b -> (i, j) with 0 <= j <= i, b = i (i + 1) / 2 + j
  int ii = (int)((sqrt(8.0 * (double)b + 1.0) - 1.0) * 0.5);
  while ((ii + 1) * (ii + 2) / 2 <= b) ++ii;
  while (ii * (ii + 1) / 2 > b) --ii;
  i = ii;
  j = b - ii * (ii + 1) / 2;
}

// An empty asm that takes all sixteen values: every load feeding them is
// issued before it and they are waited for once, instead of the compiler
// turning each select of a loaded value into a branch with its own wait.
__device__ inline void regs_ready(double (&v)[16]) {
  asm volatile(""
               : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]),
                 "+v"(v[6]), "+v"(v[7]), "+v"(v[8]), "+v"(v[9]), "+v"(v[10]), "+v"(v[11]),
                 "+v"(v[12]), "+v"(v[13]), "+v"(v[14]), "+v"(v[15]));
}

// ---------------------------------------------------------------------------
// Single-launch tiled Cholesky.  Persistent workgroups claim lower tiles in
// column-major order from a ticket counter; the workgroup that owns tile
// (i, j) accumulates sum_{k<j} L_ik L_jk^T on the matrix cores as soon as each
// pair of operand tiles is published (operands double-buffered through LDS
// with the next chunk's loads in flight during the current products), then
// either factors the diagonal tile (blocked, in LDS) and publishes L_jj and its
// inverse, or waits for Linv_jj and forms L_ij = (A_ij - acc) Linv_jj^T.  Each
// factor tile is also written transposed into the upper triangle, so the
// backward substitution reads L^T with unit stride.  A task only waits on
// tasks with a smaller ticket, all of which belong to running workgroups, so
// the schedule cannot deadlock; waits are bounded and raise *err instead.
// Resets the task ticket and advances the launch epoch kept in ctr[1]; the
// factorization kernel reads the epoch from memory, so a captured graph that
// replays the pair still gets a fresh epoch every time.
__global__ void k_reset_counter(unsigned* ctr) {
  ctr[0] = 0u;
  ctr[1] = ctr[1] + 1u;
}

// Paired layout of a wave's 32 x 32 share of a tile: accumulator element
// (mb, nb, q) of a lane is the tile's (pair_row(t, mb), pair_col(nb, q)).  A lane's
// two row (column) operands are neighbours, so one 16-byte LDS read fetches both.
__device__ inline int pair_row(int t, int mb) {
  return (t >> 7) * 32 + 2 * (t & 15) + mb;
}
__device__ inline int pair_col(int t, int nb, int q) {
  return ((t >> 6) & 1) * 32 + 2 * (((t & 63) >> 4) + 4 * q) + nb;
}

// acc(r, c) += sum_{k0 <= k < k1} As[k][r] Bs[k][c] (paired layout).
__device__ __forceinline__ void pair_product(Acc& acc, double (*As)[LDS_LD], double (*Bs)[LDS_LD],
                                             int k0, int k1) {
  const int t = task_tid(), lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int ar = (w >> 1) * 32 + 2 * (lane & 15), bc = (w & 1) * 32 + 2 * (lane & 15);
#pragma unroll
  for (int ks = k0; ks < k1; ks += 4) {
    const double2_t a = *(const double2_t*)&As[ks + (lane >> 4)][ar];
    const double2_t b = *(const double2_t*)&Bs[ks + (lane >> 4)][bc];
    acc.c[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(b[0], a[0], acc.c[0][0], 0, 0, 0);
    acc.c[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(b[1], a[0], acc.c[0][1], 0, 0, 0);
    acc.c[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(b[0], a[1], acc.c[1][0], 0, 0, 0);
    acc.c[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(b[1], a[1], acc.c[1][1], 0, 0, 0);
  }
}

// T[c][r] = f(element of this thread, its index 0..15) in the paired layout.
template <typename F>
__device__ __forceinline__ void pair_to_lds(double (*T)[LDS_LD], F f) {
  const int t = task_tid();
#pragma unroll
  for (int nb = 0; nb < 2; ++nb)
#pragma unroll
    for (int qq = 0; qq < 4; ++qq) {
      const double2_t v = {f(0, nb, qq), f(1, nb, qq)};
      *(double2_t*)&T[pair_col(t, nb, qq)][pair_row(t, 0)] = v;
    }
}

// The sixteen elements of this thread (paired layout, index 8 mb + 4 nb + q) of
// the mr x mc tile of A at (r0, c0), read coherently: a task's own input tile
// (0 outside the tile).
__device__ __forceinline__ void load_own_tile(double (&v)[16], const double* A, long lda, int r0,
                                              int c0, int mr, int mc) {
  const int t = task_tid();
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int r = pair_row(t, e >> 3), c = pair_col(t, (e >> 2) & 1, e & 3);
    v[e] = coherent_load(&A[(long)(r0 + min(r, mr - 1)) + (long)(c0 + min(c, mc - 1)) * lda]);
  }
  regs_ready(v);
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int r = pair_row(t, e >> 3), c = pair_col(t, (e >> 2) & 1, e & 3);
    if (r >= mr || c >= mc) v[e] = 0.0;
  }
}

// acc[u] += sum_{k<kend} L_ik L_{j+u,k}^T, u < CT (paired layout): one tile row
// and CT tile columns.  The operands pass through LDS in chunks of KD columns,
// double-buffered (each buffer the row operand's chunk over the column
// operands'): the products of chunk q run while chunk q + 1 is written to the
// other buffer from registers and chunk q + 2 is loaded into them, with one
// barrier a chunk.  Thread 0 reads the ready flags of a later 64-column step
// during each chunk, so neither the flag round trip nor the operand latency is
// on the path when the producers are ahead; a step whose flags are not set yet
// is awaited after the last chunk before it.  512 workgroups of 45 steps each,
// all operands ready: 53 TFLOP/s for CT = 1 (41 with one buffer, two barriers a
// step and 8-byte LDS reads) and 58 for CT = 2; the rest is the barrier and the
// LDS round trip per chunk (128 x 128 tiles reach 69, but finish a row's tile
// too late for the next one).  buf: 2 NB rows; s_rdy: three LDS ints.
template <int CT>
__device__ bool df_accumulate(Acc (&acc)[CT], double (*buf)[LDS_LD], const double* __restrict__ Ar,
                              int ldar, int r0, int mr, const double* __restrict__ A, int lda,
                              int c0, int mc, int i, int j, int kend, int nt, const int* flags,
                              int epoch, int* err, int* s_rdy, const int* mark) {
  if (kend == 0) return true;
  constexpr int KD = CT == 1 ? 32 : 16;                      // columns per chunk
  constexpr int CPS = NB / KD;                               // chunks per 64-column step
  static_assert(2 * (1 + CT) * KD <= 2 * NB, "two chunks must fit the two tile buffers");
  const int t = task_tid();
  const int rp = 2 * (t & 31), k8 = t >> 5;
  // rows past the tile's edge: the address is clamped to the last pair of rows
  // (leading dimensions are even, so a pair never leaves its column) and the
  // value replaced by zero
  const double* pa = Ar + r0 + min(rp, (mr - 1) & ~1) + (long)k8 * ldar;
  const double* pb = A + c0 + min(rp, (mc - 1) & ~1) + (long)k8 * lda;
  const bool ragged = mr < NB || mc < NB;
  double2_t va[KD / 8], vb[CT][KD / 8];
  const auto load = [&](int ch) {
#pragma unroll
    for (int q = 0; q < KD / 8; ++q) {
      va[q] = *(const double2_t*)(pa + (long)(ch * KD + 8 * q) * ldar);
#pragma unroll
      for (int u = 0; u < CT; ++u)
        vb[u][q] = *(const double2_t*)(pb + u * NB + (long)(ch * KD + 8 * q) * lda);
    }
  };
  const auto put = [&](double (*b)[LDS_LD]) {
    if (ragged) {
#pragma unroll
      for (int q = 0; q < KD / 8; ++q) {
        va[q] = double2_t{rp < mr ? va[q][0] : 0.0, rp + 1 < mr ? va[q][1] : 0.0};
        if (CT == 1) vb[0][q] = double2_t{rp < mc ? vb[0][q][0] : 0.0, rp + 1 < mc ? vb[0][q][1] : 0.0};
      }
    }
#pragma unroll
    for (int q = 0; q < KD / 8; ++q) {
      *(double2_t*)&b[k8 + 8 * q][rp] = va[q];
#pragma unroll
      for (int u = 0; u < CT; ++u) *(double2_t*)&b[(1 + u) * KD + k8 + 8 * q][rp] = vb[u][q];
    }
  };
  // columns k0 .. k1 - 1 of a chunk in LDS
  const auto products = [&](double (*b)[LDS_LD], int k0, int k1) {
    const int lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int ar = (w >> 1) * 32 + 2 * (lane & 15), bc = (w & 1) * 32 + 2 * (lane & 15);
#pragma unroll
    for (int ks = k0; ks < k1; ks += 4) {
      const double2_t a = *(const double2_t*)&b[ks + (lane >> 4)][ar];
#pragma unroll
      for (int u = 0; u < CT; ++u) {
        const double2_t c = *(const double2_t*)&b[(1 + u) * KD + ks + (lane >> 4)][bc];
        acc[u].c[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(c[0], a[0], acc[u].c[0][0], 0, 0, 0);
        acc[u].c[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(c[1], a[0], acc[u].c[0][1], 0, 0, 0);
        acc[u].c[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(c[0], a[1], acc[u].c[1][0], 0, 0, 0);
        acc[u].c[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(c[1], a[1], acc[u].c[1][1], 0, 0, 0);
      }
    }
  };
  const int* const fi = &flags[i * nt];
  const int* const fj = &flags[j * nt];
  // thread 0 waits for the flags of 64-column step k
  const auto await = [&](int k) {
    if (t == 0)
      s_rdy[2] = df_wait(&fi[k], epoch, err) && df_wait(&fj[k], epoch, err) &&
                         (CT == 1 || df_wait(&fj[nt + k], epoch, err))
                     ? k + 1 : -1;
    __syncthreads();
    return s_rdy[2];
  };
  double (*const oth0)[LDS_LD] = buf + (1 + CT) * KD;
  const int nch = kend * CPS;
  int rdy = await(0);                          // 64-column steps known to be published
  if (rdy < 0) return false;
  load(0);
  put(buf);
  load(1);
  int held = 1;                                // chunk in va, vb (-1: none)
  __syncthreads();
  for (int ch = 0; ch < nch; ++ch) {
    double (*const cur)[LDS_LD] = (ch & 1) ? oth0 : buf;
    double (*const oth)[LDS_LD] = (ch & 1) ? buf : oth0;
    int gi = 0, gj = 0, gj1 = 0, gm = 0;
    const bool peek = t == 0 && rdy < kend;
    if (peek) {
      gi = __hip_atomic_load(&fi[rdy], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      gj = __hip_atomic_load(&fj[rdy], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      gj1 = CT == 1 ? epoch
                    : __hip_atomic_load(&fj[nt + rdy], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (t == 0 && mark) gm = __hip_atomic_load(mark, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    products(cur, 0, KD / 2);
    const bool have = held == ch + 1;
    if (have) {
      put(oth);
      held = -1;
    }
    const int want = have ? ch + 2 : ch + 1;
    if (held < 0 && want < nch && want / CPS < rdy) {
      load(want);
      held = want;
    }
    products(cur, KD / 2, KD);
    if (t == 0) s_rdy[ch & 1] = rdy + (peek && gi == epoch && gj == epoch && gj1 == epoch ? 1 : 0);
    if (t == 0 && mark && gm == epoch) cu_pause(mark, epoch);
    __syncthreads();
    rdy = s_rdy[ch & 1];                       // not written again before the next barrier
    if (ch + 1 < nch && !have) {
      if (held < 0) {
        if ((ch + 1) / CPS >= rdy) {
          rdy = await((ch + 1) / CPS);
          if (rdy < 0) return false;
        }
        load(ch + 1);
      }
      put(oth);
      held = -1;
      if (ch + 2 < nch && (ch + 2) / CPS < rdy) {
        load(ch + 2);
        held = ch + 2;
      }
      __syncthreads();
    }
  }
  return true;
}

// Triangular right factor: acc(r, c) = sum_k As[k][r] Bs[k][c] where
// Bs[k][c] = 0 for k > c (Bs holds the transpose of a lower-triangular
// tile), so column block cb only takes the k-blocks 0..cb.  The waves of
// column half 0 own column blocks 0 and 3 and those of half 1 blocks 1 and 2
// (40 products per wave instead of 64); accumulator block nb of this wave is
// column block tri_cb(nb).  Only exact zeros are skipped, so the result is
// the full product's.
__device__ inline int tri_cb(int t, int nb) {
  const int wc = __builtin_amdgcn_readfirstlane(t >> 6) & 1;
  return wc ? 1 + nb : 3 * nb;
}
__device__ inline int tri_col(int t, int nb, int q) {
  return 16 * tri_cb(t, nb) + ((t & 63) >> 4) + 4 * q;
}
__device__ inline int tri_row(int t, int mb) { return (t >> 7) * 32 + mb * 16 + (t & 15); }
__device__ inline void lds_product_tri(Acc& acc, double (*As)[LDS_LD], double (*Bs)[LDS_LD]) {
  const int t = task_tid(), lane = t & 63;
  const int wr = __builtin_amdgcn_readfirstlane(t >> 6) >> 1;
  const int cb0 = tri_cb(t, 0), cb1 = tri_cb(t, 1);
  const int kA = 4 * (cb0 + 1), kB = 4 * (cb1 + 1);     // 4-deep steps per block, kA < kB
#pragma unroll 4
  for (int ks = 0; ks < kA; ++ks) {
    const int k = ks * 4 + (lane >> 4);
    const double a0 = As[k][wr * 32 + (lane & 15)];
    const double a1 = As[k][wr * 32 + 16 + (lane & 15)];
    const double b0 = Bs[k][16 * cb0 + (lane & 15)];
    const double b1 = Bs[k][16 * cb1 + (lane & 15)];
    acc.c[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(b0, a0, acc.c[0][0], 0, 0, 0);
    acc.c[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(b1, a0, acc.c[0][1], 0, 0, 0);
    acc.c[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(b0, a1, acc.c[1][0], 0, 0, 0);
    acc.c[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(b1, a1, acc.c[1][1], 0, 0, 0);
  }
#pragma unroll 4
  for (int ks = kA; ks < kB; ++ks) {
    const int k = ks * 4 + (lane >> 4);
    const double a0 = As[k][wr * 32 + (lane & 15)];
    const double a1 = As[k][wr * 32 + 16 + (lane & 15)];
    const double b1 = Bs[k][16 * cb1 + (lane & 15)];
    acc.c[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(b1, a0, acc.c[0][1], 0, 0, 0);
    acc.c[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(b1, a1, acc.c[1][1], 0, 0, 0);
  }
}

// T[c][r] = src[r + c ld] for a full 64 x 64 tile of published data, 16 bytes
// a load, with all eight loads of a thread in flight before the LDS writes.
__device__ inline void stage_tile(double (*T)[LDS_LD], const double* __restrict__ src, long ld) {
  const int t = task_tid();
  double2_t v[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) v[q] = *(const double2_t*)&src[2 * (t & 31) + ((t >> 5) + 8 * q) * ld];
#pragma unroll
  for (int q = 0; q < 8; ++q) *(double2_t*)&T[(t >> 5) + 8 * q][2 * (t & 31)] = v[q];
}

// Task kinds in column j (tickets in this order):
//  * diagonal (j, j): accumulates k < j - 2, finishes the two tiles to its left
//    itself and factors the tile:
//      L_{j,j-2} = (A_{j,j-2} - P2_j) Linv_{j-2}^T, while Linv_{j-1} is awaited,
//      L_{j,j-1} = (A_{j,j-1} - P1_j - L_{j,j-2} L_{j-1,j-2}^T) Linv_{j-1}^T,
//    with the partial sums P1_j, P2_j (k < j - 2) of the two tasks below.  The
//    chain diag(j-1) -> diag(j), the critical path, thus has one hand-off per
//    column, Linv_{j-1}, and what feeds it from the column before that is
//    computed by the diagonal's own workgroup.
//  * (j + 1, j) and (j + 2, j): the partial sums P1_{j+1} (k < j - 1) and
//    P2_{j+2} (k < j) of tiles left of a diagonal, into the workspace sbuf
//    (published with flags of their own, no Linv wait).
//  * (i, j), i >= j + 3: accumulates k < j, waits for Linv_jj, forms
//    L_ij = (A_ij - acc) Linv_jj^T.  Large matrices (df64_wide) take two tiles
//    of a row, (i, j) and (i, j + 1) with j even and i >= j + 4, as one task:
//    they share the row operand, and after L_ij the step k = j of the second
//    tile is added from LDS.  Not a 2 x 2 block of tiles: the time from Linv_jj
//    to the published L_ij, which the next tile of the row waits for, is a
//    chain in every row (n = 6,498: 2.6 ms with 2 x 2 blocks from the eighth
//    pair below the diagonal on).
//  * with Yt != NULL the three right-hand sides ride along as an extra tile
//    row (Yt: 64 x n, column-major, rows 0..2 = g^T on entry): its tasks
//    compute Y_j = (G_j - sum_{k<j} Y_k L_jk^T) Linv_jj^T, i.e. the forward
//    substitution y = L^-1 g, on the same schedule.
// Flags and slots of sbuf: df_schedule.h; a partial sum is kept in the register
// order of the task that writes it.
template <int WIDE>
__global__ __launch_bounds__(256, 2) void k_potrf_dataflow(double* A, int lda, int n, int nt,
                                                           double* linv_ws, double* sbuf,
                                                           int* flags, unsigned* ticket, int* info,
                                                           int* err, double* Yt, int* cu_marks) {
  const int epoch = (int)ticket[1];
  const int rhs = Yt != nullptr ? 1 : 0;
  int* const mark = cu_marks ? cu_marks + cu_slot() : nullptr;
  int* const pflags = flags + df_part_flag(0, nt);
  // two 64 x 68 double tiles (69,632 bytes): the operand chunks of the
  // accumulation, then a tile and an operand of the finishing steps
  __shared__ __attribute__((aligned(16))) double buf0[2 * NB][LDS_LD];
  double (*const buf1)[LDS_LD] = buf0 + NB;
  __shared__ int s_task, s_ok, s_rdy[3], s_drained;
  const int ntask = df64_task_count(nt, WIDE, rhs);
  // thread 0 waits for a flag; false (for every thread) if the wait was given up
  const auto await = [&](const int* f) {
    if (threadIdx.x == 0 && !df_wait(f, epoch, err)) s_ok = 0;
    __syncthreads();
    return s_ok != 0;
  };
  for (;;) {
    const int t = task_tid();
    __syncthreads();
    if (t == 0) {
      s_task = (int)atomicAdd(ticket, 1u);
      s_ok = 1;
      s_drained = 0;
    }
    __syncthreads();
    const int q = s_task;
    if (q >= ntask) return;
    const DfTask task = df64_task(q, nt, WIDE, rhs);
    const int i = task.i, j = task.j;
    const bool rrow = (i == nt);
    const bool diag = (i == j), part = !rrow && !diag && i <= j + 2;
    const int kend = df_acc_steps(i, j, nt);
    if (part && kend == 0) continue;             // an empty sum: nobody reads it
    double* Ai = rrow ? Yt : A;
    const int ldai = rrow ? NB : lda;
    const int r0 = rrow ? 0 : i * NB, c0 = j * NB;
    const int mr = rrow ? 3 : min(NB, n - r0), mc = min(NB, n - c0);
    // l -> T (T[c][r]), the layout of lds_product_tri
    const auto tri_to_lds = [&](const Acc& l, double (*T)[LDS_LD]) {
      const int t = task_tid();
#pragma unroll
      for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
          for (int qq = 0; qq < 4; ++qq) T[tri_col(t, nb, qq)][tri_row(t, mb)] = l.c[mb][nb][qq];
    };
    // l -> rows < mr and columns < mc of the tile of M at (r0, cj * NB), straight from the registers
    const auto tri_to_mem = [&](const Acc& l, double* M, long ld, int cj, int mcols) {
      const int t = task_tid();
#pragma unroll
      for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
          for (int qq = 0; qq < 4; ++qq) {
            const int r = tri_row(t, mb), c = tri_col(t, nb, qq);
            if (r < mr && c < mcols)
              coherent_store(&M[(long)(r0 + r) + (long)(cj * NB + c) * ld], l.c[mb][nb][qq]);
          }
    };
    // transposed copy of the tile (i, cj) in T (T[c][r] = L(r, c)), read only by
    // the backward solve after this launch:
    // U(cj NB + r', r0 + c') = L(r0 + c', cj NB + r') with r' = e & 63, c' = e >> 6
    const auto transposed = [&](double (*T)[LDS_LD], int cj, int mcols) {
      for (int e = task_tid(); e < NB * NB; e += 256) {
        const int r = e & 63, c = e >> 6;
        if (c < mr && r < mcols) A[(long)(cj * NB + r) + (long)(r0 + c) * lda] = T[r][c];
      }
    };
    if (WIDE && task.cols == 2) {
      Acc acc[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        double v[16];
        load_own_tile(v, A, lda, r0, c0 + u * NB, mr, NB);
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[u].c[e >> 3][(e >> 2) & 1][e & 3] = -v[e];
      }
      if (!df_accumulate<2>(acc, buf0, A, lda, r0, mr, A, lda, c0, NB, i, j, j, nt, flags, epoch,
                            err, s_rdy, mark))
        return;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        pair_to_lds(buf0, [&](int mb, int nb, int qq) { return -acc[u].c[mb][nb][qq]; });
        if (!await(&flags[(j + u) * nt + (j + u)])) return;
        stage_tile(buf1, linv_ws + (long)(j + u) * NB * NB, NB);
        __syncthreads();
        Acc l;
        acc_zero(l);
        lds_product_tri(l, buf0, buf1);
        tri_to_mem(l, A, lda, j + u, NB);
        __syncthreads();
        tri_to_lds(l, buf0);
        if (u == 0) {
          if (!await(&flags[(j + 1) * nt + j])) return;
          stage_tile(buf1, A + (long)(j + 1) * NB + (long)c0 * lda, lda);
          __syncthreads();
          pair_product(acc[1], buf0, buf1, 0, NB);
        }
        publish_flag(&flags[i * nt + j + u], epoch);
        transposed(buf0, j + u, NB);
        __syncthreads();
      }
      continue;
    }
    // the diagonal chain issues first
    const bool critical = diag || part;
    if (critical) __builtin_amdgcn_s_setprio(2);
    // acc <- -A_ij (read now so that the load is off the path after the last
    // product; padding: identity on the diagonal tile, zero elsewhere), or 0
    Acc acc1[1];
    Acc& acc = acc1[0];
    {
      double v[16];
      if (part) {
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = 0.0;
      } else {
        load_own_tile(v, Ai, ldai, r0, c0, mr, mc);
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int mb = e >> 3, nb = (e >> 2) & 1, qq = e & 3;
        const bool pad = diag && pair_row(t, mb) == pair_col(t, nb, qq) && pair_row(t, mb) >= mr;
        acc.c[mb][nb][qq] = pad ? -1.0 : -v[e];
      }
    }
    if (!df_accumulate<1>(acc1, buf0, Ai, ldai, r0, mr, A, lda, c0, mc, i, j, kend, nt, flags, epoch,
                          err, s_rdy, critical ? nullptr : mark))
      return;
    // the diagonal task's local phase: no waits from here to the inverse's flag
    const auto mark_unit = [&]() {
      if (t == 0 && mark) __hip_atomic_store(mark, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    if (part) {
      const int slot = df_part_slot(i, j, nt);
      double* Sb = sbuf + (long)slot * NB * NB;
#pragma unroll
      for (int e = 0; e < 16; ++e) coherent_store(&Sb[e * 256 + t], acc.c[e >> 3][(e >> 2) & 1][e & 3]);
      publish_flag(&pflags[slot], epoch);
      __builtin_amdgcn_s_setprio(0);
      continue;
    }
    // v -= the partial sum in a slot of sbuf (paired layout)
    const auto subtract_part = [&](double (&v)[16], int slot) {
      const int tt = task_tid();
      const double* Sb = sbuf + (long)slot * NB * NB;
#pragma unroll
      for (int e = 0; e < 16; ++e) v[e] -= Sb[e * 256 + tt];
    };
    const auto own_to_lds = [&](const double (&v)[16], double (*T)[LDS_LD]) {
      pair_to_lds(T, [&](int mb, int nb, int qq) { return v[8 * mb + 4 * nb + qq]; });
    };
    if (diag) {
      if (j > 0) {
        double v[16];                              // what becomes L_{j,j-1}
        load_own_tile(v, A, lda, r0, (j - 1) * NB, mr, NB);
        if (j > 1) {
          {
            double v2[16];                         // what becomes L_{j,j-2}
            load_own_tile(v2, A, lda, r0, (j - 2) * NB, mr, NB);
            if (!await(&flags[(j - 2) * nt + (j - 2)])) return;
            stage_tile(buf1, linv_ws + (long)(j - 2) * NB * NB, NB);   // buf1[kk][c] = Linv(c, kk)
            if (j > 2) {
              if (!await(&pflags[df_part_slot(j, j - 2, nt)])) return;
              subtract_part(v2, df_part_slot(j, j - 2, nt));
            }
            own_to_lds(v2, buf0);
          }
          __syncthreads();
          Acc l;
          acc_zero(l);
          lds_product_tri(l, buf0, buf1);
          __syncthreads();
          tri_to_lds(l, buf0);
          tri_to_mem(l, A, lda, j - 2, NB);
          __syncthreads();
          pair_product(acc, buf0, buf0, 0, NB);
          publish_flag(&flags[j * nt + (j - 2)], epoch);
          if (t == 0 && (!df_wait(&flags[(j - 1) * nt + (j - 2)], epoch, err) ||
                         (j > 2 && !df_wait(&pflags[df_part_slot(j, j - 1, nt)], epoch, err))))
            s_ok = 0;
          __syncthreads();
          if (!s_ok) return;
          stage_tile(buf1, A + (long)(j - 1) * NB + (long)(j - 2) * NB * lda, lda);
          if (j > 2) subtract_part(v, df_part_slot(j, j - 1, nt));
          __syncthreads();
          Acc s;                                   // L_{j,j-2} L_{j-1,j-2}^T
          acc_zero(s);
          pair_product(s, buf0, buf1, 0, NB);
#pragma unroll
          for (int e = 0; e < 16; ++e) v[e] -= s.c[e >> 3][(e >> 2) & 1][e & 3];
          __syncthreads();
        }
        own_to_lds(v, buf0);
        if (!await(&flags[(j - 1) * nt + (j - 1)])) return;
        mark_unit();
        stage_tile(buf1, linv_ws + (long)(j - 1) * NB * NB, NB);
        __syncthreads();
        Acc l;
        acc_zero(l);
        lds_product_tri(l, buf0, buf1);            // L = S Linv^T
        __syncthreads();
        // L into buf1 (the tile factor's inverse slot, which takes the last
        // rank-64 update C -= L L^T block by block), C without that term into
        // buf0; the tile factor also writes L and the inverse to memory
        tri_to_lds(l, buf1);
      } else {
        mark_unit();
      }
      pair_to_lds(buf0, [&](int mb, int nb, int qq) { return -acc.c[mb][nb][qq]; });
      __syncthreads();
      TilePublish pub;
      pub.epoch = epoch;
      pub.inv = linv_ws + (long)j * NB * NB;
      if (j > 0) {
        pub.lflag = &flags[j * nt + (j - 1)];
        pub.l = A + (long)r0 + (long)(j - 1) * NB * lda;
        pub.ldl = lda;
        pub.lrows = mr;
        pub.drained = &s_drained;
      }
      factor_tile_blocked(buf0, buf1, mr, r0, info, pub);
      // only the inverse is read inside this launch: it is published first,
      // then L (lower) and its transposed copy (strictly upper) are written for
      // the solves.  The mark is cleared before the flag is stored
      // (publish_flag waits for both), so the next diagonal task, which may run
      // on this unit, sets its own mark after this clear
      if (t == 0 && mark) __hip_atomic_store(mark, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      publish_flag(&flags[i * nt + j], epoch);
      for (int e = t; e < NB * NB; e += 256) {
        const int r = e & 63, c = e >> 6;
        if (r < mr && c < mr)
          A[(long)(r0 + r) + (long)(r0 + c) * lda] = (r >= c) ? buf0[c][r] : buf0[r][c];
      }
      // transposed copies of the tiles finished above, read back (coalesced,
      // coherent) and turned through LDS: U(cs + r', r0 + c') = L(r0 + c', cs + r')
      for (int cj = max(j - 2, 0); cj < j; ++cj) {
        const int cs = cj * NB;
        __syncthreads();
        {
          const int r = t & 63;
          double v[16];
#pragma unroll
          for (int qq = 0; qq < 16; ++qq)
            v[qq] = coherent_load(&A[(long)(r0 + min(r, mr - 1)) + (long)(cs + (t >> 6) + 4 * qq) * lda]);
          regs_ready(v);
#pragma unroll
          for (int qq = 0; qq < 16; ++qq) buf1[(t >> 6) + 4 * qq][r] = (r < mr) ? v[qq] : 0.0;
        }
        __syncthreads();
        for (int e = t; e < NB * NB; e += 256) {
          const int r = e & 63, c = e >> 6;
          if (c < mr) A[(long)(cs + r) + (long)(r0 + c) * lda] = buf1[r][c];
        }
      }
    } else {
      pair_to_lds(buf0, [&](int mb, int nb, int qq) { return -acc.c[mb][nb][qq]; });
      if (!await(&flags[j * nt + j])) return;
      stage_tile(buf1, linv_ws + (long)j * NB * NB, NB);
      __syncthreads();
      acc_zero(acc);
      lds_product_tri(acc, buf0, buf1);            // (A_ij - sum) Linv_jj^T
      // (the right-hand-side row also runs over the last, ragged, column
      // block); the LDS copy is for the transposed copy below
      tri_to_mem(acc, rrow ? Yt : A, ldai, j, mc);
      __syncthreads();
      if (!rrow) tri_to_lds(acc, buf0);
      publish_flag(&flags[i * nt + j], epoch);
      if (!rrow) transposed(buf0, j, mc);
    }
    if (critical) __builtin_amdgcn_s_setprio(0);
  }
}

void potrf_dataflow(double* A, int lda, int n, double* linv_ws, double* sbuf, int* flags,
                    unsigned* ticket, int* info, int* err, int n_wg, double* Yt, hipStream_t st,
                    int* cu_marks, hipEvent_t after_reset) {
  const int nt = (n + NB - 1) / NB;
  const int wide = df64_wide(nt);
  const int ntask = df64_task_count(nt, wide, Yt ? 1 : 0);
  if (!Yt) k_reset_counter<<<1, 1, 0, st>>>(ticket);     // with Yt: done by rhs_pack
  if (after_reset) (void)hipEventRecord(after_reset, st);
  // two instances: the code of the two-tile task, unused, would cost the
  // diagonal chain 1.7 us per column through the register allocation
  const auto kernel = wide ? k_potrf_dataflow<1> : k_potrf_dataflow<0>;
  kernel<<<std::min(ntask, n_wg), 256, 0, st>>>(A, lda, n, nt, linv_ws, sbuf, flags, ticket, info,
                                                err, Yt, cu_marks);
}

int potrf_cu_slots() { return CU_SLOTS; }

// Before a factorization that carries its right-hand side: Yt[v + r * 64] =
// g[v * ldg + r] (v < 3), the sentinel into fill (may alias g) for the solve that
// follows, the pivot report cleared and the launch epoch advanced.  One launch
// instead of four (about 2 us each beside a small system).
__global__ void k_rhs_pack(int n, const double* g, int ldg, double* __restrict__ Yt, double* fill,
                           int* info, unsigned* ticket) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r == 0) {
    *info = 0;
    ticket[0] = 0u;
    ticket[1] = ticket[1] + 1u;
  }
  if (r >= n) return;
  for (int v = 0; v < 3; ++v) {
    Yt[v + (long)r * NB] = g[(long)v * ldg + r];
    fill[(long)v * ldg + r] = __builtin_bit_cast(double, SENTINEL);
  }
}
void rhs_pack(int n, const double* g, int ldg, double* Yt, double* fill, int* info,
              unsigned* ticket, hipStream_t st) {
  k_rhs_pack<<<(n + 255) / 256, 256, 0, st>>>(n, g, ldg, Yt, fill, info, ticket);
}

__global__ void k_copy_f64(long n, const double* __restrict__ src, double* __restrict__ dst) {
  const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n) dst[e] = src[e];
}void copy_f64(long n, const double* src, double* dst, hipStream_t st) {
  if (n > 0) k_copy_f64<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(n, src, dst);
}

__global__ void k_zero_int(int* p) { *p = 0; }
void zero_int(int* p, hipStream_t st) { k_zero_int<<<1, 1, 0, st>>>(p); }

__global__ void k_zero_f64(long n, double* p) {
  const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n) p[e] = 0.0;
}
void zero_f64(long n, double* p, hipStream_t st) {
  if (n > 0) k_zero_f64<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(n, p);
}

// ---------------------------------------------------------------------------
// Triangular inverse X = L^-1 from the tiled factor:
//   M_ip = Linv_ii L_ip (p < i), X_ii = Linv_ii, X_ic = -sum_{p=c}^{i-1} M_ip X_pc.

__global__ __launch_bounds__(256) void k_scale_offdiag(const double* L, int ldl, int n,
                                                       const double* linv_ws, double* M,
                                                       int ldm) {
  __shared__ double As[KC][LDS_LD];
  __shared__ double Bs[KC][LDS_LD];
  int i, p;
  tri_index(blockIdx.x, i, p);
  i += 1;                                   // strictly lower tiles: p < i
  const int r0 = i * NB, mr = min(NB, n - r0);
  Acc acc;
  acc_zero(acc);
  // C(r, c) = sum_kk Linv_ii(r, kk) L_ip(kk, c): Ahat = Linv (normal), Bhat(c, kk) = L(i*NB+kk, p*NB+c)
  gemm_acc<false, true>(acc, As, Bs, linv_ws + (long)i * NB * NB, NB, 0, NB, 0, L, ldl,
                        p * NB, NB, i * NB, mr);
#pragma unroll
  for (int mb = 0; mb < 2; ++mb)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = acc_row(mb), c = acc_col(nb, q);
        if (r < mr) M[(long)(r0 + r) + (long)(p * NB + c) * ldm] = acc.c[mb][nb][q];
      }
}

// Block row i of X: workgroup c < i computes X_ic, workgroup c = i copies Linv_ii.
__global__ __launch_bounds__(256) void k_trtri_row(const double* M, int ldm, int n, int i,
                                                   const double* linv_ws, double* X, int ldx) {
  __shared__ double As[KC][LDS_LD];
  __shared__ double Bs[KC][LDS_LD];
  const int c = blockIdx.x;
  const int r0 = i * NB, mr = min(NB, n - r0);
  if (c == i) {
    const double* Li = linv_ws + (long)i * NB * NB;
    for (int e = threadIdx.x; e < NB * NB; e += 256) {
      const int r = e & 63, cc = e >> 6;
      if (r < mr && cc < mr) X[(long)(r0 + r) + (long)(r0 + cc) * ldx] = Li[e];
    }
    return;
  }
  Acc acc;
  acc_zero(acc);
  // C(r, cc) = sum_kk M(r0 + r, c*NB + kk) X(c*NB + kk, c*NB + cc), kk < (i - c) * NB
  gemm_acc<false, true>(acc, As, Bs, M, ldm, r0, mr, c * NB, X, ldx, c * NB, NB, c * NB,
                        (i - c) * NB);
#pragma unroll
  for (int mb = 0; mb < 2; ++mb)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = acc_row(mb), cc = acc_col(nb, q);
        if (r < mr) X[(long)(r0 + r) + (long)(c * NB + cc) * ldx] = -acc.c[mb][nb][q];
      }
}

void trtri_from_factor(const double* L, int ldl, int n, const double* linv_ws, double* M,
                       double* X, int ldx, hipStream_t st) {
  // M (strictly lower tiles, leading dimension ldx) and X must not alias:
  // block row i of X reads every M_ip of its row while writing X_ic.
  const int nt = (n + NB - 1) / NB;
  if (nt > 1) {
    const int cnt = (nt - 1) * nt / 2;
    k_scale_offdiag<<<cnt, 256, 0, st>>>(L, ldl, n, linv_ws, M, ldx);
  }
  for (int i = 0; i < nt; ++i) k_trtri_row<<<i + 1, 256, 0, st>>>(M, ldx, n, i, linv_ws, X, ldx);
}

// Z = X^T X (X lower) written in full symmetric storage.
__global__ __launch_bounds__(256) void k_lauum_full(const double* X, int ldx, int n, double* Z,
                                                    int ldz) {
  __shared__ double As[KC][LDS_LD];
  __shared__ double Bs[KC][LDS_LD];
  int i, j;
  tri_index(blockIdx.x, i, j);
  const int r0 = i * NB, c0 = j * NB;
  const int mr = min(NB, n - r0), mc = min(NB, n - c0);
  Acc acc;
  acc_zero(acc);
  // Z(r0 + r, c0 + c) = sum_{p >= r0} X(p, r0 + r) X(p, c0 + c)
  gemm_acc<true, true>(acc, As, Bs, X, ldx, r0, mr, r0, X, ldx, c0, mc, r0, n - r0);
#pragma unroll
  for (int mb = 0; mb < 2; ++mb)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = acc_row(mb), c = acc_col(nb, q);
        if (r < mr && c < mc) {
          Z[(long)(r0 + r) + (long)(c0 + c) * ldz] = acc.c[mb][nb][q];
          Z[(long)(c0 + c) + (long)(r0 + r) * ldz] = acc.c[mb][nb][q];
        }
      }
}

void lauum_full(const double* X, int ldx, int n, double* Z, int ldz, hipStream_t st) {
  const int nt = (n + NB - 1) / NB;
  k_lauum_full<<<nt * (nt + 1) / 2, 256, 0, st>>>(X, ldx, n, Z, ldz);
}

// C = beta C + alpha A B^T, one 64 x 64 tile of C per workgroup (tiles on or
// below the diagonal only when lower; B lower triangular when blower, so the
// sum for a column tile j stops at the end of B's diagonal tile j).
__global__ __launch_bounds__(256) void k_gemm_nt(const double* A, long lda, const double* B,
                                                 long ldb, double* C, long ldc, int m, int nc,
                                                 int K, double alpha, double beta, int lower,
                                                 int blower) {
  __shared__ double As[KC][LDS_LD];
  __shared__ double Bs[KC][LDS_LD];
  int i, j;
  if (lower) {
    tri_index(blockIdx.x, i, j);
  } else {
    const int mt = (m + NB - 1) / NB;
    i = blockIdx.x % mt;
    j = blockIdx.x / mt;
  }
  const int r0 = i * NB, c0 = j * NB;
  const int mr = min(NB, m - r0), mc = min(NB, nc - c0);
  const int kend = blower ? min(K, c0 + NB) : K;
  Acc acc;
  acc_zero(acc);
  gemm_acc<false, false>(acc, As, Bs, A, lda, r0, mr, 0, B, ldb, c0, mc, 0, kend);
#pragma unroll
  for (int mb = 0; mb < 2; ++mb)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = acc_row(mb), c = acc_col(nb, q);
        if (r < mr && c < mc) {
          double* p = C + (long)(r0 + r) + (long)(c0 + c) * ldc;
          const double v = alpha * acc.c[mb][nb][q];
          *p = beta == 0.0 ? v : beta * *p + v;
        }
      }
}

void gemm_nt(const double* A, long lda, const double* B, long ldb, double* C, long ldc, int m,
             int nc, int K, double alpha, double beta, int lower, int blower, hipStream_t st) {
  if (m <= 0 || nc <= 0) return;
  const long mt = (m + NB - 1) / NB, ntc = (nc + NB - 1) / NB;
  const long cnt = lower ? mt * (mt + 1) / 2 : mt * ntc;
  k_gemm_nt<<<(unsigned)cnt, 256, 0, st>>>(A, lda, B, ldb, C, ldc, m, nc, K, alpha, beta, lower,
                                           blower);
}

__global__ __launch_bounds__(256) void k_copy_lower_tiles(const double* S, int lds, double* H,
                                                          int ldh, int n) {
  int i, j;
  tri_index(blockIdx.x, i, j);
  const int r0 = i * NB, c0 = j * NB;
  const int mr = min(NB, n - r0), mc = min(NB, n - c0);
  for (int e = threadIdx.x; e < NB * NB; e += 256) {
    const int r = e & 63, c = e >> 6;
    if (r < mr && c < mc) H[(long)(r0 + r) + (long)(c0 + c) * ldh] = S[(long)(r0 + r) + (long)(c0 + c) * lds];
  }
}

void copy_lower_tiles(const double* S, int lds, double* H, int ldh, int n, hipStream_t st) {
  const int nt = (n + NB - 1) / NB;
  k_copy_lower_tiles<<<nt * (nt + 1) / 2, 256, 0, st>>>(S, lds, H, ldh, n);
}

__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// ---------------------------------------------------------------------------
// y = alpha * A v + beta * y, A symmetric in full storage: element i of the
// product is the dot of column i with v.  A workgroup owns 8 columns (two per
// wave); the three right-hand sides are staged through LDS in chunks of 512
// rows, so each matrix element costs one 16-byte-per-lane streaming load and
// the vector is read from L2 once per 8 columns.
constexpr int SV_CHUNK = 512;
__global__ __launch_bounds__(256) void k_symv3(const double* __restrict__ A, long lda, int n,
                                               const double* __restrict__ v, long ldv,
                                               double alpha, double beta, double* y, long ldy) {
  __shared__ double vs[3][SV_CHUNK];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int c0 = blockIdx.x * 8 + w * 2;
  const bool has0 = c0 < n, has1 = c0 + 1 < n;
  const double* a0 = A + (long)min(c0, n - 1) * lda;
  const double* a1 = A + (long)min(c0 + 1, n - 1) * lda;
  const bool vec = ((lda & 1) == 0) && ((((unsigned long)A) & 15) == 0);
  double s[2][3] = {{0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}};
  for (int j0 = 0; j0 < n; j0 += SV_CHUNK) {
    const int cnt = min(SV_CHUNK, n - j0);
    __syncthreads();
    for (int e = t; e < 3 * SV_CHUNK; e += 256) {
      const int vv = e / SV_CHUNK, jj = e % SV_CHUNK;
      vs[vv][jj] = (jj < cnt) ? v[(long)vv * ldv + j0 + jj] : 0.0;
    }
    __syncthreads();
    if (vec && cnt == SV_CHUNK) {
#pragma unroll
      for (int it = 0; it < SV_CHUNK / 128; ++it) {
        const int jj = it * 128 + 2 * lane;
        const double2 x0 = *(const double2*)(a0 + j0 + jj);
        const double2 x1 = *(const double2*)(a1 + j0 + jj);
#pragma unroll
        for (int vv = 0; vv < 3; ++vv) {
          const double p = vs[vv][jj], q = vs[vv][jj + 1];
          s[0][vv] += x0.x * p + x0.y * q;
          s[1][vv] += x1.x * p + x1.y * q;
        }
      }
    } else {
      for (int jj = lane; jj < cnt; jj += 64) {
        const double x0 = a0[j0 + jj], x1 = a1[j0 + jj];
#pragma unroll
        for (int vv = 0; vv < 3; ++vv) {
          s[0][vv] += x0 * vs[vv][jj];
          s[1][vv] += x1 * vs[vv][jj];
        }
      }
    }
  }
#pragma unroll
  for (int cc = 0; cc < 2; ++cc)
#pragma unroll
    for (int vv = 0; vv < 3; ++vv) s[cc][vv] = wave_sum(s[cc][vv]);
  if (lane == 0) {
#pragma unroll
    for (int cc = 0; cc < 2; ++cc) {
      if (!(cc == 0 ? has0 : has1)) continue;
      const int col = c0 + cc;
#pragma unroll
      for (int vv = 0; vv < 3; ++vv) {
        double* yo = y + (long)vv * ldy + col;
        *yo = (beta == 0.0) ? alpha * s[cc][vv] : alpha * s[cc][vv] + beta * *yo;
      }
    }
  }
}

void symv3(const double* A, int lda, int n, const double* v, int ldv, double alpha, double beta,
           double* y, int ldy, hipStream_t st) {
  if (n > 0) k_symv3<<<(n + 7) / 8, 256, 0, st>>>(A, lda, n, v, ldv, alpha, beta, y, ldy);
}

}  // namespace pdk
