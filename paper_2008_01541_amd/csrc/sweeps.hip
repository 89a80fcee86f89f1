// Condensation sweeps through the interior factor (one-way dissection in
// breadth-first levels, Z_k = S_k^-1 dense and symmetric, B_k the sparse
// coupling of level k to level k+1 or to the region).  The level chain is
// sequential; each level is a dense product with Z_k, the assembly of its
// result, and a sparse coupling update.  Contexts whose levels have at most
// LEVEL_MAX nodes run a sweep in one launch (k_level_sweep below); wider ones,
// where the bytes of Z_k outweigh the launches, take the three launches of a
// level (sweep_symv, sweep_assemble, csr_spmv3).
//
// Dense product y = Z_k x with only the lower triangle read: Z_k is stored in
// full (column-major), but the kernels walk the lower 64 x 64 tiles (I, J),
// J <= I, once each, computing
//   row part  Z_IJ x_J      (I > J), and
//   col part  Z_IJ^T x_I,
// each into the tile's slot of a workspace.  y_I is then the sum of the row
// parts of tiles (I, J < I) and the col parts of tiles (I' >= I, I), taken
// in that fixed order by the assembly kernel, so results do not depend on
// scheduling.  HBM traffic is half the full matrix.
#include <algorithm>
#include "common.h"
#include "publish.h"

namespace pdk {

namespace {

constexpr int TS = 64;                 // tile size of the level products
constexpr int SLOT = 3 * TS;           // doubles per part slot: [rhs][64]

// One workgroup per lower tile (I, J), wave w owning columns 16 w .. 16 w + 15:
// the wave loads its 64 x 16 block into registers (lane = row, sixteen
// coalesced column loads in flight), adds its share of the row part Z_IJ x_J
// in-lane, and forms the col part Z_IJ^T x_I of its sixteen columns through a
// wave-private LDS transpose, 32 rows at a time (lane = (column, row group),
// then two cross-lane additions).  The four row-part shares are added in wave
// order.  Row parts go to slot t(I, J) of Prow (off-diagonal tiles), col parts
// to slot t(I, J) of Pcol.  26 KB of LDS per workgroup, so that the products
// still find room next to a running factorization.
__global__ __launch_bounds__(256) void k_sweep_symv(const double* __restrict__ Z, long ldz, int w,
                                                    int nb, const double* __restrict__ x, long ldx,
                                                    double* __restrict__ Prow,
                                                    double* __restrict__ Pcol) {
  __shared__ double Ts[4][TS / 2][17];     // per wave: 32 rows x 16 columns (+1 pad)
  __shared__ double xs[2][3][TS];          // x_J, x_I
  __shared__ double rp[4][3][TS];          // per-wave shares of the row part
  const int t = threadIdx.x, lane = t & 63;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int tt = blockIdx.x;
  int I = (int)((sqrt(8.0 * (double)tt + 1.0) - 1.0) * 0.5);
  while ((I + 1) * (I + 2) / 2 <= tt) ++I;
  while (I * (I + 1) / 2 > tt) --I;
  I = __builtin_amdgcn_readfirstlane(I);
  const int J = tt - I * (I + 1) / 2;
  const int i0 = I * TS, j0 = J * TS;
  const int nr = min(TS, w - i0), nc = min(TS, w - j0);
  const int c0 = 16 * wv;                  // first column of this wave
  const int ncw = max(0, min(16, nc - c0));
  // buffer loads: one 32-bit lane offset (the row) for all sixteen columns, the
  // column offset in a scalar register; lanes past the last row get an offset
  // beyond the buffer's range and read zero
  // (base and size are wave-uniform; readfirstlane keeps the descriptor scalar)
  const unsigned long long zb = reinterpret_cast<unsigned long long>(
      Z + (long)(j0 + (ncw > 0 ? c0 : 0)) * ldz);
  const unsigned zlo = __builtin_amdgcn_readfirstlane((unsigned)zb);
  const unsigned zhi = __builtin_amdgcn_readfirstlane((unsigned)(zb >> 32));
  const int zbytes = __builtin_amdgcn_readfirstlane((int)(max(ncw, 1) * ldz * (long)sizeof(double)));
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
      reinterpret_cast<void*>(((unsigned long long)zhi << 32) | zlo), 0, zbytes, 0x00020000);
  const int voff = lane < nr ? (i0 + lane) * (int)sizeof(double) : 0x7ffffff0;
  // x_J and x_I: two loads per thread (t and t + 256 of the 384 entries),
  // issued before the tile so that waiting for them does not wait for it
  double xv[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int e = t + 256 * k;
    const int h = e >= 3 * TS ? 1 : 0, v = (e / TS) % 3, r = e % TS;
    const int base = h ? i0 : j0, lim = h ? nr : nc;
    const bool ok = e < 2 * 3 * TS && r < lim;
    xv[k] = x[ok ? (long)v * ldx + base + r : 0] * (ok ? 1.0 : 0.0);
  }
  // columns past the last one (ragged tile) re-read the last column, so every
  // address stays inside the matrix: they meet zeros of x_J in the row part,
  // and their col parts are never read
  const int clast = __builtin_amdgcn_readfirstlane(max(ncw, 1) - 1);
  double z[16];
#pragma unroll
  for (int c = 0; c < 16; ++c)
    z[c] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(
                                          rs, voff, min(c, clast) * (int)(ldz * sizeof(double)), 0));
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int e = t + 256 * k;
    if (e < 2 * 3 * TS) (&xs[0][0][0])[e] = xv[k];
  }
  __syncthreads();
  // this wave's share of the row part, lane = row
  double s0 = 0.0, s1 = 0.0, s2 = 0.0;
#pragma unroll
  for (int c = 0; c < 16; ++c) {
    s0 += z[c] * xs[0][0][c0 + c];
    s1 += z[c] * xs[0][1][c0 + c];
    s2 += z[c] * xs[0][2][c0 + c];
    // four columns at a time: keeps the scheduler from loading all 48
    // operands of the row part into registers at once
    if ((c & 3) == 3) __builtin_amdgcn_sched_barrier(0);
  }
  rp[wv][0][lane] = s0;
  rp[wv][1][lane] = s1;
  rp[wv][2][lane] = s2;
  // col part of the sixteen columns, 32 rows at a time: lane = (cc = lane & 15, rg = lane >> 4)
  const int cc = lane & 15, rg = lane >> 4;
  double a0 = 0.0, a1 = 0.0, a2 = 0.0;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    // the transpose goes through wave-private LDS: the wave barriers keep the
    // compiler from moving a lane's loads across other lanes' stores
    __builtin_amdgcn_wave_barrier();
    if ((lane >> 5) == h) {
#pragma unroll
      for (int c = 0; c < 16; ++c) Ts[wv][lane & 31][c] = z[c];
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int r = 8 * rg + q;
      const double zz = Ts[wv][r][cc];
      a0 += zz * xs[1][0][32 * h + r];
      a1 += zz * xs[1][1][32 * h + r];
      a2 += zz * xs[1][2][32 * h + r];
      if ((q & 3) == 3) __builtin_amdgcn_sched_barrier(0);
    }
  }
  a0 += __shfl_xor(a0, 16, 64);
  a1 += __shfl_xor(a1, 16, 64);
  a2 += __shfl_xor(a2, 16, 64);
  a0 += __shfl_xor(a0, 32, 64);
  a1 += __shfl_xor(a1, 32, 64);
  a2 += __shfl_xor(a2, 32, 64);
  double* pc = Pcol + (long)tt * SLOT;
  if (lane < 16) {
    pc[c0 + lane] = a0;
    pc[TS + c0 + lane] = a1;
    pc[2 * TS + c0 + lane] = a2;
  }
  if (I > J) {
    __syncthreads();
    if (t < 3 * TS) {
      const int v = t >> 6, r = t & 63;
      Prow[(long)tt * SLOT + v * TS + r] = ((rp[0][v][r] + rp[1][v][r]) + rp[2][v][r]) + rp[3][v][r];
    }
  }
}

// out[v][g] = s or base[v][g] - s, s = (Z x)[v][g].  Output row g of block I
// has nb terms k = 0 .. nb - 1: the row part of tile (I, k) for k < I and the
// col part of tile (k, I) for k >= I.  Four lanes share an output, lane q
// adding terms k = q, q + 4, ...; the four partial sums are combined as
// (s0 + s1) + (s2 + s3), so the result does not depend on scheduling.
__global__ void k_sweep_assemble(int w, int nb, const double* __restrict__ Prow,
                                 const double* __restrict__ Pcol, const double* __restrict__ base,
                                 long ldb, double* __restrict__ out, long ldo) {
  const int gt = blockIdx.x * blockDim.x + threadIdx.x;
  const int q = gt & 3, o = gt >> 2;
  const int v = o / w, g = o - v * w;
  const bool live = v < 3;
  double s = 0.0;
  if (live) {
    const int I = g / TS, r = g - I * TS;
    const double* row = Prow + (long)(I * (I + 1) / 2) * SLOT + v * TS + r;
    const double* col = Pcol + v * TS + r;
#pragma unroll 4
    for (int k = q; k < nb; k += 4)
      s += (k < I) ? row[(long)k * SLOT] : col[(long)(k * (k + 1) / 2 + I) * SLOT];
  }
  const double s1 = __shfl_xor(s, 1, 64);
  const double pair = (q & 1) ? s1 + s : s + s1;           // (s0 + s1) or (s2 + s3)
  const double other = __shfl_xor(pair, 2, 64);
  const double tot = (q & 2) ? other + pair : pair + other;
  if (live && q == 0) out[(long)v * ldo + g] = base ? base[(long)v * ldb + g] - tot : tot;
}


// ---------------------------------------------------------------------------
// All levels of a sweep in one launch, for levels of up to LEVEL_MAX nodes.
//
// A chain of K levels in separate launches (product, assembly, coupling) is
// bound by the launches: 12 us a level, of which the bytes of a level of 1,184
// nodes need 2.  Here a workgroup takes 16 rows of one level, by ticket in the
// order of the sweep, and hands its 48 values on by value: the vector that a
// sweep produces holds a sentinel before it (a signalling NaN, which no
// arithmetic returns), each value is one agent-coherent store, and a workgroup
// of the next level polls the whole vector of the level before it.  Whatever
// does not depend on that vector is read before it is awaited: the 16 rows of
// Z_k (in registers; past 1,024 nodes a part of them, see below), the right-hand
// side, and the first coupling entries of every row.  What is left on the
// chain is one hand-off, the coupling product (every workgroup forms the whole
// operand of its level itself: a second hand-off would take longer), and
// 16 x w products per column.  The full Z_k is read, twice the bytes of the
// lower triangle.  A workgroup only waits for lower tickets, whose workgroups
// are running, so any number of resident workgroups makes progress.
//
// The published vectors are kept twice; a launch uses the copy of its parity
// (from the ticket, so that replays of a captured launch alternate too) and
// puts the sentinel back into the other.
//
// A workgroup fits on a compute unit beside one workgroup of a factorization
// (at most 224 of the 512 registers of a lane, 70 KB of LDS): two waves per SIMD of
// up to 144 registers each.  Up to 1,024 nodes the rows of Z_k and the coupling
// read ahead fit in that.  Past it, only the first pairs of columns are read
// before the wait, more into the registers that the awaited values leave, the
// rest once the operand has left its own (read_ahead), and up to 1,792 nodes a
// part of the coupling entries goes to LDS.  With all of Z_k held (up to 246
// registers) a sweep beside another handle's factorization of 256 workgroups
// waited for its end, 12 ms instead of 0.2 to 0.6, and one in the two-stream
// loop until units were empty: a pipelined iteration took 705 us, now 692, at
// 1,184 nodes, 1,030, now 934, at 1,560 and 1,633, now 1,400, at 2,025.  Alone, both
// sweeps: 1,184 nodes 170 -> 176 us, 1,369 183 -> 185, 1,521 305 -> 291, 1,560
// 248 -> 257, 2,025 446 -> 466.  Eight rows a task hold half as much, but read half
// lines and form the operand twice as often (1,184 nodes: 253 us); the rest of
// Z_k in LDS (87 KB and more in all) leaves no room either.
//
// Three launches a level against this kernel, both sweeps alone: 928 nodes (16
// levels) 312 -> 118 us, 1,184 (18) 349 -> 176, 1,369 (16) 332 -> 185, 1,935 (16)
// 408 -> 360, 2,025 (20) 544 -> 466.  The gain ends near LEVEL_MAX, where the full Z_k
// bounds it (2.8 TB/s).
constexpr int LT = 512;                // threads of a workgroup
constexpr int LB = 16;                 // rows of a task

// What an instance reads before the wait, as far as 144 registers and 72 KB of LDS
// reach: the first coupling entries of a row (le in registers, ls in LDS) and n1
// pairs of columns; n2 by the end of the wait, n3 before the product.
struct Ahead {
  int le, ls, n1, n2, n3;
};
constexpr Ahead read_ahead(int np, bool fwd) {
  return np <= 16   ? Ahead{4, 0, np, np, np}
         : np <= 24 ? (fwd ? Ahead{2, 2, 12, 18, np} : Ahead{2, 2, 14, 20, np})
         : np <= 28 ? (fwd ? Ahead{3, 1, 2, 10, np} : Ahead{3, 1, 4, 12, np})
                    : Ahead{2, 0, 6, 13, 26};
}

// Pairs I0 .. I1 - 1 of a thread's columns of its row zp; columns past the last
// one re-read it: they meet zeros of the operand.
template <int I0, int I1, int N>
__device__ __forceinline__ void read_z(double (&z)[N], const double* zp, int ld, int cg, int w) {
#pragma unroll
  for (int i = I0; i < I1; ++i)
    if (64 * i < w) {
      const int c = 2 * (cg + 32 * i);
      z[2 * i] = zp[(long)min(c, w - 1) * ld];
      z[2 * i + 1] = zp[(long)min(c + 1, w - 1) * ld];
    }
}

// NP: pairs of columns per thread (thread t holds row t & 15 and the columns
// 2 (t / 16 + 32 i) + {0, 1}); levels of up to 64 NP nodes.
template <int NP, bool FWD>
__global__ __launch_bounds__(LT, NP > 16 ? 3 : 2) void k_level_sweep(LevelSweep a) {
  constexpr int S = 64 * NP, RPT = (S + LT - 1) / LT;
  constexpr Ahead A = read_ahead(NP, FWD);
  constexpr int LE = A.le, LS = A.ls, N1 = A.n1, N2 = A.n2, N3 = A.n3;
  __shared__ __attribute__((aligned(16))) double xs[3][S];
  __shared__ double red[LT / 64][3][LB];
  __shared__ double lv[LS > 0 ? LS : 1][LS > 0 ? S : 1];             // a thread's own rows
  __shared__ unsigned short lc[LS > 0 ? LS : 1][LS > 0 ? S : 1];
  __shared__ int s_bad[LT / 64];
  __shared__ unsigned long long s_tk;
  const int t = threadIdx.x, wv = t >> 6;
  if (t == 0) s_tk = atomicAdd(a.ticket, 1ull);
  lds_barrier();
  const unsigned long long tk = s_tk;
  const int epoch = __builtin_amdgcn_readfirstlane((int)((tk / (unsigned)a.ntask) & 1));
  const int id = __builtin_amdgcn_readfirstlane((int)(tk % (unsigned)a.ntask));
  double* pub = a.pub + (epoch ? 3L * a.n1 : 0);
  double* clear = a.pub + (epoch ? 0 : 3L * a.n1);
  const int k = a.task[2 * id], blk = a.task[2 * id + 1];
  const bool region = k == a.K;
  if (!FWD && region) {                 // x2 += delta2
    const int r = blk * LT + t;
    if (r < a.m) {
      const int g = a.region[r];
      for (int c = 0; c < 3; ++c) a.out[c * a.ldo + g] += a.in[c * a.ldi + r];
    }
    return;
  }
  const SweepLevel L = a.lev[k];
  const int r0 = (region ? LT : LB) * blk;
  const int w = region ? min(LT, a.m - r0) : L.w;      // rows of the operand formed here
  const int rb = region ? r0 : 0;                      // first of them
  // ---- everything that does not depend on the level before
  double z[2 * NP];
  const int r = t & (LB - 1), cg = t / LB;
  if (!region) {                        // r0 + r < ld, a multiple of 16
    read_z<0, N1>(z, a.Z + L.mat + r0 + r, L.ld, cg, w);
    if (t < 3 * LB && r0 + r < w)
      clear[(long)cg * a.n1 + L.off + r0 + r] = __builtin_bit_cast(double, SENTINEL);
  }
  double b[RPT][3], cv[RPT][LE];
  int es[RPT], ee[RPT], cc[RPT][LE];
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int row = t + LT * i;
    es[i] = ee[i] = 0;
    b[i][0] = b[i][1] = b[i][2] = 0.0;
    if (row < w) {
      if (L.ptr >= 0) {
        es[i] = a.ptr[L.ptr + rb + row];
        ee[i] = a.ptr[L.ptr + rb + row + 1];
      }
      if (FWD) {
        const int g = region ? a.region[rb + row] : a.nodes[L.off + row];
#pragma unroll
        for (int c = 0; c < 3; ++c) b[i][c] = a.in[c * a.ldi + g];
      }
    }
  }
#pragma unroll
  for (int i = 0; i < RPT; ++i)
#pragma unroll
    for (int j = 0; j < LE; ++j) {
      cv[i][j] = 0.0;
      cc[i][j] = 0;
      if (es[i] + j < ee[i]) {
        cv[i][j] = a.val[L.nnz + es[i] + j];
        cc[i][j] = a.col[L.nnz + es[i] + j];
      }
    }
  if constexpr (LS > 0) {
#pragma unroll
    for (int i = 0; i < RPT; ++i)
#pragma unroll
      for (int j = 0; j < LS; ++j)
        if (t + LT * i < S) {
          const bool on = es[i] + LE + j < ee[i];
          lv[j][t + LT * i] = on ? a.val[L.nnz + es[i] + LE + j] : 0.0;
          lc[j][t + LT * i] = on ? (unsigned short)a.col[L.nnz + es[i] + LE + j] : 0;
        }
  }
  double vown = 0.0;
  if (!FWD && a.v && t < 3 * LB && r0 + r < w) vown = a.v[(long)cg * a.n1 + L.off + r0 + r];
  // ---- the level before: nothing (first of a forward sweep), the caller's
  // region vector (first of a backward one), or the published vector
  const bool polled = L.poff >= 0;
  if (polled) {
    bool bad = false;
    // far from its turn, a workgroup polls one value of the level before that
    if (L.goff >= 0) {
      long spins = 0;
      while (is_sentinel(coherent_load(&pub[L.goff]))) {
        __builtin_amdgcn_s_sleep(8);
        if (++spins > a.polls ||
            __hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
          bad = true;
          break;
        }
      }
    }
    double pv[RPT][3];
#pragma unroll
    for (int i = 0; i < RPT; ++i)
#pragma unroll
      for (int c = 0; c < 3; ++c)
        pv[i][c] = t + LT * i < L.pw ? __builtin_bit_cast(double, SENTINEL) : 0.0;
    for (long spins = 0; !bad; ++spins) {
      int miss = 0;
#pragma unroll
      for (int i = 0; i < RPT; ++i)
#pragma unroll
        for (int c = 0; c < 3; ++c)
          if (is_sentinel(pv[i][c])) pv[i][c] = coherent_load(&pub[(long)c * a.n1 + L.poff + t + LT * i]);
#pragma unroll
      for (int i = 0; i < RPT; ++i)
#pragma unroll
        for (int c = 0; c < 3; ++c) miss |= is_sentinel(pv[i][c]) ? 1 : 0;
      if (__ballot(miss) == 0) break;
      if (spins > a.polls ||
          __hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)
        bad = true;
    }
    if ((t & 63) == 0) s_bad[wv] = bad ? 1 : 0;
#pragma unroll
    for (int i = 0; i < RPT; ++i)
#pragma unroll
      for (int c = 0; c < 3; ++c)
        if (t + LT * i < S) xs[c][t + LT * i] = pv[i][c];
    if (N2 > N1 && !region) read_z<N1, N2>(z, a.Z + L.mat + r0 + r, L.ld, cg, w);
    lds_barrier();
    int any = 0;
#pragma unroll
    for (int q = 0; q < LT / 64; ++q) any |= s_bad[q];
    if (any) {
      if (t == 0) {
        atomicExch(a.err, 1);
        __hip_atomic_store(a.gave_up, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      }
      return;
    }
  } else if (N2 > N1 && !region) {
    read_z<N1, N2>(z, a.Z + L.mat + r0 + r, L.ld, cg, w);
  }
  // ---- operand of this level: f - B v (forward) or B^T x (backward)
  const double* src = polled ? &xs[0][0] : a.in;
  const long lds = polled ? S : a.ldi;
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    if (polled) {
#pragma unroll
      for (int j = 0; j < LE; ++j) {
        s0 += cv[i][j] * xs[0][cc[i][j]];
        s1 += cv[i][j] * xs[1][cc[i][j]];
        s2 += cv[i][j] * xs[2][cc[i][j]];
      }
      if constexpr (LS > 0) {
        if (t + LT * i < S) {
#pragma unroll
          for (int j = 0; j < LS; ++j) {
            const double v = lv[j][t + LT * i];
            const int c = lc[j][t + LT * i];
            s0 += v * xs[0][c];
            s1 += v * xs[1][c];
            s2 += v * xs[2][c];
          }
        }
      }
      for (int e = es[i] + LE + LS; e < ee[i]; ++e) {
        const double v = a.val[L.nnz + e];
        const int c = a.col[L.nnz + e];
        s0 += v * xs[0][c];
        s1 += v * xs[1][c];
        s2 += v * xs[2][c];
      }
    } else {
      for (int e = es[i]; e < ee[i]; ++e) {
        const double v = a.val[L.nnz + e];
        const long c = a.col[L.nnz + e];
        s0 += v * src[c];
        s1 += v * src[lds + c];
        s2 += v * src[2 * lds + c];
      }
    }
    b[i][0] = FWD ? b[i][0] - s0 : s0;
    b[i][1] = FWD ? b[i][1] - s1 : s1;
    b[i][2] = FWD ? b[i][2] - s2 : s2;
  }
  if (region) {                         // y2 = f2 - B v
    if (t < w)
#pragma unroll
      for (int c = 0; c < 3; ++c) a.out[c * a.ldo + rb + t] = b[0][c];
    return;
  }
  lds_barrier();
#pragma unroll
  for (int i = 0; i < RPT; ++i)
    if (t + LT * i < S)
#pragma unroll
      for (int c = 0; c < 3; ++c) xs[c][t + LT * i] = b[i][c];
  if (N3 > N2) read_z<N2, N3>(z, a.Z + L.mat + r0 + r, L.ld, cg, w);
  lds_barrier();
  // ---- the 16 rows of Z times the operand
  double s[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int i = 0; i < NP; ++i)
    if (64 * i < w) {
      const int c = 2 * (cg + 32 * i);
#pragma unroll
      for (int v = 0; v < 3; ++v) {
        const double2 x2 = *reinterpret_cast<const double2*>(&xs[v][c]);
        s[v] += z[2 * i] * x2.x;
        s[v] += z[2 * i + 1] * x2.y;
      }
      if (NP > N3 && i == NP - N3 - 1) {               // into the registers of the first pairs
        __builtin_amdgcn_sched_barrier(0);
        read_z<N3, NP>(z, a.Z + L.mat + r0 + r, L.ld, cg, w);
      }
    }
#pragma unroll
  for (int v = 0; v < 3; ++v) {
    s[v] += __shfl_xor(s[v], 16, 64);
    s[v] += __shfl_xor(s[v], 32, 64);
    if ((t & 63) < LB) red[wv][v][r] = s[v];
  }
  lds_barrier();
  if (t < 3 * LB && r0 + r < w) {
    double y = red[0][cg][r];
#pragma unroll
    for (int q = 1; q < LT / 64; ++q) y += red[q][cg][r];
    if (!FWD) y = vown - y;
    const long e = (long)cg * a.n1 + L.off + r0 + r;
    coherent_store(&pub[e], y);
    if (FWD)
      a.v[e] = y;
    else
      a.out[cg * a.ldo + a.nodes[L.off + r0 + r]] += y;
  }
}

template <bool FWD>
void launch_level_sweep(const LevelSweep& a, int maxw, hipStream_t st) {
  const dim3 g((unsigned)a.ntask);
  if (maxw <= 128)
    k_level_sweep<2, FWD><<<g, LT, 0, st>>>(a);
  else if (maxw <= 256)
    k_level_sweep<4, FWD><<<g, LT, 0, st>>>(a);
  else if (maxw <= 512)
    k_level_sweep<8, FWD><<<g, LT, 0, st>>>(a);
  else if (maxw <= 1024)
    k_level_sweep<16, FWD><<<g, LT, 0, st>>>(a);
  else if (maxw <= 1280)
    k_level_sweep<20, FWD><<<g, LT, 0, st>>>(a);
  else if (maxw <= 1536)
    k_level_sweep<24, FWD><<<g, LT, 0, st>>>(a);
  else if (maxw <= 1792)
    k_level_sweep<28, FWD><<<g, LT, 0, st>>>(a);
  else
    k_level_sweep<32, FWD><<<g, LT, 0, st>>>(a);
}

}  // namespace

void level_sweep(const LevelSweep& a, int maxw, bool forward, hipStream_t st) {
  if (a.ntask <= 0) return;
  if (forward)
    launch_level_sweep<true>(a, maxw, st);
  else
    launch_level_sweep<false>(a, maxw, st);
}

int level_sweep_rows(bool region) { return region ? LT : LB; }

int64_t sweep_workspace(int64_t maxw) {
  const int64_t nb = (maxw + TS - 1) / TS;
  return std::max<int64_t>(1, nb * (nb + 1) / 2) * 2 * SLOT;
}

void sweep_symv(const double* Z, long ldz, int w, const double* x, long ldx, double* P,
                hipStream_t st) {
  if (w <= 0) return;
  const int nb = (w + TS - 1) / TS, ntiles = nb * (nb + 1) / 2;
  k_sweep_symv<<<ntiles, 256, 0, st>>>(Z, ldz, w, nb, x, ldx, P, P + (long)ntiles * SLOT);
}

void sweep_assemble(int w, const double* P, const double* base, long ldb, double* out, long ldo,
                    hipStream_t st) {
  if (w <= 0) return;
  const int nb = (w + TS - 1) / TS, ntiles = nb * (nb + 1) / 2;
  k_sweep_assemble<<<(12 * w + 255) / 256, 256, 0, st>>>(w, nb, P, P + (long)ntiles * SLOT, base,
                                                         ldb, out, ldo);
}

}  // namespace pdk
