// Three-right-hand-side triangular solves with the tiled factor of the
// dataflow Cholesky (Alg. 1 step 4.5: the forward and backward substitution
// of the region system, one factor for the x, y and z columns).
#include <algorithm>
#include "common.h"
#include "publish.h"

namespace pdk {

// ---------------------------------------------------------------------------
// Three-right-hand-side triangular solves with the tiled factor.  One
// workgroup per pair of block rows; rows are claimed in dependency order
// through a ticket counter, so every claimed row only waits on rows claimed
// earlier by running workgroups.
//
// Publication by value: the vector a solve produces (y of the forward solve,
// x of the backward one) holds a sentinel before the solve (a signalling NaN
// bit pattern, which no arithmetic produces: every NaN an operation returns
// is quiet); each value is published by its own agent-coherent 8-byte store,
// and a consumer polls the values of a block row with coherent loads until
// none is the sentinel.  This takes one round trip per hand-off instead of a
// flag (stores drained, flag stored, flag polled, data loaded).  The
// sentinels are written by the solve that consumes the previous content:
// the forward solve puts them into x as it reads each value of its right-hand
// side (so x may alias the right-hand side), the backward solve puts them
// back into y as it reads y, and sentinel_fill() prepares a vector once.

constexpr long SPIN_LIMIT = 1L << 24;

__global__ void k_sentinel_fill(long n, double* p) {
  const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n) p[e] = __builtin_bit_cast(double, SENTINEL);
}
void sentinel_fill(long n, double* p, hipStream_t st) {
  if (n > 0) k_sentinel_fill<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(n, p);
}

// Loads of a column panel of a column-major matrix through a buffer
// descriptor: the row goes in the lane offset, the column (relative to the
// panel's first one) in the scalar offset, so that a load needs no 64-bit
// address registers.  Byte offsets stay below 2^32 within a panel.
template <typename T>
__device__ inline __amdgpu_buffer_rsrc_t panel_rsrc(const T* L, long ld, int col0, int ncol) {
  const unsigned long long b = reinterpret_cast<unsigned long long>(L + (long)col0 * ld);
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)b);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(b >> 32));
  const unsigned long long bytes = (unsigned long long)ncol * ld * sizeof(T);
  const unsigned nrec = bytes < 0xffffffffull ? (unsigned)bytes : 0xffffffffu;
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(((unsigned long long)hi << 32) | lo),
                                           0, (int)__builtin_amdgcn_readfirstlane(nrec), 0x00020000);
}
template <typename T>
__device__ inline T panel_load(__amdgpu_buffer_rsrc_t rs, int voff, int soff);
template <>
__device__ inline double panel_load<double>(__amdgpu_buffer_rsrc_t rs, int voff, int soff) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, voff, soff, 0));
}
template <>
__device__ inline float panel_load<float>(__amdgpu_buffer_rsrc_t rs, int voff, int soff) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, voff, soff, 0));
}

// Forward: L y = g.  Backward: L^T x = y, with L^T read from the upper triangle
// (U(r, c) = L(c, r)), super-rows from the bottom.  A super-row of 128 rows is
// two tile rows i0, i0 + 1, and each workgroup finishes one:
//   y = D^-1 (g - sum over the finished super-rows),
//   D^-1 = [ A 0 ; V B ],  A = Linv_i0, B = Linv_i0+1, V = -B L_i0+1,i0 A
// (transposed in the backward solve).  The chain of super-rows bounds the
// solve (the factor is read at 1.7 TB/s at n = 12,155), so what one hand-off
// costs is what counts: the publication (a store and a poll through memory,
// about 1.5 us), the product with the 128 values awaited, and D^-1.  V makes the
// latter one product instead of one per tile row with the coupling between
// them, at the price of two 64^3 products before the first wait, about 4 us.  The
// first two super-rows of the chain, whose turn comes before that is done, and
// all of them in a chain of up to SHORT super-rows go tile row by tile row
// instead.  Both solves, V in all but the first / in none: n = 162 20.8 / 16.4 us,
// 264 30.2 / 21.4, 512 35.8 / 30.4, 760 47.1 / 43.8; at 882 (7 super-rows) 52.6 /
// 50.7, but with the float factor a refined solve of six 222 / 231.  A wave polls just the 16 columns that it multiplies, so the
// product needs no barrier; 512 threads, since a second wave per SIMD hides
// the LDS latencies of the first.  Against 256 threads, a poll of the whole
// workgroup and a product per tile row: 485 -> 350 us at n = 12,155 (5.1 -> 3.7
// per super-row), 82 -> 58 at 2,368, float factor at 4,410 158 -> 103 (backward)
// and 139 -> 101 (forward).
//
// A workgroup fits on a compute unit beside one workgroup of the factorization
// (208 of the 512 registers of a lane at most and 70 KB of LDS): two waves per
// SIMD of up to 152 registers each.  With 200 (V in registers from the start, the
// operands of both tile columns held, the edge masked in every product) a solve
// beside another handle's factorization of 256 workgroups waited for its end,
// 13 ms instead of 0.8; alone it takes 372 us here and took 374 (both solves, n =
// 6,498).
//
// With fflags, the factor is still being computed by a dataflow Cholesky
// launch on another stream (its tile flags and its ticket[2], whose epoch
// ticket[1] that launch uses): each super-row first waits until the diagonal
// tile of its last row is published, which implies that every tile of its
// rows and both tile inverses are final.
//
// The right-hand side of row i is rhs[v ldr + i rstep]; fill (may alias rhs)
// gets the sentinel at each value once it is read.
constexpr int SR = 2 * NB;               // rows of a super-row
constexpr int TT = 512;                  // threads; thread t: rows t & 63 of both tiles,
constexpr int CG = 8;                    // columns 8 (t / 64) .. + 7 of each tile
constexpr int HEADS = 2, SHORT = 6;

// One wave's two 16 x 16 tiles (row block wv / 2) of the product X Y of two
// 64 x 64 matrices in LDS, X(r, k) = xm[k][r] and Y(k, c) = ym[c][k].
__device__ inline void mul64(const double (*xm)[NB + 1], const double (*ym)[NB + 1], int wv,
                             int lane, double4_t (&acc)[2]) {
  const int rr = 16 * (wv >> 1) + (lane & 15), c0 = 32 * (wv & 1) + (lane & 15);
  acc[0] = acc[1] = double4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
  for (int ks = 0; ks < NB; ks += 4) {
    const int k = ks + (lane >> 4);
    const double x = xm[k][rr];
    acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(ym[c0][k], x, acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(ym[c0 + 16][k], x, acc[1], 0, 0, 0);
  }
}
// m[c][r] = sign times the product above.
__device__ inline void put64(double (*m)[NB + 1], int wv, int lane, double sign,
                             const double4_t (&acc)[2]) {
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      m[32 * (wv & 1) + 16 * h + (lane >> 4) + 4 * q][16 * (wv >> 1) + (lane & 15)] =
          sign * acc[h][q];
}

// s[v] += sum_c l[c] x[v][c], c = 0 .. 7, x in LDS (16-byte aligned).
__device__ inline void dot8(const double (&l)[CG], const double (*x)[SR], int c0, double (&s)[3]) {
#pragma unroll
  for (int v = 0; v < 3; ++v)
#pragma unroll
    for (int c = 0; c < CG; c += 2) {
      const double2 w = *reinterpret_cast<const double2*>(&x[v][c0 + c]);
      s[v] += l[c] * w.x;
      s[v] += l[c + 1] * w.y;
    }
}

// FOLD: the instance with V, for chains of more than SHORT super-rows.
template <typename T, bool FWD, bool FOLD>
__global__ __launch_bounds__(TT, 2) void k_trsv3(const T* __restrict__ L, int ld, int n, int nt,
                                                 const T* __restrict__ linv, const double* rhs,
                                                 int ldr, int rstep, double* out, int ldo,
                                                 unsigned long long* ticket, int* err,
                                                 const int* fflags, const unsigned* fticket,
                                                 double* fill, int ldf) {
  __shared__ int s_row, s_bad;
  __shared__ double m0[NB][NB + 1], m1[NB][NB + 1];    // [column][row]; later partial sums
  __shared__ __attribute__((aligned(16))) double ys[3][SR];   // values of a finished super-row
  __shared__ __attribute__((aligned(16))) double zs[3][SR];   // right-hand side less the sums
  double (*part)[3][SR] = reinterpret_cast<double (*)[3][SR]>(&m0[0][0]);
  static_assert(sizeof(double) * CG * 3 * SR <= sizeof(double) * NB * (NB + 1), "partial sums");
  const int t = threadIdx.x, lane = t & 63;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int ns = (nt + 1) / 2;
  if (t == 0) {
    const unsigned long long tk = atomicAdd(ticket, 1ull);
    const int q = (int)(tk % (unsigned long long)ns);
    s_row = FWD ? q : ns - 1 - q;
    s_bad = 0;
  }
  lds_barrier();
  const int sr = __builtin_amdgcn_readfirstlane(s_row);
  const int r = lane, c8 = CG * wv;
  const int i0 = 2 * sr, nu = min(2, nt - i0), row0 = i0 * NB;
  const int pos = FWD ? sr : ns - 1 - sr;      // place in the chain
  const bool head = nu == 2 && (!FOLD || pos < HEADS);
  // right-hand-side value of thread t = 128 v + row (rows past n: 0)
  const int rv = t >> 7, rr = t & 127;
  double b = 0.0;
  if (t < 3 * SR && row0 + rr < n) {
    b = rhs[(long)rv * ldr + (long)(row0 + rr) * rstep];
    if (fill) fill[(long)rv * ldf + row0 + rr] = __builtin_bit_cast(double, SENTINEL);
  }
  if (fflags) {
    if (t == 0) {
      const int fe = (int)__hip_atomic_load(&fticket[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int il = i0 + nu - 1;
      if (!df_wait(&fflags[il * nt + il], fe, err)) s_bad = 1;
    }
    lds_barrier();
    if (s_bad) return;
  }
  // ---- the tile inverses and the coupling tile: la = A, lb = B (the transposes in
  // the backward solve), and in m1 V or, for a super-row taken tile row by tile
  // row, the coupling tile
  double la[CG], lb[CG];
  const T* La = linv + (long)i0 * NB * NB;
  const T* Lb = linv + (long)(i0 + nu - 1) * NB * NB;
  // m[c][r] = element (r, c) of a tile, from a thread's elements t + 512 q
  const auto put = [&](double (*m)[NB + 1], const double (&x)[CG]) {
#pragma unroll
    for (int q = 0; q < CG; ++q) m[wv + CG * q][lane] = x[q];
  };
  if (nu == 2) {
    // L_i0+1,i0, or its transpose from the upper triangle; what lies past the
    // edge re-reads the last row or column and is masked
#pragma unroll
    for (int q = 0; q < CG; ++q) {
      const int ec = wv + CG * q;
      const int lr = row0 + (FWD ? NB : 0) + lane, lc = row0 + (FWD ? 0 : NB) + ec;
      const double ok = (lr < n && lc < n) ? 1.0 : 0.0;
      const double v = (double)L[min(lr, n - 1) + (long)min(lc, n - 1) * ld] * ok;
      if (FWD) m1[ec][lane] = v;
      else m1[lane][ec] = v;                    // m1[c][r] = L_i0+1,i0(r, c) in both
    }
  }
  if (FOLD && nu == 2 && !head) {
    double va[CG], vb[CG];
#pragma unroll
    for (int q = 0; q < CG; ++q) {
      va[q] = La[t + TT * q];
      vb[q] = Lb[t + TT * q];
    }
    double4_t acc4[2];
    put(m0, va);
    lds_barrier();
#pragma unroll
    for (int c = 0; c < CG; ++c) la[c] = FWD ? m0[c8 + c][r] : m0[r][c8 + c];
    mul64(m1, m0, wv, lane, acc4);              // P = L_i0+1,i0 A
    lds_barrier();
    put(m0, vb);
    put64(m1, wv, lane, 1.0, acc4);
    lds_barrier();
#pragma unroll
    for (int c = 0; c < CG; ++c) lb[c] = FWD ? m0[c8 + c][r] : m0[r][c8 + c];
    mul64(m0, m1, wv, lane, acc4);              // V = -B P
    lds_barrier();
    put64(m1, wv, lane, -1.0, acc4);
    lds_barrier();
  } else if (FWD) {
#pragma unroll
    for (int c = 0; c < CG; ++c) {
      la[c] = La[r + NB * (c8 + c)];
      lb[c] = Lb[r + NB * (c8 + c)];
    }
  } else {
    // B, which is needed first, is turned through LDS; A straight from memory
    // (64 lines a load, behind the first tile row)
    double vb[CG];
#pragma unroll
    for (int q = 0; q < CG; ++q) vb[q] = Lb[t + TT * q];
    if (nu == 2)
#pragma unroll
      for (int c = 0; c < CG; ++c) la[c] = La[c8 + c + NB * r];
    put(m0, vb);
    lds_barrier();
#pragma unroll
    for (int c = 0; c < CG; ++c) lb[c] = m0[r][c8 + c];
    if (nu == 1)
#pragma unroll
      for (int c = 0; c < CG; ++c) la[c] = lb[c];
    lds_barrier();
  }
  // ---- products with the finished super-rows
  double acc[2][3];
#pragma unroll
  for (int u = 0; u < 2; ++u) acc[u][0] = acc[u][1] = acc[u][2] = 0.0;
  // this lane's value of the 3 x 16 that the wave polls
  const int pv = lane >> 4, pc = ((lane >> 3) & 1) * NB + c8 + (lane & 7);
  bool bad = false;
  for (int p = 0; p < pos && !bad; ++p) {
    const int q = FWD ? p : ns - 1 - p;
    const int col0 = q * SR;
    // both tiles' 16 columns of both tile rows load while the values are awaited
    // (a row past the edge re-reads the last one and gives a sum that is not
    // used; a column past the edge re-reads the last one and meets a zero)
    T lv[2][2][CG];
    const __amdgpu_buffer_rsrc_t prs = panel_rsrc(L, ld, col0, min(SR, n - col0));
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int voff = min(row0 + u * NB + r, n - 1) * (int)sizeof(T);
#pragma unroll
      for (int w = 0; w < 2; ++w)
#pragma unroll
        for (int c = 0; c < CG; ++c)
          lv[u][w][c] = panel_load<T>(prs, voff, min(w * NB + c8 + c, n - 1 - col0) * ld * (int)sizeof(T));
    }
    double val = 0.0;
    long spins = 0;
    for (;;) {
      if (pv < 3 && col0 + pc < n) val = coherent_load(&out[(long)pv * ldo + col0 + pc]);
      if (__ballot(is_sentinel(val)) == 0) break;
      if (++spins > SPIN_LIMIT ||
          __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
        bad = true;
        break;
      }
    }
    // this wave's own columns of ys: only their order within the wave matters
    if (pv < 3) ys[pv][pc] = val;
    __builtin_amdgcn_wave_barrier();
    // one tile column at a time, so that the values of only one are held
    // beside the tiles
#pragma unroll
    for (int w = 0; w < 2; ++w) {
#pragma unroll
      for (int v = 0; v < 3; ++v) {
        double x[CG];
#pragma unroll
        for (int c = 0; c < CG; c += 2) {
          const double2 y2 = *reinterpret_cast<const double2*>(&ys[v][w * NB + c8 + c]);
          x[c] = y2.x;
          x[c + 1] = y2.y;
        }
#pragma unroll
        for (int c = 0; c < CG; ++c)
#pragma unroll
          for (int u = 0; u < 2; ++u) acc[u][v] += (double)lv[u][w][c] * x[c];
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_wave_barrier();
  }
  auto total = [&]() {
    double y = part[0][rv][rr];
#pragma unroll
    for (int q = 1; q < CG; ++q) y += part[q][rv][rr];
    return y;
  };
  const bool mine = t < 3 * SR && row0 + rr < n;
  double lx[CG];                                // V, or the coupling tile
  const auto read_lx = [&]() {
#pragma unroll
    for (int c = 0; c < CG; ++c) lx[c] = FWD ? m1[c8 + c][r] : m1[r][c8 + c];
  };
  // ---- zs = right-hand side less the sums
  if (pos > 0) {
    if (bad && lane == 0) {
      atomicExch(err, 1);
      s_bad = 1;
    }
    lds_barrier();
    if (s_bad) return;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int v = 0; v < 3; ++v) part[wv][v][u * NB + r] = acc[u][v];
    if (nu == 2) read_lx();
    lds_barrier();
    if (mine) b -= total();
  }
  if (t < 3 * SR) zs[rv][rr] = b;
  lds_barrier();
  // ---- D^-1 zs in one product, or the first tile row (h = 0), then the second,
  // less the coupling
  if (nu == 2 && !head) {
    double s[2][3];
#pragma unroll
    for (int u = 0; u < 2; ++u) s[u][0] = s[u][1] = s[u][2] = 0.0;
    dot8(la, zs, c8, s[0]);
    dot8(lb, zs, NB + c8, s[1]);
    dot8(lx, zs, (FWD ? 0 : NB) + c8, s[FWD ? 1 : 0]);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int v = 0; v < 3; ++v) part[wv][v][u * NB + r] = s[u][v];
    lds_barrier();
    if (mine) coherent_store(&out[(long)rv * ldo + row0 + rr], total());
    return;
  }
  const auto tile_row = [&](const double (&l)[CG], int h) {
    double s[3] = {0.0, 0.0, 0.0};
    dot8(l, zs, h * NB + c8, s);
#pragma unroll
    for (int v = 0; v < 3; ++v) part[wv][v][h * NB + r] = s[v];
    lds_barrier();
    if (t < 3 * SR && (rr >> 6) == h) {
      const double y = total();
      if (mine) coherent_store(&out[(long)rv * ldo + row0 + rr], y);
      ys[rv][rr] = y;
    }
  };
  constexpr int H0 = FWD ? 0 : 1;
  if (nu == 1) {
    tile_row(la, 0);
    return;
  }
  if (pos == 0) read_lx();
  tile_row(H0 == 0 ? la : lb, H0);
  lds_barrier();
  double k[3] = {0.0, 0.0, 0.0};
  dot8(lx, ys, H0 * NB + c8, k);
#pragma unroll
  for (int v = 0; v < 3; ++v) part[wv][v][(1 - H0) * NB + r] = k[v];
  lds_barrier();
  if (t < 3 * SR && (rr >> 6) == 1 - H0) zs[rv][rr] -= total();
  lds_barrier();
  tile_row(H0 == 0 ? lb : la, 1 - H0);
}

template <typename T, bool FWD>
static void launch_trsv3(const T* L, int ld, int n, const T* linv, const double* rhs, int ldr,
                         int rstep, double* out, int ldo, unsigned long long* ticket, int* err,
                         const int* fflags, const unsigned* fticket, double* fill, int ldf,
                         hipStream_t st) {
  const int nt = (n + NB - 1) / NB, ns = (nt + 1) / 2;
  const auto kernel = ns <= SHORT ? k_trsv3<T, FWD, false> : k_trsv3<T, FWD, true>;
  kernel<<<ns, TT, 0, st>>>(L, ld, n, nt, linv, rhs, ldr, rstep, out, ldo, ticket, err, fflags,
                            fticket, fill, ldf);
}

void trsv3_forward(const double* L, int ld, int n, const double* linv_ws, const double* g,
                   int ldg, double* y, int ldy, unsigned long long* ticket, int* err,
                   double* xfill, int ldxf, hipStream_t st, const int* fflags,
                   const unsigned* fticket) {
  launch_trsv3<double, true>(L, ld, n, linv_ws, g, ldg, 1, y, ldy, ticket, err, fflags, fticket,
                             xfill, ldxf, st);
}

void trsv3_backward(const double* L, int ld, int n, const double* linv_ws, double* y, int ldy,
                    double* x, int ldx, unsigned long long* ticket, int* err, hipStream_t st) {
  launch_trsv3<double, false>(L, ld, n, linv_ws, y, ldy, 1, x, ldx, ticket, err, nullptr, nullptr,
                              y, ldy, st);
}

void trsv3_backward_packed(const double* L, int ld, int n, const double* linv_ws,
                           const double* Yt, double* x, int ldx, unsigned long long* ticket,
                           int* err, hipStream_t st) {
  launch_trsv3<double, false>(L, ld, n, linv_ws, Yt, 1, NB, x, ldx, ticket, err, nullptr, nullptr,
                              nullptr, 0, st);
}

// The same solves with a float factor (FP64 vectors and arithmetic).
void trsv3_forward(const float* L, int ld, int n, const float* linv_ws, const double* g, int ldg,
                   double* y, int ldy, unsigned long long* ticket, int* err, double* xfill,
                   int ldxf, hipStream_t st) {
  launch_trsv3<float, true>(L, ld, n, linv_ws, g, ldg, 1, y, ldy, ticket, err, nullptr, nullptr,
                            xfill, ldxf, st);
}
void trsv3_backward(const float* L, int ld, int n, const float* linv_ws, double* y, int ldy,
                    double* x, int ldx, unsigned long long* ticket, int* err, hipStream_t st) {
  launch_trsv3<float, false>(L, ld, n, linv_ws, y, ldy, 1, x, ldx, ticket, err, nullptr, nullptr,
                             y, ldy, st);
}

}  // namespace pdk
