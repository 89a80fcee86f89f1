// Warm-start MLP kernels: BF16-operand GEMMs with FP32 accumulation on the
// matrix cores (v_mfma_f32_16x16x32_bf16), fused epilogues, loss, bias
// gradients and Adam.  Activations and gradients are FP32 in memory and are
// rounded to BF16 (round to nearest even) when staged as GEMM operands;
// weights keep an FP32 master copy and a BF16 copy used by the products.
#include <algorithm>
#include "common.h"

namespace pdk {

typedef __bf16 bf16x8m_t __attribute__((ext_vector_type(8)));
constexpr int MT = 64;          // output tile
constexpr int MKC = 32;         // K chunk
constexpr int MLD = MKC + 8;    // LDS row (bf16), 16-byte aligned

// Stage a 64 x 32 operand chunk into LDS as S[row][k] (bf16) from FP32 rows
// over the batch: element (row, k) is at G[k * ld + row].
__device__ inline void stage(__bf16 (*S)[MLD], const float* __restrict__ G, long ld, int row0,
                             int nrow, int k0, int kend) {
  const int t = threadIdx.x;
  const int row = t & 63, kq = (t >> 6) * 8;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int k = k0 + kq + e;
    float v = 0.f;
    if (row0 + row < nrow && k < kend) v = G[(long)k * ld + row0 + row];
    S[row][kq + e] = (__bf16)v;
  }
}

// acc[mb][nb] += the 64 x 64 tile of A^T B over one chunk in LDS, this wave's
// 32 x 32 share: lane l, register q: row wr 32 + mb 16 + l % 16, column
// wc 32 + nb 16 + 4 (l / 16) + q
__device__ __forceinline__ void chunk_product(float4_t (&acc)[2][2], __bf16 (*As)[MLD],
                                              __bf16 (*Bs)[MLD]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int wr = w >> 1, wc = w & 1, ko = 8 * (lane >> 4);
  const bf16x8m_t a0 = *(const bf16x8m_t*)&As[wr * 32 + (lane & 15)][ko];
  const bf16x8m_t a1 = *(const bf16x8m_t*)&As[wr * 32 + 16 + (lane & 15)][ko];
  const bf16x8m_t b0 = *(const bf16x8m_t*)&Bs[wc * 32 + (lane & 15)][ko];
  const bf16x8m_t b1 = *(const bf16x8m_t*)&Bs[wc * 32 + 16 + (lane & 15)][ko];
  acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b0, a0, acc[0][0], 0, 0, 0);
  acc[0][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b1, a0, acc[0][1], 0, 0, 0);
  acc[1][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b0, a1, acc[1][0], 0, 0, 0);
  acc[1][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b1, a1, acc[1][1], 0, 0, 0);
}

// C[z][m][n] = sum_{k in split z} A[k][m] B[k][n]   (FP32 out, row-major, ldc = N)
__global__ __launch_bounds__(256) void k_gemm_bf16(int M, int N, int K, const float* __restrict__ A,
                                                   long lda, const float* __restrict__ B, long ldb,
                                                   float* __restrict__ C, int ksplit) {
  __shared__ __attribute__((aligned(16))) __bf16 As[MT][MLD];
  __shared__ __attribute__((aligned(16))) __bf16 Bs[MT][MLD];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int wr = w >> 1, wc = w & 1;
  const int m0 = blockIdx.y * MT, n0 = blockIdx.x * MT;
  const int z = blockIdx.z;
  const int kbeg = z * ksplit, kend = min(K, kbeg + ksplit);
  float4_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = float4_t{0.f, 0.f, 0.f, 0.f};
  for (int k0 = kbeg; k0 < kend; k0 += MKC) {
    __syncthreads();
    stage(As, A, lda, m0, M, k0, kend);
    stage(Bs, B, ldb, n0, N, k0, kend);
    __syncthreads();
    chunk_product(acc, As, Bs);
  }
  float* Cz = C + (long)z * M * N;
#pragma unroll
  for (int mb = 0; mb < 2; ++mb)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int m = m0 + wr * 32 + mb * 16 + (lane & 15);
        const int n = n0 + wc * 32 + nb * 16 + 4 * (lane >> 4) + q;
        if (m < M && n < N) Cz[(long)m * N + n] = acc[mb][nb][q];
      }
}

// ---------------------------------------------------------------------------
// Products with the BF16 weights, 16 or 32 rows of the batch per workgroup.  For
// a batch of up to 32 they are bound by reading the weights once: every 16-byte
// load of a lane is one MFMA operand (eight k of one row, no LDS), and the loads
// of KG chunks are in flight while the ones before are multiplied.  A larger
// batch reads the weights again for every 32 rows, mostly from the caches.  An
// output's sum goes over chunks of MKC, splits in order, as the gradients' in
// k_gemm_bf16.  Network 25,992-512-512-19,494, forward / training step in us,
// 64 x 64 tiles staged through LDS (the kernel before) -> these: batch 1 117 -> 32
// / 449 -> 187, 32 131 -> 54 / 512 -> 269, 64 156 -> 82 / 570 -> 352, 128 215 -> 132 /
// 761 -> 537, 1,024 1,378 -> 808 / 4,042 -> 3,200; so all batches take them.

typedef float float4u_t __attribute__((ext_vector_type(4), aligned(4)));
typedef __bf16 bf16x8u_t __attribute__((ext_vector_type(8), aligned(2)));
constexpr int KG = 4;           // chunks of MKC in flight

// eight floats of a row from k on as BF16; zero from kend on
__device__ __forceinline__ bf16x8m_t act8(const float* __restrict__ p, int k, int kend) {
  bf16x8m_t o;
  if (k + 8 <= kend) {
    const float4u_t u = *(const float4u_t*)(p + k), v = *(const float4u_t*)(p + k + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      o[e] = (__bf16)u[e];
      o[4 + e] = (__bf16)v[e];
    }
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (__bf16)(k + e < kend ? p[k + e] : 0.f);
  }
  return o;
}
__device__ __forceinline__ bf16x8m_t wgt8(const __bf16* __restrict__ p, int k, int kend) {
  if (k + 8 <= kend) return *(const bf16x8u_t*)(p + k);
  bf16x8m_t o;
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = k + e < kend ? p[k + e] : (__bf16)0.f;
  return o;
}

// acc[b](m = lane % 16, n = 4 (lane / 16) + q) of the rows m0 + 16 b .. of X and the 16
// rows n0 .. of W, over k in [kbeg, kend)
template <int MB>
__device__ __forceinline__ void rows_times_weights(float4_t (&acc)[MB], int M, int N, int K, int m0,
                                                   int n0, int kbeg, int kend,
                                                   const float* __restrict__ X,
                                                   const __bf16* __restrict__ W) {
  const int lane = threadIdx.x & 63, ko = 8 * (lane >> 4);
  const __bf16* pw = W + (long)min(n0 + (lane & 15), N - 1) * K;
  const float* px[MB];
#pragma unroll
  for (int b = 0; b < MB; ++b) {
    px[b] = X + (long)min(m0 + 16 * b + (lane & 15), M - 1) * K;
    acc[b] = float4_t{0.f, 0.f, 0.f, 0.f};
  }
  bf16x8m_t w[KG], x[KG][MB];
  const auto load = [&](int k0) {
#pragma unroll
    for (int g = 0; g < KG; ++g) {
      const int k = k0 + g * MKC + ko;
      w[g] = wgt8(pw, k, kend);
#pragma unroll
      for (int b = 0; b < MB; ++b) x[g][b] = act8(px[b], k, kend);
    }
  };
  load(kbeg);
  for (int k0 = kbeg; k0 < kend; k0 += KG * MKC) {
    bf16x8m_t cw[KG], cx[KG][MB];
#pragma unroll
    for (int g = 0; g < KG; ++g) {
      cw[g] = w[g];
#pragma unroll
      for (int b = 0; b < MB; ++b) cx[g][b] = x[g][b];
    }
    if (k0 + KG * MKC < kend) load(k0 + KG * MKC);
#pragma unroll
    for (int g = 0; g < KG; ++g) {
      if (k0 + g * MKC >= kend) break;
#pragma unroll
      for (int b = 0; b < MB; ++b)
        acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cw[g], cx[g][b], acc[b], 0, 0, 0);
    }
  }
}

// Block of outputs (of nb) and first row of a workgroup.  The blocks of rows lie
// in the grid's z, what passes its bound (ZMAX blocks of 32 rows, 2,097,120 rows)
// behind the blocks of outputs in x.  All of them in x: the division at the start
// costs a small network's forward pass 1.5 % (22.9 us), and at batch 33 the order of
// the blocks 7 % (25,992-512-512-19,494: 68.6 us).
constexpr int ZMAX = 65535;
template <int MB>
__device__ __forceinline__ bool rows_block(int M, int nb, int& nblk, int& m0) {
  const int q = (M - 1) / (16 * MB) >= ZMAX ? blockIdx.x / nb : 0;
  nblk = blockIdx.x - q * nb;
  const long first = ((long)q * ZMAX + blockIdx.z) * 16 * MB;
  m0 = (int)first;
  return first < M;                     // false: past the last row
}
static dim3 rows_grid(int nb, int nz, int M) {
  const unsigned gm = (unsigned)((M + 31) / 32);
  return dim3((unsigned)nb * ((gm + ZMAX - 1) / ZMAX), (unsigned)nz, gm < ZMAX ? gm : ZMAX);
}

// part[z][m][n] = sum over the k of split z; four waves of 16 n each
template <int MB>
__global__ __launch_bounds__(256) void k_rows_part(int M, int N, int K, int ks,
                                                   const float* __restrict__ X,
                                                   const __bf16* __restrict__ W,
                                                   float* __restrict__ part) {
  const int lane = threadIdx.x & 63;
  int nblk, m0;
  if (!rows_block<MB>(M, (N + 63) / 64, nblk, m0)) return;
  const int n0 = nblk * 64 + 16 * (threadIdx.x >> 6), z = blockIdx.y;
  if (n0 >= N) return;
  float4_t acc[MB];
  rows_times_weights<MB>(acc, M, N, K, m0, n0, z * ks, min(K, (z + 1) * ks), X, W);
#pragma unroll
  for (int b = 0; b < MB; ++b) {
    const int m = m0 + 16 * b + (lane & 15), n = n0 + 4 * (lane >> 4);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (m < M && n + q < N) part[((long)z * M + m) * N + n + q] = acc[b][q];
  }
}

// out[m][n] = sum_z (+ bias[n]) (relu) in one launch: one wave per split (up
// to four), 16 n per workgroup, the splits added in order through LDS
template <int MB>
__global__ __launch_bounds__(256) void k_rows_full(int M, int N, int K, int ks, int relu,
                                                   const float* __restrict__ X,
                                                   const __bf16* __restrict__ W,
                                                   const float* __restrict__ bias,
                                                   float* __restrict__ out) {
  __shared__ float4_t red[4][MB][64];
  const int lane = threadIdx.x & 63, z = threadIdx.x >> 6, nz = blockDim.x >> 6;
  int nblk, m0;
  if (!rows_block<MB>(M, (N + 15) / 16, nblk, m0)) return;
  const int n0 = nblk * 16;
  float4_t acc[MB];
  rows_times_weights<MB>(acc, M, N, K, m0, n0, z * ks, min(K, (z + 1) * ks), X, W);
#pragma unroll
  for (int b = 0; b < MB; ++b) red[z][b][lane] = acc[b];
  __syncthreads();
  if (z > 0) return;
#pragma unroll
  for (int b = 0; b < MB; ++b) {
    const int m = m0 + 16 * b + (lane & 15), n = n0 + 4 * (lane >> 4);
    float4_t s = {0.f, 0.f, 0.f, 0.f};
    for (int y = 0; y < nz; ++y) s += red[y][b][lane];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (m < M && n + q < N) {
        float v = s[q];
        if (bias) v += bias[n + q];
        if (relu) v = fmaxf(v, 0.f);
        out[(long)m * N + n + q] = v;
      }
  }
}

// part[z][m][n] = sum over the k of split z of X[m][k] W[k][n] (the weights of
// the layer above, read by columns): a chunk's 32 x 64 weights are loaded
// eight n per lane, KG chunks ahead, and turned through LDS into the operand
// layout (eight k per lane).
template <int MB>
__global__ __launch_bounds__(256) void k_cols_part(int M, int N, int K, int ks,
                                                   const float* __restrict__ X,
                                                   const __bf16* __restrict__ W,
                                                   float* __restrict__ part) {
  __shared__ __attribute__((aligned(16))) __bf16 Ws[2][64][MLD];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, ko = 8 * (lane >> 4);
  int nblk, m0;
  if (!rows_block<MB>(M, (N + 63) / 64, nblk, m0)) return;
  const int n0 = nblk * 64, z = blockIdx.y;
  const int kbeg = z * ks, kend = min(K, kbeg + ks);
  const int kr = t >> 3, nc = n0 + 8 * (t & 7);        // this thread's weights of a chunk
  const float* px[MB];
  float4_t acc[MB];
#pragma unroll
  for (int b = 0; b < MB; ++b) {
    px[b] = X + (long)min(m0 + 16 * b + (lane & 15), M - 1) * K;
    acc[b] = float4_t{0.f, 0.f, 0.f, 0.f};
  }
  bf16x8m_t wv[KG], x[KG][MB];
  const auto load = [&](int g, int k0) {
    wv[g] = k0 + kr < kend ? wgt8(W + (long)(k0 + kr) * N, nc, N) : wgt8(W, 0, 0);
#pragma unroll
    for (int b = 0; b < MB; ++b) x[g][b] = act8(px[b], k0 + ko, kend);
  };
#pragma unroll
  for (int g = 0; g < KG; ++g) load(g, kbeg + g * MKC);
  for (int k0 = kbeg; k0 < kend; k0 += KG * MKC) {
#pragma unroll
    for (int g = 0; g < KG; ++g) {
      if (k0 + g * MKC >= kend) break;
#pragma unroll
      for (int e = 0; e < 8; ++e) Ws[g & 1][8 * (t & 7) + e][kr] = wv[g][e];
      bf16x8m_t cx[MB];
#pragma unroll
      for (int b = 0; b < MB; ++b) cx[b] = x[g][b];
      load(g, k0 + (KG + g) * MKC);
      __syncthreads();             // the other buffer was last read before this barrier
      const bf16x8m_t b0 = *(const bf16x8m_t*)&Ws[g & 1][16 * w + (lane & 15)][ko];
#pragma unroll
      for (int b = 0; b < MB; ++b)
        acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b0, cx[b], acc[b], 0, 0, 0);
    }
  }
#pragma unroll
  for (int b = 0; b < MB; ++b) {
    const int m = m0 + 16 * b + (lane & 15), n = n0 + 16 * w + 4 * (lane >> 4);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (m < M && n + q < N) part[((long)z * M + m) * N + n + q] = acc[b][q];
  }
}

// out[m][n] = sum_z part[z][m][n] (+ bias[n]) (relu), zero where H is given
// and not positive (fixed summation order; eight loads in flight)
__global__ void k_split_reduce(int M, int N, int nsplit, const float* __restrict__ part,
                               const float* __restrict__ bias, int relu,
                               const float* __restrict__ H, float* __restrict__ out) {
  const long e = (long)blockIdx.x * blockDim.x + threadIdx.x, mn = (long)M * N;
  if (e >= mn) return;
  float s = 0.f;
  int z = 0;
  for (; z + 8 <= nsplit; z += 8) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = part[(z + u) * mn + e];
#pragma unroll
    for (int u = 0; u < 8; ++u) s += v[u];
  }
  for (; z < nsplit; ++z) s += part[z * mn + e];
  if (bias) s += bias[e % N];
  if (relu) s = fmaxf(s, 0.f);
  if (H && !(H[e] > 0.f)) s = 0.f;
  out[e] = s;
}

void mlp_gemm(int M, int N, int K, const float* A, long lda, const float* B, long ldb, float* part,
              int nsplit, hipStream_t st) {
  const int ks = ((K + nsplit - 1) / nsplit + MKC - 1) / MKC * MKC;
  const int nz = (K + ks - 1) / ks;
  dim3 g((N + MT - 1) / MT, (M + MT - 1) / MT, nz);
  k_gemm_bf16<<<g, 256, 0, st>>>(M, N, K, A, lda, B, ldb, part, ks);
}

int mlp_gemm_nsplit(int M, int N, int K, int nsplit) {
  const int ks = ((K + nsplit - 1) / nsplit + MKC - 1) / MKC * MKC;
  return (K + ks - 1) / ks;
}

void mlp_split_reduce(int M, int N, int nsplit, const float* part, const float* bias, int relu,
                      const float* H, float* out, hipStream_t st) {
  const long n = (long)M * N;
  k_split_reduce<<<(unsigned)((n + 63) / 64), 64, 0, st>>>(M, N, nsplit, part, bias, relu, H, out);
}

// out = X W^T (+ bias) (relu), W [N][K]
void mlp_rows(int M, int N, int K, const float* X, const __bf16* W, const float* bias, int relu,
              float* part, int nsplit, float* out, hipStream_t st) {
  const int ks = ((K + nsplit - 1) / nsplit + MKC - 1) / MKC * MKC;
  const int nz = (K + ks - 1) / ks;
  if (nz <= 4) {
    const dim3 g = rows_grid((N + 15) / 16, 1, M);
    if (M <= 16) k_rows_full<1><<<g, 64 * nz, 0, st>>>(M, N, K, ks, relu, X, W, bias, out);
    else k_rows_full<2><<<g, 64 * nz, 0, st>>>(M, N, K, ks, relu, X, W, bias, out);
    return;
  }
  const dim3 g = rows_grid((N + 63) / 64, nz, M);
  if (M <= 16) k_rows_part<1><<<g, 256, 0, st>>>(M, N, K, ks, X, W, part);
  else k_rows_part<2><<<g, 256, 0, st>>>(M, N, K, ks, X, W, part);
  mlp_split_reduce(M, N, nz, part, bias, relu, nullptr, out, st);
}

// out = X W, zero where H is not positive, W [K][N]
void mlp_cols(int M, int N, int K, const float* X, const __bf16* W, const float* H, float* part,
              int nsplit, float* out, hipStream_t st) {
  const int ks = ((K + nsplit - 1) / nsplit + MKC - 1) / MKC * MKC;
  const int nz = (K + ks - 1) / ks;
  const dim3 g = rows_grid((N + 63) / 64, nz, M);
  if (M <= 16) k_cols_part<1><<<g, 256, 0, st>>>(M, N, K, ks, X, W, part);
  else k_cols_part<2><<<g, 256, 0, st>>>(M, N, K, ks, X, W, part);
  mlp_split_reduce(M, N, nz, part, nullptr, 0, H, out, st);
}

// dY = (Y - T) / (B n); partial loss sums per block (fixed order)
__global__ __launch_bounds__(256) void k_loss_grad(long total, float scale, const float* __restrict__ Y,
                                                   const float* __restrict__ T, float* __restrict__ dY,
                                                   double* __restrict__ part) {
  __shared__ double red[256];
  double s = 0.0;
  for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < total; e += (long)gridDim.x * 256) {
    const float d = Y[e] - T[e];
    dY[e] = d * scale;
    s += (double)d * (double)d;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ void k_sum_parts(int n, const double* part, double scale, double* out) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    double s = 0.0;
    for (int i = 0; i < n; ++i) s += part[i];
    *out = s * scale;
  }
}

void mlp_loss_grad(long total, int n_out_times_b, const float* Y, const float* T, float* dY,
                   double* part, double* loss, hipStream_t st) {   // loss may be null
  const int nb = 256;
  k_loss_grad<<<nb, 256, 0, st>>>(total, 1.f / (float)n_out_times_b, Y, T, dY, part);
  if (loss) k_sum_parts<<<1, 1, 0, st>>>(nb, part, 0.5 / (double)n_out_times_b, loss);
}

// gb[n] = sum_m dZ[m][n]
__global__ void k_colsum(int M, int N, const float* __restrict__ dZ, float* __restrict__ gb) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  float s = 0.f;
  for (int m = 0; m < M; ++m) s += dZ[(long)m * N + n];
  gb[n] = s;
}

void mlp_colsum(int M, int N, const float* dZ, float* gb, hipStream_t st) {
  k_colsum<<<(N + 255) / 256, 256, 0, st>>>(M, N, dZ, gb);
}

struct AdamRate {
  float lr, b1, b2, eps, c1, c2;
};
// Adam with bias correction on an FP32 master weight; returns the new weight.
// (The fused multiply-adds are written out, so that every caller rounds alike.)
__device__ __forceinline__ float adam_update(float w, float g, float& m, float& v, const AdamRate& a) {
  const float me = fmaf(1.f - a.b1, g, a.b1 * m);
  const float ve = fmaf(g, (1.f - a.b2) * g, a.b2 * v);
  m = me;
  v = ve;
  return w - a.lr * (me / a.c1) / (sqrtf(ve / a.c2) + a.eps);
}

// One layer's weights W [M][N] with their gradient dZ^T X: dZ [B][M], X [B][N].
struct AdamLayer {
  const float *dZ, *X;
  float *w, *m, *v;
  __bf16* wb;
  int M, N, blk0;                  // first workgroup of the layer
};
struct AdamLayers {
  AdamLayer l[3];
};

// Gradient and Adam update of all weight matrices in one launch, one 64 x 64
// tile per workgroup: the gradient tile (BF16 operands, FP32 sums over the
// batch in k_gemm_bf16's order) goes through LDS to the threads that hold the
// same elements of the weight and its moments, so that it is never written to
// memory.  Bound by those three FP32 arrays read and written once, 26 B per
// weight with the BF16 copy (23.6M weights: 613 MB); their loads are issued
// before the product.
__global__ __launch_bounds__(256) void k_grad_adam(int B, AdamLayers ls, AdamRate rate) {
  __shared__ __attribute__((aligned(16))) __bf16 As[MT][MLD];
  __shared__ __attribute__((aligned(16))) __bf16 Bs[MT][MLD];
  __shared__ __attribute__((aligned(16))) float Gs[MT][MT + 4];
  const int blk = blockIdx.x;
  const AdamLayer L = blk >= ls.l[2].blk0 ? ls.l[2] : (blk >= ls.l[1].blk0 ? ls.l[1] : ls.l[0]);
  const int ntn = (L.N + MT - 1) / MT, b0 = blk - L.blk0;
  const int m0 = (b0 / ntn) * MT, n0 = (b0 % ntn) * MT;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int wr = w >> 1, wc = w & 1;
  // this thread's elements: rows m0 + (t >> 4) + 16 u, columns n0 + 4 (t & 15) ..
  const int n = n0 + 4 * (t & 15);
  const bool full = n + 4 <= L.N;
  float4u_t wv[4], mv[4], vv[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int m = m0 + (t >> 4) + 16 * u;
    if (m < L.M && full) {
      const long e = (long)m * L.N + n;
      wv[u] = *(const float4u_t*)&L.w[e];
      mv[u] = *(const float4u_t*)&L.m[e];
      vv[u] = *(const float4u_t*)&L.v[e];
    }
  }
  float4_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = float4_t{0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < B; k0 += MKC) {
    __syncthreads();
    stage(As, L.dZ, L.M, m0, L.M, k0, B);
    stage(Bs, L.X, L.N, n0, L.N, k0, B);
    __syncthreads();
    chunk_product(acc, As, Bs);
  }
#pragma unroll
  for (int mb = 0; mb < 2; ++mb)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
      *(float4_t*)&Gs[wr * 32 + mb * 16 + (lane & 15)][wc * 32 + nb * 16 + 4 * (lane >> 4)] = acc[mb][nb];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int r = (t >> 4) + 16 * u, m = m0 + r;
    if (m >= L.M) continue;
    const long e = (long)m * L.N + n;
    const float4_t g = *(const float4_t*)&Gs[r][4 * (t & 15)];
    if (full) {
      typedef __bf16 bf16x4u_t __attribute__((ext_vector_type(4), aligned(2)));
      bf16x4u_t o;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float me = mv[u][q], ve = vv[u][q];
        wv[u][q] = adam_update(wv[u][q], g[q], me, ve, rate);
        mv[u][q] = me;
        vv[u][q] = ve;
        o[q] = (__bf16)wv[u][q];
      }
      *(float4u_t*)&L.w[e] = wv[u];
      *(float4u_t*)&L.m[e] = mv[u];
      *(float4u_t*)&L.v[e] = vv[u];
      *(bf16x4u_t*)&L.wb[e] = o;
    } else {
      for (int q = 0; q < 4 && n + q < L.N; ++q) {
        float me = L.m[e + q], ve = L.v[e + q];
        const float we = adam_update(L.w[e + q], g[q], me, ve, rate);
        L.w[e + q] = we;
        L.m[e + q] = me;
        L.v[e + q] = ve;
        L.wb[e + q] = (__bf16)we;
      }
    }
  }
}

// The three bias vectors: gradient (column sums of dZ) and Adam update.
struct AdamBias {
  const float* dZ[3];
  float *w[3], *m[3], *v[3];
  int N[3];
};
__global__ void k_bias_adam(int B, AdamBias p, AdamRate rate) {
  int n = blockIdx.x * blockDim.x + threadIdx.x, k = 0;
  while (k < 3 && n >= p.N[k]) n -= p.N[k++];
  if (k == 3) return;
  float s = 0.f;
  for (int b = 0; b < B; ++b) s += p.dZ[k][(long)b * p.N[k] + n];
  float me = p.m[k][n], ve = p.v[k][n];
  p.w[k][n] = adam_update(p.w[k][n], s, me, ve, rate);
  p.m[k][n] = me;
  p.v[k][n] = ve;
}

// Adam step of the whole network; layer i of sizes M[i] x N[i], arrays packed
// as the parameters (offsets off[0..5]), BF16 copies at boff.
void mlp_grad_adam(int B, const int* M, const int* N, const float* const* dZ, const float* const* X,
                   float* w, float* m, float* v, __bf16* wb, const long* off, const long* boff,
                   float lr, int step, hipStream_t st) {
  AdamRate r;
  r.lr = lr;
  r.b1 = 0.9f;
  r.b2 = 0.999f;
  r.eps = 1e-8f;
  r.c1 = 1.f - powf(r.b1, (float)step);
  r.c2 = 1.f - powf(r.b2, (float)step);
  AdamLayers ls;
  AdamBias bs;
  int blk = 0, nb = 0;
  for (int i = 0; i < 3; ++i) {
    const long o = off[2 * i], ob = off[2 * i + 1];
    ls.l[i] = AdamLayer{dZ[i], X[i], w + o, m + o, v + o, wb + boff[i], M[i], N[i], blk};
    blk += ((M[i] + MT - 1) / MT) * ((N[i] + MT - 1) / MT);
    bs.dZ[i] = dZ[i];
    bs.w[i] = w + ob;
    bs.m[i] = m + ob;
    bs.v[i] = v + ob;
    bs.N[i] = M[i];
    nb += M[i];
  }
  k_grad_adam<<<(unsigned)blk, 256, 0, st>>>(B, ls, r);
  k_bias_adam<<<(unsigned)((nb + 63) / 64), 64, 0, st>>>(B, bs, r);
}

// dst[b][k] = src[rows[b]][k] * (k < n_scaled ? scale : 1), rows of n_cols floats.
__global__ void k_gather_rows_scaled(int n_cols, const float* __restrict__ src,
                                     const int32_t* __restrict__ rows, int n_scaled, float scale,
                                     float* __restrict__ dst) {
  const int b = blockIdx.y;
  const long r = rows[b];
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < n_cols; k += gridDim.x * blockDim.x) {
    const float v = src[r * n_cols + k];
    dst[(long)b * n_cols + k] = k < n_scaled ? v * scale : v;
  }
}

void mlp_gather_rows_scaled(int B, int n_cols, const float* src, const int32_t* rows, int n_scaled,
                            float scale, float* dst, hipStream_t st) {
  const int gx = std::min((n_cols + 255) / 256, 64);
  k_gather_rows_scaled<<<dim3(gx, B), 256, 0, st>>>(n_cols, src, rows, n_scaled, scale, dst);
}

// out = sum |a| / n over n floats, one workgroup, fixed order.
__global__ __launch_bounds__(1024) void k_abs_mean(long n, const float* __restrict__ a,
                                                   double* __restrict__ out) {
  __shared__ double red[1024];
  double s = 0.0;
  for (long e = threadIdx.x; e < n; e += 1024) s += fabs((double)a[e]);
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 512; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = n > 0 ? red[0] / (double)n : 0.0;
}

void mlp_abs_mean(long n, const float* a, double* out, hipStream_t st) {
  k_abs_mean<<<1, 1024, 0, st>>>(n, a, out);
}

__global__ void k_to_bf16(long n, const float* __restrict__ w, __bf16* __restrict__ wb) {
  const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n) wb[e] = (__bf16)w[e];
}

void mlp_to_bf16(long n, const float* w, __bf16* wb, hipStream_t st) {
  k_to_bf16<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(n, w, wb);
}

}  // namespace pdk
