// Dense float64 kernels for the coarsest level.
//
// Setup (once): blocked right-looking Cholesky A = L L^T with 64x64 tiles, the
// triangular inverse X = L^{-1} by doubling (pairs of inverted diagonal blocks joined
// into blocks of twice the size), and the lower tiles of A^{-1} = X^T X.  All of it
// runs on the FP64 matrix cores (v_mfma_f64_16x16x4f64); the 64x64 diagonal tiles are
// factored and inverted inside one workgroup in LDS, in panels of 16 columns.
// Measured at 4096 rows (the 64^3 setup, whose coarsest level it is, 40 -> 10 ms): the factorisation of a diagonal
// tile, the serial link of the chain, 181 -> 25 us; the inverse was a chain of 63 block rows,
// one narrow product after the other, and is now six batched products.
// Per cycle: x = A^{-1} b, one dense matrix-vector product per problem (the
// forward and back substitutions with L, applied through the inverse formed
// at setup: same bytes, no dependent sweep).
#include <algorithm>

#include "internal.h"

namespace amgp {

namespace {

typedef double dbl4 __attribute__((ext_vector_type(4)));

constexpr int TM = 64;  // output tile of a workgroup (TM x TM)
constexpr int TK = 16;  // k-chunk staged in LDS

// The 16x16x4 products of a 64x64 tile from K columns of A and rows of B: 256 threads = 4 waves in
// a 2x2 arrangement, each wave a 32x32 sub-tile of four 16x16 MFMA accumulators.
// MFMA 16x16x4 f64 operand layout: lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16];
// accumulator element r of lane l is D[l / 16 + 4 r][l % 16] (checked on gfx950).
// op(A)[m][k] = A[m * lda + k], or A[k * lda + m] (TA); op(B) likewise.
template <bool TA, bool TB>
__device__ __forceinline__ void tile_product(int K, const double* __restrict__ A, int lda,
                                             const double* __restrict__ B, int ldb, dbl4 (&acc)[2][2]) {
  __shared__ double As[TM][TK + 1];
  __shared__ double Bs[TK][TM + 1];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int wr = w >> 1, wc = w & 1;
  for (int a = 0; a < 2; ++a)
    for (int b = 0; b < 2; ++b) acc[a][b] = dbl4{0.0, 0.0, 0.0, 0.0};
  for (int k0 = 0; k0 < K; k0 += TK) {
    // stage A[0:64, k0:k0+16] and B[k0:k0+16, 0:64]: 1024 elements each, 4 per thread
    for (int e = t; e < TM * TK; e += 256) {
      int mm, kk;
      if (TA) {  // A^T: consecutive threads walk m (contiguous in memory)
        mm = e % TM;
        kk = e / TM;
        As[mm][kk] = A[(long long)(k0 + kk) * lda + mm];
      } else {
        kk = e % TK;
        mm = e / TK;
        As[mm][kk] = A[(long long)mm * lda + (k0 + kk)];
      }
      int nn, kb;
      if (TB) {
        kb = e % TK;
        nn = e / TK;
        Bs[kb][nn] = B[(long long)nn * ldb + (k0 + kb)];
      } else {
        nn = e % TM;
        kb = e / TM;
        Bs[kb][nn] = B[(long long)(k0 + kb) * ldb + nn];
      }
    }
    __syncthreads();
#pragma unroll
    for (int k4 = 0; k4 < TK; k4 += 4) {
      double av[2], bv[2];
      for (int a = 0; a < 2; ++a) av[a] = As[wr * 32 + a * 16 + (lane & 15)][k4 + (lane >> 4)];
      for (int b = 0; b < 2; ++b) bv[b] = Bs[k4 + (lane >> 4)][wc * 32 + b * 16 + (lane & 15)];
      for (int a = 0; a < 2; ++a)
        for (int b = 0; b < 2; ++b) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[b], acc[a][b], 0, 0, 0);
    }
    __syncthreads();
  }
}

// f(row, column, value) for this thread's elements of the 64x64 tile
template <typename F>
__device__ __forceinline__ void for_tile(const dbl4 (&acc)[2][2], F f) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int wr = w >> 1, wc = w & 1;
  for (int a = 0; a < 2; ++a)
    for (int b = 0; b < 2; ++b)
      for (int r = 0; r < 4; ++r)
        f(wr * 32 + a * 16 + (lane >> 4) + 4 * r, wc * 32 + b * 16 + (lane & 15), acc[a][b][r]);
}

// C = alpha op(A) op(B) for M, N, K multiples of 64 (row-major).  blockIdx.z = problem * inner + item:
// strides sX per problem and iX per item.
template <bool TA, bool TB>
__global__ __launch_bounds__(256) void k_gemm(int K, double alpha, const double* __restrict__ A, int lda,
                                              long long sA, long long iA, const double* __restrict__ B, int ldb,
                                              long long sB, long long iB, double* __restrict__ C, int ldc,
                                              long long sC, long long iC, int inner) {
  const long long p = blockIdx.z / inner, q = blockIdx.z % inner;
  const int m0 = blockIdx.y * TM, n0 = blockIdx.x * TM;
  A += p * sA + q * iA + (TA ? m0 : (long long)m0 * lda);
  B += p * sB + q * iB + (TB ? (long long)n0 * ldb : n0);
  C += p * sC + q * iC + (long long)m0 * ldc + n0;
  dbl4 acc[2][2];
  tile_product<TA, TB>(K, A, lda, B, ldb, acc);
  for_tile(acc, [&](int i, int j, double v) { C[(long long)i * ldc + j] = alpha * v; });
}

// The 16x16 products of the diagonal tile's factorisation, in LDS with rows of TM + 1: one wave's
// acc += A[r0:, k0:k0+16] op(B), op(B)[k][n] = B[k0 + k][c0 + n] or, TB, B[c0 + n][k0 + k].
template <bool TB>
__device__ __forceinline__ dbl4 mfma16(dbl4 acc, const double (*A)[TM + 1], int r0, int ka, const double (*B)[TM + 1],
                                       int kb, int c0, int lane) {
#pragma unroll
  for (int k4 = 0; k4 < 16; k4 += 4) {
    const int k = k4 + (lane >> 4);
    const double av = A[r0 + (lane & 15)][ka + k];
    const double bv = TB ? B[c0 + (lane & 15)][kb + k] : B[kb + k][c0 + (lane & 15)];
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc, 0, 0, 0);
  }
  return acc;
}

__device__ __forceinline__ double readlane_f64(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                          __builtin_amdgcn_readlane(__double2loint(v), l));
}

// Factor the 64x64 diagonal tile at (k, k) of every batch matrix in place
// (lower triangle := L_kk, upper := 0) and write inv(L_kk) to dinv.
// Panels of 16 columns: one wave factors a panel with a row per lane in registers, all four update
// the columns behind it; then the 16x16 diagonal blocks are inverted (a column per lane) and
// joined block row by block row.  (A column at a time over the whole tile, with three barriers per
// column and the inverse by one thread per column, took 181 us.)
__global__ __launch_bounds__(256) void k_potrf_tile(double* __restrict__ Ab, long long sA, int ld, int k,
                                                    double* __restrict__ dinv, long long sD,
                                                    int* __restrict__ flag) {
  __shared__ double T[TM][TM + 1];
  __shared__ double X[TM][TM + 1];
  constexpr int PB = 16, NP = TM / PB;
  double* A = Ab + blockIdx.x * sA + (long long)k * TM * ld + (long long)k * TM;
  double* D = dinv + blockIdx.x * sD;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  for (int e = t; e < TM * TM; e += 256) {
    T[e / TM][e % TM] = A[(long long)(e / TM) * ld + (e % TM)];
    X[e / TM][e % TM] = 0.0;
  }
  __syncthreads();
  for (int p = 0; p < NP; ++p) {
    const int c0 = p * PB;
    if (w == 0) {
      double r[PB];
      bool bad = false;
#pragma unroll
      for (int j = 0; j < PB; ++j) r[j] = T[lane][c0 + j];
#pragma unroll
      for (int c = 0; c < PB; ++c) {
        const double d = readlane_f64(r[c], c0 + c);
        bad = bad || !(d > 0.0);
        const double piv = sqrt(d > 0.0 ? d : 1.0);
        r[c] = lane == c0 + c ? piv : lane > c0 + c ? r[c] / piv : 0.0;
#pragma unroll
        for (int j = c + 1; j < PB; ++j) r[j] -= r[c] * readlane_f64(r[c], c0 + j);
      }
      if (bad && lane == 0) flag[F_NOTSPD] = 1;
#pragma unroll
      for (int j = 0; j < PB; ++j) T[lane][c0 + j] = lane >= c0 + j ? r[j] : 0.0;
    }
    __syncthreads();
    // lower 16x16 blocks (bi, bj), p < bj <= bi, of the columns behind: T -= L_bi,p L_bj,p^T
    const int m = NP - 1 - p;
    for (int q = w; q < m * (m + 1) / 2; q += 4) {
      int bi = 0;
      while ((bi + 1) * (bi + 2) / 2 <= q) ++bi;
      const int bj = q - bi * (bi + 1) / 2;
      const int r0 = (p + 1 + bi) * PB, n0 = (p + 1 + bj) * PB;
      const dbl4 acc = mfma16<true>(dbl4{0.0, 0.0, 0.0, 0.0}, T, r0, c0, T, c0, n0, lane);
      for (int e = 0; e < 4; ++e) T[r0 + (lane >> 4) + 4 * e][n0 + (lane & 15)] -= acc[e];
    }
    __syncthreads();
  }
  // inverse of the diagonal blocks: wave w inverts block w, lane c < 16 its column c (L X = I)
  if (lane < PB) {
    const int o = w * PB;
    double x[PB];
#pragma unroll
    for (int i = 0; i < PB; ++i) {
      double s = i == lane ? 1.0 : 0.0;
#pragma unroll
      for (int j = 0; j < i; ++j) s -= T[o + i][o + j] * x[j];
      x[i] = s / T[o + i][o + i];
    }
#pragma unroll
    for (int i = 0; i < PB; ++i) X[o + i][o + lane] = x[i];
  }
  __syncthreads();
  // block rows: X_ij = -X_ii sum_{j <= m < i} L_im X_mj, wave j on block column j; the sum waits
  // in the (still zero) block X_ji, transposed position, between the two products
  for (int i = 1; i < NP; ++i) {
    if (w < i) {
      dbl4 acc{0.0, 0.0, 0.0, 0.0};
      for (int m = w; m < i; ++m) acc = mfma16<false>(acc, T, i * PB, m * PB, X, m * PB, w * PB, lane);
      for (int e = 0; e < 4; ++e) X[w * PB + (lane >> 4) + 4 * e][i * PB + (lane & 15)] = acc[e];
    }
    __syncthreads();
    dbl4 acc{0.0, 0.0, 0.0, 0.0};
    if (w < i) {
#pragma unroll
      for (int k4 = 0; k4 < PB; k4 += 4) {
        const int kk = k4 + (lane >> 4);
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(X[i * PB + (lane & 15)][i * PB + kk],
                                                   X[w * PB + kk][i * PB + (lane & 15)], acc, 0, 0, 0);
      }
    }
    __syncthreads();
    if (w < i)
      for (int e = 0; e < 4; ++e) {
        X[i * PB + (lane >> 4) + 4 * e][w * PB + (lane & 15)] = -acc[e];
        X[w * PB + (lane >> 4) + 4 * e][i * PB + (lane & 15)] = 0.0;
      }
    __syncthreads();
  }
  for (int e = t; e < TM * TM; e += 256) {
    const int i = e / TM, j = e % TM;
    A[(long long)i * ld + j] = (j <= i) ? T[i][j] : 0.0;
    D[(long long)i * TM + j] = X[i][j];
  }
}

// Panel below diagonal tile k, a 64x64 tile per block: A_ik := A_ik inv(L_kk)^T, in place (a block
// reads and writes its own tile alone).
__global__ __launch_bounds__(256) void k_panel(double* __restrict__ Ab, long long sA, int ld, int k,
                                               const double* __restrict__ dinv, long long sD) {
  double* tile = Ab + blockIdx.y * sA + (long long)(k + 1 + blockIdx.x) * TM * ld + (long long)k * TM;
  dbl4 acc[2][2];
  tile_product<false, true>(TM, tile, ld, dinv + blockIdx.y * sD, TM, acc);
  // tile_product ends with a barrier: every read of the tile is done
  for_tile(acc, [&](int i, int j, double v) { tile[(long long)i * ld + j] = v; });
}

// Tile q = J (J + 1) / 2 + I of the packed lower triangle holds block (J, I), J >= I.
__device__ __forceinline__ void tile_of(int q, int& J, int& I) {
  J = (int)((sqrt(8.0 * q + 1.0) - 1.0) * 0.5);
  while ((J + 1) * (J + 2) / 2 <= q) ++J;
  while (J * (J + 1) / 2 > q) --J;
  I = q - J * (J + 1) / 2;
}

// Trailing update behind panel k, lower tiles alone: A_ij -= A_ik A_jk^T, k < j <= i.
__global__ __launch_bounds__(256) void k_trailing(double* __restrict__ Ab, long long sA, int ld, int k) {
  int J, I;
  tile_of(blockIdx.x, J, I);
  double* A = Ab + blockIdx.y * sA;
  const long long ri = (long long)(k + 1 + J) * TM * ld, rj = (long long)(k + 1 + I) * TM * ld;
  dbl4 acc[2][2];
  tile_product<false, true>(TM, A + ri + (long long)k * TM, ld, A + rj + (long long)k * TM, ld, acc);
  double* C = A + ri + (long long)(k + 1 + I) * TM;
  for_tile(acc, [&](int i, int j, double v) { C[(long long)i * ld + j] -= v; });
}

// copy the 64x64 tiles dinv into X's diagonal tiles
__global__ __launch_bounds__(256) void k_put_tiles(const double* __restrict__ D, long long sD, double* __restrict__ X,
                                                   long long sX, int ld) {
  const int i = blockIdx.x;
  const double* d = D + blockIdx.y * sD + (long long)i * TM * TM;
  double* x = X + blockIdx.y * sX + (long long)i * TM * ld + (long long)i * TM;
  for (int e = threadIdx.x; e < TM * TM; e += 256) x[(long long)(e / TM) * ld + (e % TM)] = d[e];
}

// Lower tile (J, I) of A^{-1} = X^T X, X lower triangular (its rows from block J on), into the
// packed contiguous tiles.
__global__ __launch_bounds__(256) void k_inverse_tiles(int np, int ntiles, const double* __restrict__ X,
                                                       double* __restrict__ packed) {
  int J, I;
  tile_of(blockIdx.x, J, I);
  const double* x = X + (long long)blockIdx.y * np * np + (long long)J * TM * np;
  dbl4 acc[2][2];
  tile_product<true, false>(np - J * TM, x + (long long)J * TM, np, x + (long long)I * TM, np, acc);
  double* dst = packed + ((long long)blockIdx.y * ntiles + blockIdx.x) * TM * TM;
  for_tile(acc, [&](int i, int j, double v) { dst[i * TM + j] = v; });
}

// One l1-Jacobi sweep on the columns of X (np x np, row-major): X_new = X + M^{-1} (I - A X), the sweep of
// k_jacobi for the right-hand sides e_c; a block serves 256 columns of one row.
__global__ __launch_bounds__(256) void k_sweep_columns(int n, int np, const int32_t* __restrict__ ptr,
                                                       const int32_t* __restrict__ col,
                                                       const double* __restrict__ val,
                                                       const double* __restrict__ minv, const double* __restrict__ X,
                                                       double* __restrict__ Xnew) {
  const int i = blockIdx.x, c = blockIdx.y * 256 + threadIdx.x;
  if (c >= n) return;
  double ax = 0.0;
#pragma unroll 4
  for (int p = ptr[i]; p < ptr[i + 1]; ++p) ax += val[p] * X[(long long)col[p] * np + c];
  const double b = i == c ? 1.0 : 0.0;
  Xnew[(long long)i * np + c] = X[(long long)i * np + c] + minv[i] * (b - ax);
}

__global__ void k_diagonal(int n, int np, const double* __restrict__ d, double* __restrict__ X) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) X[(long long)i * np + i] = d[i];
}

// Copy the lower 64x64 blocks of an np x np matrix into contiguous 32 KB tiles.
__global__ __launch_bounds__(256) void k_pack_tiles(int np, const double* __restrict__ dense,
                                                    double* __restrict__ packed) {
  int J, I;
  tile_of(blockIdx.x, J, I);
  const double* src = dense + (long long)J * TM * np + (long long)I * TM;
  double* dst = packed + (long long)blockIdx.x * TM * TM;
  for (int e = threadIdx.x; e < TM * TM; e += 256) dst[e] = src[(long long)(e / TM) * np + e % TM];
}

// x = A^{-1} b for the symmetric dense inverse, reading only its lower 64x64
// blocks, each exactly once, from the packed contiguous tiles.  Tile (J, I) of
// problem p is handled by one wavefront that streams its 64 rows (one 512 B
// load each): it contributes A_JI b_I to rows of block J (row sums, through an
// LDS transpose) and, when J > I, A_JI^T b_J to rows of block I (column sums,
// in registers).  The 64-vectors land in part[p][row block][column block]; a
// second kernel sums them in a fixed order.  b and x are level vectors (nl rows
// per problem); padding rows read as 0.
// RB: rows of the tile transposed through LDS at a time (RB x (TM + 1) doubles of LDS per
// wavefront); every row sum still adds its 64 products in column order.
template <typename T, int RB = TM>
__global__ __launch_bounds__(TM) void k_symv_tiles(int nb, int ntiles, int64_t nl, const double* __restrict__ packed,
                                                   const T* __restrict__ b, double* __restrict__ part) {
  __shared__ double prod[RB][TM + 1];
  const int q = blockIdx.x, p = blockIdx.y, lane = threadIdx.x;
  int J, I;
  tile_of(q, J, I);
  const T* bp = b + (int64_t)p * nl;
  const int64_t ri = (int64_t)I * TM + lane, rj = (int64_t)J * TM + lane;
  const double bI = ri < nl ? (double)bp[ri] : 0.0;
  const double bJ = rj < nl ? (double)bp[rj] : 0.0;
  const double* src = packed + ((int64_t)p * ntiles + q) * TM * TM + lane;
  double col = 0.0, row = 0.0;
  // the tiles (67 MB at 4096 rows) are read once per cycle with streaming loads, so that they do
  // not displace the fine level's matrix and vectors from the caches (measured at 128^3: 18.3 to
  // 16.2 us here, and the whole PCG solve 9.20 to 9.00 ms)
  for (int a0 = 0; a0 < TM; a0 += RB) {
#pragma unroll 16
    for (int a = 0; a < RB; ++a) {
      const double v = __builtin_nontemporal_load(src + (a0 + a) * TM);
      col += v * __shfl(bJ, a0 + a, TM);
      prod[a][lane] = v * bI;
    }
    __syncthreads();
    if (lane >= a0 && lane < a0 + RB) {
#pragma unroll 8
      for (int c = 0; c < TM; ++c) row += prod[lane - a0][c];
    }
    __syncthreads();
  }
  double* out = part + (int64_t)p * nb * nb * TM;
  out[((int64_t)J * nb + I) * TM + lane] = row;
  if (J > I) out[((int64_t)I * nb + J) * TM + lane] = col;
}

// x_I = sum_J part[I][J]: four waves each sum a quarter of the J range, combined in a fixed order.
template <typename T>
__global__ __launch_bounds__(256) void k_symv_sum(int nb, int64_t nl, const double* __restrict__ part,
                                                  T* __restrict__ x) {
  __shared__ double sm[4][TM];
  const int p = blockIdx.y, I = blockIdx.x, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const double* in = part + (int64_t)p * nb * nb * TM + (int64_t)I * nb * TM;
  const int per = (nb + 3) / 4;
  double s = 0.0;
  for (int J = w * per; J < min(nb, (w + 1) * per); ++J) s += in[(int64_t)J * TM + lane];
  sm[w][lane] = s;
  __syncthreads();
  if (w == 0) {
    const double tot = ((sm[0][lane] + sm[1][lane]) + sm[2][lane]) + sm[3][lane];
    const int64_t row = (int64_t)I * TM + lane;
    if (row < nl) x[(int64_t)p * nl + row] = (T)tot;
  }
}

}  // namespace

int dense_spd_inverse(hipStream_t s, int nbatch, int64_t np64, double* dense, double** packed, int* flag) {
  const int np = (int)np64;
  const int nb = np / TM, ntiles = nb * (nb + 1) / 2;
  const long long sA = (long long)np * np, sD = (long long)nb * TM * TM;
  double* dinv = nullptr;  // inverse diagonal tiles [batch][nb][64][64]
  double* X = nullptr;     // L^{-1}
  *packed = nullptr;
  const int rc = [&]() -> int {
    if (temp_malloc(&dinv, sizeof(double) * nbatch * sD) != hipSuccess ||
        temp_malloc(&X, sizeof(double) * nbatch * sA) != hipSuccess)
      return AMG_ENOMEM;
    // 1. Cholesky, right looking, on the lower tiles
    for (int k = 0; k < nb; ++k) {
      hipLaunchKernelGGL(k_potrf_tile, dim3(nbatch), dim3(256), 0, s, dense, sA, np, k,
                         dinv + (long long)k * TM * TM, sD, flag);
      const int rem = nb - 1 - k;
      if (rem == 0) break;
      hipLaunchKernelGGL(k_panel, dim3(rem, nbatch), dim3(256), 0, s, dense, sA, np, k,
                         (const double*)(dinv + (long long)k * TM * TM), sD);
      hipLaunchKernelGGL(k_trailing, dim3(rem * (rem + 1) / 2, nbatch), dim3(256), 0, s, dense, sA, np, k);
    }
    AMGP_HIP(hipGetLastError());
    // 2. X = L^{-1} by doubling: with the diagonal blocks of b tiles inverted, a pair (1, 2) of them
    // gives X_21 = -X_22 (L_21 X_11).  (L_21 X_11)^T waits where L's upper triangle has its block 12.
    AMGP_HIP(hipMemsetAsync(X, 0, sizeof(double) * nbatch * sA, s));
    hipLaunchKernelGGL(k_put_tiles, dim3(nb, nbatch), dim3(256), 0, s, (const double*)dinv, sD, X, sA, np);
    for (int b = 1; b < nb; b *= 2) {
      const long long step = 2LL * b * TM * (np + 1);  // from a pair's block 11 to the next pair's
      auto join = [&](long long from, int b2, int pairs) {  // b2 tiles in the second blocks
        const long long o = from * TM * (np + 1), d = (long long)b * TM;
        hipLaunchKernelGGL((k_gemm<true, true>), dim3(b2, b, nbatch * pairs), dim3(256), 0, s, b * TM, 1.0,
                           (const double*)X + o, np, sA, step, (const double*)dense + o + d * np, np, sA, step,
                           dense + o + d, np, sA, step, pairs);
        hipLaunchKernelGGL((k_gemm<false, true>), dim3(b, b2, nbatch * pairs), dim3(256), 0, s, b2 * TM, -1.0,
                           (const double*)X + o + d * (np + 1), np, sA, step, (const double*)dense + o + d, np, sA,
                           step, X + o + d * np, np, sA, step, pairs);
      };
      const int whole = nb / (2 * b), left = nb - whole * 2 * b;
      const int most = std::max(1, 65535 / nbatch);  // pairs of one launch (grid.z)
      for (int q = 0; q < whole; q += most) join(2LL * b * q, b, std::min(most, whole - q));
      if (left > b) join(2LL * b * whole, left - b, 1);
    }
    // 3. the lower tiles of A^{-1} = X^T X, in place of L (a setup holds two dense matrices at most)
    AMGP_HIP(hipGetLastError());
    dev_free(dense);
    dense = nullptr;
    if (keep_malloc(packed, sizeof(double) * (size_t)nbatch * ntiles * TM * TM) != hipSuccess) return AMG_ENOMEM;
    hipLaunchKernelGGL(k_inverse_tiles, dim3(ntiles, nbatch), dim3(256), 0, s, np, ntiles, (const double*)X, *packed);
    AMGP_HIP(hipGetLastError());
    AMGP_HIP(hipStreamSynchronize(s));
    return AMG_OK;
  }();
  if (rc != AMG_OK) hipStreamSynchronize(s);
  dev_free(dense);
  dev_free(dinv);
  dev_free(X);
  return rc;
}

int sweep_operator(hipStream_t s, int64_t n, int64_t np, const int32_t* ptr, const int32_t* col, const double* val,
                   const double* minv, int sweeps, double** packed) {
  const int nb = (int)(np / TM), ntiles = nb * (nb + 1) / 2;
  const size_t bytes = sizeof(double) * (size_t)np * np;
  double* X[2] = {nullptr, nullptr};
  *packed = nullptr;
  const int rc = [&]() -> int {
    if (temp_malloc(&X[0], bytes) != hipSuccess || temp_malloc(&X[1], bytes) != hipSuccess ||
        keep_malloc(packed, sizeof(double) * (size_t)ntiles * TM * TM) != hipSuccess)
      return AMG_ENOMEM;
    // the rows and columns past n stay zero in both
    AMGP_HIP(hipMemsetAsync(X[0], 0, bytes, s));
    AMGP_HIP(hipMemsetAsync(X[1], 0, bytes, s));
    hipLaunchKernelGGL(k_diagonal, dim3(grid_for(n)), dim3(kBlock), 0, s, (int)n, (int)np, minv, X[0]);
    for (int k = 1; k < sweeps; ++k) {
      hipLaunchKernelGGL(k_sweep_columns, dim3((unsigned)n, grid_for(n, 256)), dim3(256), 0, s, (int)n, (int)np, ptr,
                         col, val, minv, (const double*)X[0], X[1]);
      std::swap(X[0], X[1]);
    }
    hipLaunchKernelGGL(k_pack_tiles, dim3(ntiles), dim3(256), 0, s, (int)np, (const double*)X[0], *packed);
    AMGP_HIP(hipGetLastError());
    AMGP_HIP(hipStreamSynchronize(s));
    return AMG_OK;
  }();
  if (rc != AMG_OK) hipStreamSynchronize(s);
  dev_free(X[0]);
  dev_free(X[1]);
  return rc;
}

// Half a tile through LDS at a time (16.6 KB per wavefront instead of 33 KB, so twice the
// wavefronts per CU): 4096 rows 21.8 -> 19.7 us, 32 stacked problems of 4096 rows (2.2 GB of
// tiles) 428 -> 391 us; a quarter (16 rows) is slower (30.6 and 565 us).
constexpr int kSymvRows = 32;

template <typename T>
int launch_coarse_symv(hipStream_t s, int nbatch, int64_t nl, int64_t np, const double* ainv, const T* b, T* x,
                       double* part) {
  const int nb = (int)(np / TM), ntiles = nb * (nb + 1) / 2;
  hipLaunchKernelGGL((k_symv_tiles<T, kSymvRows>), dim3(ntiles, nbatch), dim3(TM), 0, s, nb, ntiles, nl, ainv, b, part);
  hipLaunchKernelGGL(k_symv_sum<T>, dim3(nb, nbatch), dim3(256), 0, s, nb, nl, (const double*)part, x);
  return hipGetLastError() == hipSuccess ? AMG_OK : AMG_EHIP;
}
template int launch_coarse_symv<double>(hipStream_t, int, int64_t, int64_t, const double*, const double*, double*,
                                        double*);
template int launch_coarse_symv<float>(hipStream_t, int, int64_t, int64_t, const double*, const float*, float*,
                                       double*);

}  // namespace amgp
