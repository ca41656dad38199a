// General sparse products for the hierarchies whose prolongator is not the
// plain 2x2x2 box indicator: the smoothed prolongator of Section 4,
// P = (I - omega D^{-1} A) P_hat, and box aggregates of any edge.  Setup only.
//
// * spgemm: C = X Y for CSR X (m x k) and Y (k x n), one wavefront per row of
//   C.  The distinct columns of the row are collected in an LDS hash table,
//   compacted and sorted; the values are then accumulated in X-row order
//   (the lanes of a wavefront take distinct entries of one Y row, so no two
//   lanes add to the same slot), which makes C bitwise reproducible.
// * drop_small: removes the entries whose magnitude is at most tau times the
//   largest of their row (tau = 2^-46): the Galerkin product and the smoothed
//   prolongator create exact cancellations that rounding turns into +-1e-17.
// * transpose: column counts, a scan, scatter, then each row of the
//   transpose sorted by column (unique keys), so the result is deterministic.
#include <algorithm>

#include "graph.h"
#include "internal.h"

namespace amgp {

namespace {

constexpr int kMaxHash = 4096;  // distinct columns per product row (LDS table size)

__device__ __forceinline__ unsigned hslot(int key, int cap) {
  return ((unsigned)key * 2654435761u) & (unsigned)(cap - 1);
}

// Insert key into the table; returns 1 if it was new, 0 if present, -1 if the table is full.
template <int CAP>
__device__ __forceinline__ int hinsert(int32_t* keys, int key) {
  unsigned h = hslot(key, CAP);
  for (int probe = 0; probe < CAP; ++probe) {
    const int old = atomicCAS(&keys[h], -1, key);
    if (old == -1) return 1;
    if (old == key) return 0;
    h = (h + 1) & (CAP - 1);
  }
  return -1;
}

// Upper bound of the row lengths of X Y: sum over the X row of the Y row lengths.
__global__ void k_prod_bound(int64_t m, const int32_t* __restrict__ xp, const int32_t* __restrict__ xc,
                             const int32_t* __restrict__ yp, int32_t* __restrict__ bound) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= m) return;
  int64_t s = 0;
  for (int p = xp[i]; p < xp[i + 1]; ++p) s += yp[xc[p] + 1] - yp[xc[p]];
  bound[i] = (int32_t)std::min<int64_t>(s, INT32_MAX);
}

// Symbolic pass: cnt[i] = number of distinct columns of row i of X Y.
template <int CAP>
__global__ __launch_bounds__(kWave) void k_spgemm_count(int64_t m, const int32_t* __restrict__ xp,
                                                        const int32_t* __restrict__ xc,
                                                        const int32_t* __restrict__ yp,
                                                        const int32_t* __restrict__ yc, int32_t* __restrict__ cnt,
                                                        int* flag) {
  __shared__ int32_t keys[CAP];
  __shared__ int nk;
  __shared__ int full;
  const int64_t i = blockIdx.x;
  if (i >= m) return;
  for (int t = threadIdx.x; t < CAP; t += kWave) keys[t] = -1;
  if (threadIdx.x == 0) {
    nk = 0;
    full = 0;
  }
  __syncthreads();
  for (int p = xp[i]; p < xp[i + 1]; ++p) {
    const int j = xc[p];
    for (int q = yp[j] + threadIdx.x; q < yp[j + 1]; q += kWave) {
      const int r = hinsert<CAP>(keys, yc[q]);
      if (r == 1) atomicAdd(&nk, 1);
      if (r < 0) full = 1;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    cnt[i] = nk;
    if (full || nk > CAP * 3 / 4) atomicOr(&flag[F_CAPACITY], 1);
  }
}

// Numeric pass: row i of X Y in columns cols[cptr[i] ...] (ascending) and values.
template <int CAP>
__global__ __launch_bounds__(kWave) void k_spgemm_fill(int64_t m, const int32_t* __restrict__ xp,
                                                       const int32_t* __restrict__ xc, const double* __restrict__ xv,
                                                       const int32_t* __restrict__ yp, const int32_t* __restrict__ yc,
                                                       const double* __restrict__ yv, const int32_t* __restrict__ cptr,
                                                       int32_t* __restrict__ ccol, double* __restrict__ cval) {
  __shared__ int32_t keys[CAP];
  __shared__ int32_t list[CAP];
  __shared__ double acc[CAP];
  __shared__ int nk;
  const int64_t i = blockIdx.x;
  if (i >= m) return;
  const int lane = threadIdx.x;
  for (int t = lane; t < CAP; t += kWave) keys[t] = -1;
  if (lane == 0) nk = 0;
  __syncthreads();
  for (int p = xp[i]; p < xp[i + 1]; ++p) {
    const int j = xc[p];
    for (int q = yp[j] + lane; q < yp[j + 1]; q += kWave) hinsert<CAP>(keys, yc[q]);
    __syncthreads();
  }
  // compact the occupied slots (their order is fixed by the table, not by timing)
  for (int t0 = 0; t0 < CAP; t0 += kWave) {
    const int key = keys[t0 + lane];
    const unsigned long long m_ = __ballot(key >= 0);
    const int before = __popcll(m_ & ((1ull << lane) - 1ull));
    const int base = nk;
    if (key >= 0) list[base + before] = key;
    __syncthreads();
    if (lane == 0) nk = base + __popcll(m_);
    __syncthreads();
  }
  const int len = nk;
  int pw = 1;
  while (pw < len) pw <<= 1;
  for (int t = len + lane; t < pw; t += kWave) list[t] = INT32_MAX;
  __syncthreads();
  // bitonic sort of list[0, pw)
  for (int size = 2; size <= pw; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int t = lane; t < pw; t += kWave) {
        const int u = t ^ stride;
        if (u > t) {
          const bool up = (t & size) == 0;
          const int a = list[t], b = list[u];
          if ((a > b) == up) {
            list[t] = b;
            list[u] = a;
          }
        }
      }
      __syncthreads();
    }
  }
  for (int t = lane; t < len; t += kWave) acc[t] = 0.0;
  __syncthreads();
  for (int p = xp[i]; p < xp[i + 1]; ++p) {
    const int j = xc[p];
    const double a = xv[p];
    for (int q = yp[j] + lane; q < yp[j + 1]; q += kWave) {
      const int key = yc[q];
      int lo = 0, hi = len - 1;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (list[mid] < key) lo = mid + 1; else hi = mid;
      }
      acc[lo] += a * yv[q];
    }
    __syncthreads();
  }
  const int base = cptr[i];
  for (int t = lane; t < len; t += kWave) {
    ccol[base + t] = list[t];
    cval[base + t] = acc[t];
  }
}

__global__ void k_keep_count(int64_t m, const int32_t* __restrict__ ptr, const double* __restrict__ val, double tau,
                             int32_t* __restrict__ kept) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= m) return;
  double mx = 0.0;
  for (int p = ptr[i]; p < ptr[i + 1]; ++p) mx = fmax(mx, fabs(val[p]));
  int c = 0;
  for (int p = ptr[i]; p < ptr[i + 1]; ++p) c += fabs(val[p]) > tau * mx;
  kept[i] = c;
}

__global__ void k_keep_copy(int64_t m, const int32_t* __restrict__ ptr, const int32_t* __restrict__ col,
                            const double* __restrict__ val, double tau, const int32_t* __restrict__ optr,
                            int32_t* __restrict__ ocol, double* __restrict__ oval) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= m) return;
  double mx = 0.0;
  for (int p = ptr[i]; p < ptr[i + 1]; ++p) mx = fmax(mx, fabs(val[p]));
  int o = optr[i];
  for (int p = ptr[i]; p < ptr[i + 1]; ++p) {
    if (fabs(val[p]) > tau * mx) {
      ocol[o] = col[p];
      oval[o] = val[p];
      ++o;
    }
  }
}

__global__ void k_col_count(int64_t nnz, const int32_t* __restrict__ col, int32_t* __restrict__ cnt) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < nnz) atomicAdd(&cnt[col[q]], 1);
}

__global__ void k_transpose_scatter(int64_t m, const int32_t* __restrict__ ptr, const int32_t* __restrict__ col,
                                    const double* __restrict__ val, const int32_t* __restrict__ tptr,
                                    int32_t* __restrict__ fill, int32_t* __restrict__ tcol,
                                    double* __restrict__ tval) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= m) return;
  for (int p = ptr[i]; p < ptr[i + 1]; ++p) {
    const int c = col[p];
    const int o = tptr[c] + atomicAdd(&fill[c], 1);
    tcol[o] = (int32_t)i;
    tval[o] = val[p];
  }
}

// Sorting the rows of the transpose by column (the keys of a row are distinct, so the result
// is unique): rows of up to kShortRow entries by one thread each (insertion sort), longer ones
// by one wavefront each (bitonic network in LDS, up to kSortCap entries).
constexpr int kShortRow = 64;
constexpr int kSortCap = 4096;

__device__ void insertion_sort_row(int32_t* __restrict__ col, double* __restrict__ val, int len) {
  for (int p = 1; p < len; ++p) {
    const int c = col[p];
    const double v = val[p];
    int q = p - 1;
    while (q >= 0 && col[q] > c) {
      col[q + 1] = col[q];
      val[q + 1] = val[q];
      --q;
    }
    col[q + 1] = c;
    val[q + 1] = v;
  }
}

__global__ void k_row_sort(int64_t m, const int32_t* __restrict__ ptr, int32_t* __restrict__ col,
                           double* __restrict__ val) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= m) return;
  const int b = ptr[i], len = ptr[i + 1] - b;
  if (len <= kShortRow) insertion_sort_row(col + b, val + b, len);
}

// One wavefront per listed row longer than kShortRow.
__global__ __launch_bounds__(kWave) void k_row_sort_long(const int32_t* __restrict__ rows,
                                                         const int32_t* __restrict__ ptr, int32_t* __restrict__ col,
                                                         double* __restrict__ val) {
  __shared__ int32_t key[kSortCap];
  __shared__ double v[kSortCap];
  const int i = rows[blockIdx.x];
  const int b = ptr[i], len = ptr[i + 1] - b;
  const int lane = threadIdx.x;
  if (len > kSortCap) {
    if (lane == 0) insertion_sort_row(col + b, val + b, len);
    return;
  }
  int pw = 1;
  while (pw < len) pw <<= 1;
  for (int t = lane; t < pw; t += kWave) {
    key[t] = t < len ? col[b + t] : INT_MAX;
    v[t] = t < len ? val[b + t] : 0.0;
  }
  __syncthreads();
  for (int size = 2; size <= pw; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int t = lane; t < pw; t += kWave) {
        const int u = t ^ stride;
        if (u > t) {
          const bool up = (t & size) == 0;
          const int ka = key[t], kb = key[u];
          if ((ka > kb) == up) {
            key[t] = kb;
            key[u] = ka;
            const double va = v[t];
            v[t] = v[u];
            v[u] = va;
          }
        }
      }
      __syncthreads();
    }
  }
  for (int t = lane; t < len; t += kWave) {
    col[b + t] = key[t];
    val[b + t] = v[t];
  }
}

// Diagonal and ||row of D^{-1} A||_1 of every row; the largest ratio of each stacked problem is
// accumulated into lam[p] (non-negative doubles order like their bit patterns).
__global__ void k_diag_ratio(int64_t n, int64_t rpp, const int32_t* __restrict__ ptr, const int32_t* __restrict__ col,
                             const double* __restrict__ val, double* __restrict__ diag,
                             unsigned long long* __restrict__ lam, int* flag) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double d = 0.0, s = 0.0;
  for (int p = ptr[i]; p < ptr[i + 1]; ++p) {
    if (col[p] == i) d = val[p];
    s += fabs(val[p]);
  }
  if (!(d > 0.0)) {
    atomicOr(&flag[F_NOTSPD], 1);
    d = 1.0;
  }
  diag[i] = d;
  atomicMax(&lam[i / rpp], (unsigned long long)__double_as_longlong(s / d));
}

// P = P_hat - omega_p D^{-1} (A P_hat), in place on the pattern of A P_hat, which holds the
// single entry (hcol[i], hval[i]) of row i of P_hat.
__global__ void k_smooth_prol(int64_t n, int64_t rpp, const int32_t* __restrict__ ptr, const int32_t* __restrict__ col,
                              double* __restrict__ val, const int32_t* __restrict__ hcol,
                              const double* __restrict__ hval, const double* __restrict__ diag,
                              const double* __restrict__ omega) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double s = omega[i / rpp] / diag[i];
  const int a = hcol[i];
  const double h = hval[i];
  for (int p = ptr[i]; p < ptr[i + 1]; ++p) val[p] = (col[p] == a ? h : 0.0) - s * val[p];
}

__global__ void k_identity_rows(int64_t n, const int32_t* __restrict__ agg, int32_t* __restrict__ ptr,
                                int32_t* __restrict__ col, double* __restrict__ val) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i > n) return;
  ptr[i] = (int32_t)i;
  if (i < n) {
    col[i] = agg[i];
    val[i] = 1.0;
  }
}

// Exclusive scan of counts, each rounded up to a multiple of div in units of it and scaled, in
// chunks: their sums, the sums' scan by one block (the total last), and the chunks' own scans.
// ptr may be cnt.
constexpr int kScanPer = 16;
constexpr int kScanChunk = kBlock * kScanPer;

__device__ __forceinline__ int64_t scan_value(const int32_t* cnt, int64_t i, int64_t m, int div, int scale) {
  return i < m ? (int64_t)((cnt[i] + div - 1) / div) * scale : 0;
}

// inclusive scan over a block of up to 1024 threads; every thread gets the total too
__device__ __forceinline__ int64_t block_scan(int64_t v, int64_t* total) {
  __shared__ int64_t wsum[1024 / kWave];
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave, nw = blockDim.x / kWave;
  for (int off = 1; off < kWave; off <<= 1) {
    const int64_t u = __shfl_up(v, off, kWave);
    if (lane >= off) v += u;
  }
  if (lane == kWave - 1) wsum[w] = v;
  __syncthreads();
  int64_t before = 0, all = 0;
  for (int k = 0; k < nw; ++k) {
    if (k < w) before += wsum[k];
    all += wsum[k];
  }
  __syncthreads();
  *total = all;
  return v + before;
}

__global__ __launch_bounds__(kBlock) void k_scan_part(int64_t m, const int32_t* __restrict__ cnt, int div, int scale,
                                                      int64_t* __restrict__ part) {
  int64_t v = 0, total;
  for (int k = 0; k < kScanPer; ++k)
    v += scan_value(cnt, (int64_t)blockIdx.x * kScanChunk + k * kBlock + threadIdx.x, m, div, scale);
  block_scan(v, &total);
  if (threadIdx.x == 0) part[blockIdx.x] = total;
}

__global__ __launch_bounds__(1024) void k_scan_top(int64_t nb, int64_t* __restrict__ part) {
  int64_t carry = 0;
  for (int64_t b0 = 0; b0 < nb; b0 += 1024) {
    const int64_t i = b0 + threadIdx.x;
    const int64_t v = i < nb ? part[i] : 0;
    int64_t total;
    const int64_t incl = block_scan(v, &total);
    if (i < nb) part[i] = carry + incl - v;
    carry += total;
  }
  if (threadIdx.x == 0) part[nb] = carry;
}

__global__ __launch_bounds__(kBlock) void k_scan_write(int64_t m, int64_t nb, const int32_t* cnt, int div, int scale,
                                                       const int64_t* __restrict__ part, int32_t* ptr) {
  int64_t carry = nb > 0 ? part[blockIdx.x] : 0;
  for (int k = 0; k < kScanPer; ++k) {
    const int64_t i = (int64_t)blockIdx.x * kScanChunk + k * kBlock + threadIdx.x;
    const int64_t v = scan_value(cnt, i, m, div, scale);
    int64_t total;
    const int64_t incl = block_scan(v, &total);
    if (i < m) ptr[i] = (int32_t)(carry + incl - v);
    carry += total;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) ptr[m] = (int32_t)part[nb];
}

// the largest of m counts into *most (zeroed beforehand)
__global__ __launch_bounds__(kBlock) void k_max_count(int64_t m, const int32_t* __restrict__ cnt,
                                                      int32_t* __restrict__ most) {
  int v = 0;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < m; i += (int64_t)gridDim.x * kBlock)
    v = max(v, cnt[i]);
  for (int off = 32; off > 0; off >>= 1) v = max(v, __shfl_xor(v, off, kWave));
  if ((threadIdx.x & (kWave - 1)) == 0) atomicMax(most, v);
}

__global__ void k_row_lengths(int64_t m, const int32_t* __restrict__ ptr, int32_t* __restrict__ len) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < m) len[i] = ptr[i + 1] - ptr[i];
}

// rows longer than kShortRow, in any order: list[0, *count)
__global__ void k_long_rows(int64_t m, const int32_t* __restrict__ ptr, int32_t* __restrict__ list,
                            int32_t* __restrict__ count) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < m && ptr[i + 1] - ptr[i] > kShortRow) list[atomicAdd(count, 1)] = (int32_t)i;
}

// transpose of the box prolongator (one entry 1.0 per row) from the aggregates' rows
__global__ void k_children_count(int64_t nc, const int32_t* __restrict__ ch, int32_t* __restrict__ cnt) {
  const int64_t I = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (I >= nc) return;
  int c = 0;
  while (c < kMaxChildren && ch[I * kMaxChildren + c] >= 0) ++c;
  cnt[I] = c;
}

__global__ void k_children_rows(int64_t nc, const int32_t* __restrict__ ch, const int32_t* __restrict__ ptr,
                                int32_t* __restrict__ col, double* __restrict__ val) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t I = t / kMaxChildren;
  const int c = (int)(t % kMaxChildren);
  if (I >= nc || c >= ptr[I + 1] - ptr[I]) return;
  col[ptr[I] + c] = ch[t];
  val[ptr[I] + c] = 1.0;
}

// Row I of A_c = P^T A P for the box P (one entry 1.0 per row), one wavefront per row.  Row I of R = P^T A
// (at most 64 entries) names its columns: the first lane of each aggregate J = agg[column] owns J.
// The entries of the aggregate's rows then pass through LDS 64 at a time, sorted by owner in their order, and
// every owner adds its own ones up, so that each sum takes the products row by row and in ascending
// column order as k_rap does, to the same bits.  Sums that are exactly zero (or no number) are left out.
// FILL = false: counts.  Bound by the instructions per entry, not by its 12 bytes.  Measured on the
// 27-point 320^3 matrix, both passes: 79.8 ms with k_rap (one thread per coarse row, 216 entries sorted by
// insertion into a list in scratch memory), 18.2 ms here.  A_c as R P, 64 entries a row, took 15.9 ms, but its
// sums associate otherwise: the V-cycle on 131 x 127 x 125 trilinear elements was then 8.3e-16 instead of
// 6.5e-16 from its 64-bit values.
constexpr int kOwnerHash = 2 * kWave;

template <bool FILL>
__global__ __launch_bounds__(kWave) void k_galerkin_rows(
    const int32_t* __restrict__ ptr, const int32_t* __restrict__ col, const double* __restrict__ val,
    const int32_t* __restrict__ ch, const int32_t* __restrict__ rptr, const int32_t* __restrict__ rcol,
    const int32_t* __restrict__ agg, int32_t* __restrict__ cnt_or_ptr, int32_t* __restrict__ ccol,
    double* __restrict__ cval) {
  __shared__ int32_t key[kOwnerHash], owner[kOwnerHash];
  __shared__ double sorted[kWave];
  __shared__ int32_t count[kWave], start[kWave];
  const int lane = threadIdx.x;
  const int64_t I = blockIdx.x;
  const int beg = rptr[I], len = rptr[I + 1] - beg;
  const int J = lane < len ? agg[rcol[beg + lane]] : INT_MAX;
  for (int t = lane; t < kOwnerHash; t += kWave) {
    key[t] = -1;
    owner[t] = kWave;
  }
  __syncthreads();
  unsigned mine = hslot(J, kOwnerHash);
  if (lane < len) {
    for (;;) {  // at most 64 keys: a free place is always found
      const int old = atomicCAS(&key[mine], -1, J);
      if (old == -1 || old == J) break;
      mine = (mine + 1) & (kOwnerHash - 1);
    }
    atomicMin(&owner[mine], lane);
  }
  __syncthreads();
  // lane c < 8: child row c, where its entries begin and how many come before them
  const int child = lane < kMaxChildren ? ch[I * kMaxChildren + lane] : -1;
  const int cbeg = child >= 0 ? ptr[child] : 0;
  int upto = child >= 0 ? ptr[child + 1] - cbeg : 0;
  const int clen = upto;
  for (int off = 1; off < kMaxChildren; off <<= 1) {
    const int u = __shfl_up(upto, off, kWave);
    if (lane >= off) upto += u;
  }
  const int total = __builtin_amdgcn_readlane(upto, kMaxChildren - 1);
  const int before = upto - clen;
  double sum = 0.0;
  for (int e0 = 0; e0 < total; e0 += kWave) {
    const int e = e0 + lane;
    int p = 0;
#pragma unroll
    for (int c = 0; c < kMaxChildren; ++c) {
      const int first = __builtin_amdgcn_readlane(before, c);
      if (e >= first) p = __builtin_amdgcn_readlane(cbeg, c) + (e - first);
    }
    int slot = kWave;
    double v = 0.0;
    if (e < total) {
      const int Je = agg[col[p]];
      v = val[p];
      unsigned h = hslot(Je, kOwnerHash);
      for (int probe = 0; probe < kOwnerHash && slot == kWave; ++probe, h = (h + 1) & (kOwnerHash - 1))
        if (key[h] == Je) slot = owner[h];
    }
    const bool has = slot < kWave;  // R holds every column of these rows
    unsigned long long same = __ballot(has);  // the lanes whose entries have this owner
#pragma unroll
    for (int b = 0; b < 6; ++b) {
      const unsigned long long set = __ballot((slot >> b) & 1);
      same &= (slot >> b) & 1 ? set : ~set;
    }
    const int rank = __popcll(same & ((1ull << lane) - 1));
    count[lane] = 0;
    __syncthreads();
    if (has && rank == 0) count[slot] = __popcll(same);
    __syncthreads();
    const int n = count[lane];
    int at = n;
    for (int off = 1; off < kWave; off <<= 1) {
      const int u = __shfl_up(at, off, kWave);
      if (lane >= off) at += u;
    }
    at -= n;
    start[lane] = at;
    __syncthreads();
    if (has) sorted[start[slot] + rank] = v;
    __syncthreads();
    for (int q = 0; q < n; ++q) sum += sorted[at + q];
    __syncthreads();
  }
  const bool keep = lane < len && owner[mine] == lane && fabs(sum) > 0.0;
  const unsigned long long kept = __ballot(keep);
  if constexpr (!FILL) {
    if (lane == 0) cnt_or_ptr[I] = __popcll(kept);
  } else {
    int rank = 0;
    for (unsigned long long m = kept; m; m &= m - 1)
      rank += __builtin_amdgcn_readlane(J, __builtin_amdgcn_readfirstlane(__ffsll(m) - 1)) < J;
    if (keep) {
      const int q = cnt_or_ptr[I] + rank;
      ccol[q] = J;
      cval[q] = sum;
    }
  }
}

template <int CAP>
void go_spgemm(bool fill, hipStream_t s, int64_t m, const Csr& X, const Csr& Y, int32_t* cnt, const int32_t* cptr,
               int32_t* ccol, double* cval, int* flag) {
  if (!fill)
    hipLaunchKernelGGL(k_spgemm_count<CAP>, dim3((unsigned)m), dim3(kWave), 0, s, m, X.ptr, X.col, Y.ptr, Y.col,
                       cnt, flag);
  else
    hipLaunchKernelGGL(k_spgemm_fill<CAP>, dim3((unsigned)m), dim3(kWave), 0, s, m, X.ptr, X.col, X.val, Y.ptr,
                       Y.col, Y.val, cptr, ccol, cval);
}

int run_spgemm(int cap, bool fill, hipStream_t s, int64_t m, const Csr& X, const Csr& Y, int32_t* cnt,
               const int32_t* cptr, int32_t* ccol, double* cval, int* flag) {
  switch (cap) {
    case 64: go_spgemm<64>(fill, s, m, X, Y, cnt, cptr, ccol, cval, flag); break;
    case 128: go_spgemm<128>(fill, s, m, X, Y, cnt, cptr, ccol, cval, flag); break;
    case 256: go_spgemm<256>(fill, s, m, X, Y, cnt, cptr, ccol, cval, flag); break;
    case 512: go_spgemm<512>(fill, s, m, X, Y, cnt, cptr, ccol, cval, flag); break;
    case 1024: go_spgemm<1024>(fill, s, m, X, Y, cnt, cptr, ccol, cval, flag); break;
    case 2048: go_spgemm<2048>(fill, s, m, X, Y, cnt, cptr, ccol, cval, flag); break;
    default: go_spgemm<4096>(fill, s, m, X, Y, cnt, cptr, ccol, cval, flag); break;
  }
  return hipGetLastError() == hipSuccess ? AMG_OK : AMG_EHIP;
}

int read_flag(hipStream_t s, const int* flag, int which) {
  int h[F_NFLAG];
  if (hipMemcpyAsync(h, flag, sizeof(h), hipMemcpyDeviceToHost, s) != hipSuccess) return -1;
  if (hipStreamSynchronize(s) != hipSuccess) return -1;
  return h[which];
}

}  // namespace

int64_t scan_ptr(hipStream_t s, int64_t m, const int32_t* cnt, int32_t* ptr, int* rc, int div, int scale) {
  graph::DevBuf<int64_t> part;
  const int64_t nb = (m + kScanChunk - 1) / kScanChunk;
  *rc = part.alloc(nb + 1);
  if (*rc != AMG_OK) return -1;
  int64_t total = 0;
  if (nb > 0)
    hipLaunchKernelGGL(k_scan_part, dim3((unsigned)nb), dim3(kBlock), 0, s, m, cnt, div, scale, part.p);
  hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(1024), 0, s, nb, part.p);
  hipLaunchKernelGGL(k_scan_write, dim3((unsigned)std::max<int64_t>(nb, 1)), dim3(kBlock), 0, s, m, nb, cnt, div, scale,
                     (const int64_t*)part.p, ptr);
  if (hipMemcpyAsync(&total, part.p + nb, sizeof(total), hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess) {
    *rc = AMG_EHIP;
    return -1;
  }
  if (total >= (int64_t)INT32_MAX) {
    *rc = AMG_ECAPACITY;
    return -1;
  }
  return total;
}

void free_csr(Csr& a) {
  dev_free(a.ptr);
  dev_free(a.col);
  dev_free(a.val);
  a = Csr();
}

// largest of m counts; scratch: one device int
int64_t max_count(hipStream_t s, int64_t m, const int32_t* cnt, int32_t* scratch, int* rc) {
  int32_t most = 0;
  *rc = AMG_OK;
  if (hipMemsetAsync(scratch, 0, sizeof(int32_t), s) != hipSuccess) *rc = AMG_EHIP;
  hipLaunchKernelGGL(k_max_count, dim3(std::min(1024u, grid_for(m))), dim3(kBlock), 0, s, m, cnt, scratch);
  if (hipMemcpyAsync(&most, scratch, sizeof(most), hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess)
    *rc = AMG_EHIP;
  return most;
}

int spgemm(hipStream_t s, const Csr& X, const Csr& Y, Csr* C, int* flag) {
  const int64_t m = X.m;
  *C = Csr();
  if (m <= 0 || m > (int64_t)UINT32_MAX) return AMG_EINVAL;
  int32_t* cnt = nullptr;
  if (temp_malloc(&cnt, sizeof(int32_t) * (m + 1)) != hipSuccess) return AMG_ENOMEM;
  // table size: the smallest power of two of at least twice the longest row bound
  hipLaunchKernelGGL(k_prod_bound, dim3(grid_for(m)), dim3(kBlock), 0, s, m, X.ptr, X.col, Y.ptr, cnt);
  int rc = AMG_OK;
  const int64_t bound = max_count(s, m, cnt, cnt + m, &rc);
  if (rc != AMG_OK) {
    dev_free(cnt);
    return rc;
  }
  int cap = 64;
  while (cap < 2 * bound && cap < kMaxHash) cap <<= 1;
  rc = run_spgemm(cap, false, s, m, X, Y, cnt, nullptr, nullptr, nullptr, flag);
  if (rc != AMG_OK) {
    dev_free(cnt);
    return rc;
  }
  const int full = read_flag(s, flag, F_CAPACITY);
  if (full != 0) {
    dev_free(cnt);
    return full < 0 ? AMG_EHIP : AMG_ECAPACITY;
  }
  Csr c;
  c.m = m;
  c.ncols = Y.ncols;
  if (temp_malloc(&c.ptr, sizeof(int32_t) * (m + 1)) != hipSuccess) {
    dev_free(cnt);
    return AMG_ENOMEM;
  }
  const int64_t nnz = scan_ptr(s, m, cnt, c.ptr, &rc);
  dev_free(cnt);
  if (rc != AMG_OK) {
    free_csr(c);
    return rc;
  }
  c.nnz = nnz;
  if (temp_malloc(&c.col, sizeof(int32_t) * std::max<int64_t>(nnz, 1)) != hipSuccess ||
      temp_malloc(&c.val, sizeof(double) * std::max<int64_t>(nnz, 1)) != hipSuccess) {
    free_csr(c);
    return AMG_ENOMEM;
  }
  rc = run_spgemm(cap, true, s, m, X, Y, nullptr, c.ptr, c.col, c.val, flag);
  if (rc == AMG_OK && hipStreamSynchronize(s) != hipSuccess) rc = AMG_EHIP;
  if (rc != AMG_OK) {
    free_csr(c);
    return rc;
  }
  *C = c;
  return AMG_OK;
}

int drop_small(hipStream_t s, Csr* a, double tau) {
  Csr o;
  o.m = a->m;
  o.ncols = a->ncols;
  int32_t* kept = nullptr;
  if (temp_malloc(&kept, sizeof(int32_t) * (a->m + 1)) != hipSuccess) return AMG_ENOMEM;
  hipLaunchKernelGGL(k_keep_count, dim3(grid_for(a->m)), dim3(kBlock), 0, s, a->m, a->ptr, a->val, tau, kept);
  if (temp_malloc(&o.ptr, sizeof(int32_t) * (a->m + 1)) != hipSuccess) {
    dev_free(kept);
    return AMG_ENOMEM;
  }
  int rc = AMG_OK;
  o.nnz = scan_ptr(s, a->m, kept, o.ptr, &rc);
  dev_free(kept);
  if (rc != AMG_OK) {
    free_csr(o);
    return rc;
  }
  if (temp_malloc(&o.col, sizeof(int32_t) * std::max<int64_t>(o.nnz, 1)) != hipSuccess ||
      temp_malloc(&o.val, sizeof(double) * std::max<int64_t>(o.nnz, 1)) != hipSuccess) {
    free_csr(o);
    return AMG_ENOMEM;
  }
  hipLaunchKernelGGL(k_keep_copy, dim3(grid_for(a->m)), dim3(kBlock), 0, s, a->m, a->ptr, a->col, a->val, tau,
                     o.ptr, o.col, o.val);
  if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess) {
    free_csr(o);
    return AMG_EHIP;
  }
  free_csr(*a);
  *a = o;
  return AMG_OK;
}

int transpose(hipStream_t s, const Csr& a, Csr* t) {
  Csr o;
  o.m = a.ncols;
  o.ncols = a.m;
  o.nnz = a.nnz;
  int32_t* cnt = nullptr;
  if (temp_malloc(&cnt, sizeof(int32_t) * (o.m + 1)) != hipSuccess) return AMG_ENOMEM;
  int rc = AMG_OK;
  if (hipMemsetAsync(cnt, 0, sizeof(int32_t) * (o.m + 1), s) != hipSuccess) rc = AMG_EHIP;
  if (rc == AMG_OK) {
    hipLaunchKernelGGL(k_col_count, dim3(grid_for(a.nnz)), dim3(kBlock), 0, s, a.nnz, a.col, cnt);
    if (temp_malloc(&o.ptr, sizeof(int32_t) * (o.m + 1)) != hipSuccess) rc = AMG_ENOMEM;
  }
  if (rc == AMG_OK) scan_ptr(s, o.m, cnt, o.ptr, &rc);
  if (rc == AMG_OK && (temp_malloc(&o.col, sizeof(int32_t) * std::max<int64_t>(o.nnz, 1)) != hipSuccess ||
                       temp_malloc(&o.val, sizeof(double) * std::max<int64_t>(o.nnz, 1)) != hipSuccess))
    rc = AMG_ENOMEM;
  if (rc == AMG_OK && hipMemsetAsync(cnt, 0, sizeof(int32_t) * (o.m + 1), s) != hipSuccess) rc = AMG_EHIP;
  if (rc == AMG_OK) {
    hipLaunchKernelGGL(k_transpose_scatter, dim3(grid_for(a.m)), dim3(kBlock), 0, s, a.m, a.ptr, a.col, a.val,
                       o.ptr, cnt, o.col, o.val);
    hipLaunchKernelGGL(k_row_sort, dim3(grid_for(o.m)), dim3(kBlock), 0, s, o.m, o.ptr, o.col, o.val);
    if (hipGetLastError() != hipSuccess) rc = AMG_EHIP;
  }
  if (rc == AMG_OK) {
    // the rows longer than kShortRow (the fill counters are done with: the list takes their place)
    int32_t nlong = 0;
    if (hipMemsetAsync(cnt + o.m, 0, sizeof(int32_t), s) != hipSuccess) rc = AMG_EHIP;
    hipLaunchKernelGGL(k_long_rows, dim3(grid_for(o.m)), dim3(kBlock), 0, s, o.m, o.ptr, cnt, cnt + o.m);
    if (hipMemcpyAsync(&nlong, cnt + o.m, sizeof(nlong), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
      rc = AMG_EHIP;
    if (rc == AMG_OK && nlong > 0) {
      hipLaunchKernelGGL(k_row_sort_long, dim3((unsigned)nlong), dim3(kWave), 0, s, (const int32_t*)cnt, o.ptr, o.col,
                         o.val);
      if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess) rc = AMG_EHIP;
    }
  }
  dev_free(cnt);
  if (rc != AMG_OK) {
    free_csr(o);
    return rc;
  }
  *t = o;
  return AMG_OK;
}

int children_transpose(hipStream_t s, int64_t n, int64_t nc, const int32_t* children, Csr* PT) {
  Csr o;
  o.m = nc;
  o.ncols = n;
  o.nnz = n;
  if (temp_malloc(&o.ptr, sizeof(int32_t) * (nc + 1)) != hipSuccess ||
      temp_malloc(&o.col, sizeof(int32_t) * n) != hipSuccess || temp_malloc(&o.val, sizeof(double) * n) != hipSuccess) {
    free_csr(o);
    return AMG_ENOMEM;
  }
  hipLaunchKernelGGL(k_children_count, dim3(grid_for(nc)), dim3(kBlock), 0, s, nc, children, o.ptr);
  int rc = AMG_OK;
  scan_ptr(s, nc, o.ptr, o.ptr, &rc);
  if (rc == AMG_OK) {
    hipLaunchKernelGGL(k_children_rows, dim3(grid_for(nc * kMaxChildren)), dim3(kBlock), 0, s, nc, children, o.ptr,
                       o.col, o.val);
    if (hipGetLastError() != hipSuccess) rc = AMG_EHIP;
  }
  if (rc != AMG_OK) {
    free_csr(o);
    return rc;
  }
  *PT = o;
  return AMG_OK;
}

int galerkin_from_restriction(hipStream_t s, const Csr& A, const Csr& R, const int32_t* agg, const int32_t* children,
                              Csr* Ac) {
  const int64_t nc = R.m;
  Csr o;
  o.m = nc;
  o.ncols = nc;
  graph::DevBuf<int32_t> cnt;
  AMGP_TRY(cnt.alloc(nc + 1));
  int rc = AMG_OK;
  hipLaunchKernelGGL(k_row_lengths, dim3(grid_for(nc)), dim3(kBlock), 0, s, nc, R.ptr, cnt.p);
  const int64_t longest = max_count(s, nc, cnt.p, cnt.p + nc, &rc);
  if (rc != AMG_OK) return rc;
  if (longest > kWave) return AMG_EINVAL;
  const dim3 grid((unsigned)nc), block(kWave);
  if (temp_malloc(&o.ptr, sizeof(int32_t) * (nc + 1)) != hipSuccess) return AMG_ENOMEM;
  hipLaunchKernelGGL(k_galerkin_rows<false>, grid, block, 0, s, A.ptr, A.col, A.val, children, R.ptr, R.col, agg, o.ptr,
                     nullptr, nullptr);
  o.nnz = scan_ptr(s, nc, o.ptr, o.ptr, &rc);
  if (rc == AMG_OK && (temp_malloc(&o.col, sizeof(int32_t) * std::max<int64_t>(o.nnz, 1)) != hipSuccess ||
                       temp_malloc(&o.val, sizeof(double) * std::max<int64_t>(o.nnz, 1)) != hipSuccess))
    rc = AMG_ENOMEM;
  if (rc == AMG_OK) {
    hipLaunchKernelGGL(k_galerkin_rows<true>, grid, block, 0, s, A.ptr, A.col, A.val, children, R.ptr, R.col, agg,
                       o.ptr, o.col, o.val);
    if (hipGetLastError() != hipSuccess) rc = AMG_EHIP;
  }
  if (rc != AMG_OK) {
    hipStreamSynchronize(s);
    free_csr(o);
    return rc;
  }
  *Ac = o;
  return AMG_OK;
}

int tentative_prolongator(hipStream_t s, int64_t n, int64_t nc, const int32_t* agg, Csr* P) {
  Csr o;
  o.m = n;
  o.ncols = nc;
  o.nnz = n;
  if (temp_malloc(&o.ptr, sizeof(int32_t) * (n + 1)) != hipSuccess ||
      temp_malloc(&o.col, sizeof(int32_t) * n) != hipSuccess || temp_malloc(&o.val, sizeof(double) * n) != hipSuccess) {
    free_csr(o);
    return AMG_ENOMEM;
  }
  hipLaunchKernelGGL(k_identity_rows, dim3(grid_for(n + 1)), dim3(kBlock), 0, s, n, agg, o.ptr, o.col, o.val);
  if (hipGetLastError() != hipSuccess) {
    free_csr(o);
    return AMG_EHIP;
  }
  *P = o;
  return AMG_OK;
}

int smoothed_prolongator(hipStream_t s, const Csr& A, int nbatch, const Csr& Ph, Csr* P, int* flag) {
  const int64_t n = A.m, rpp = n / nbatch;
  Csr AP;
  int rc = spgemm(s, A, Ph, &AP, flag);
  if (rc != AMG_OK) return rc;
  double* diag = nullptr;
  unsigned long long* lam = nullptr;
  double* om = nullptr;
  if (temp_malloc(&diag, sizeof(double) * n) != hipSuccess || temp_malloc(&lam, sizeof(unsigned long long) * nbatch) !=
      hipSuccess || temp_malloc(&om, sizeof(double) * nbatch) != hipSuccess)
    rc = AMG_ENOMEM;
  std::vector<double> hl(nbatch), ho(nbatch);
  if (rc == AMG_OK && hipMemsetAsync(lam, 0, sizeof(unsigned long long) * nbatch, s) != hipSuccess) rc = AMG_EHIP;
  if (rc == AMG_OK) {
    hipLaunchKernelGGL(k_diag_ratio, dim3(grid_for(n)), dim3(kBlock), 0, s, n, rpp, A.ptr, A.col, A.val, diag, lam,
                       flag);
    if (hipMemcpyAsync(hl.data(), lam, sizeof(double) * nbatch, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
      rc = AMG_EHIP;
  }
  if (rc == AMG_OK) {
    // omega = 4 / (3 lambda), lambda = ||D^{-1} A||_inf per stacked problem
    for (int p = 0; p < nbatch; ++p) ho[p] = 4.0 / (3.0 * hl[p]);
    if (hipMemcpyAsync(om, ho.data(), sizeof(double) * nbatch, hipMemcpyHostToDevice, s) != hipSuccess) rc = AMG_EHIP;
  }
  if (rc == AMG_OK) {
    hipLaunchKernelGGL(k_smooth_prol, dim3(grid_for(n)), dim3(kBlock), 0, s, n, rpp, AP.ptr, AP.col, AP.val, Ph.col,
                       Ph.val, diag, om);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess) rc = AMG_EHIP;
  }
  dev_free(diag);
  dev_free(lam);
  dev_free(om);
  if (rc == AMG_OK) rc = drop_small(s, &AP, kDropTau);
  if (rc != AMG_OK) {
    free_csr(AP);
    return rc;
  }
  *P = AP;
  return AMG_OK;
}

int galerkin_general(hipStream_t s, const Csr& A, const Csr& P, const Csr& PT, Csr* Ac, int* flag) {
  Csr AP;
  AMGP_TRY(spgemm(s, A, P, &AP, flag));
  const int rc = spgemm(s, PT, AP, Ac, flag);
  free_csr(AP);
  if (rc != AMG_OK) return rc;
  return drop_small(s, Ac, kDropTau);
}

}  // namespace amgp
