// Setup kernels: l1-Jacobi diagonal, CSR -> sliced ELL, box aggregation and the
// Galerkin product A_c = P^T A P for a piecewise-constant P.
#include <algorithm>
#include <vector>

#include <climits>

#include "graph.h"
#include "internal.h"

namespace amgp {

namespace {

// CSR validation, in two passes so that nothing is read through an
// unchecked index: first row_ptr alone, then the column indices.
__global__ void k_check_ptr(int64_t n, int64_t nnz, const int32_t* __restrict__ ptr, int* __restrict__ flag) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i > n) return;
  const int32_t v = ptr[i];
  if (i == 0 && v != 0) flag[F_BADCSR] = 1;
  if (i == n && v != nnz) flag[F_BADCSR] = 1;
  if (i < n && (ptr[i + 1] < v || v < 0 || v > nnz)) flag[F_BADCSR] = 1;
}

__global__ void k_check_col(int64_t n, const int32_t* __restrict__ ptr, const int32_t* __restrict__ col,
                            int* __restrict__ flag) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int32_t prev = -1;
  for (int p = ptr[i]; p < ptr[i + 1]; ++p) {
    const int32_t c = col[p];
    if (c <= prev || c >= n) flag[F_BADCSR] = 1;
    prev = c;
  }
}

// M_i = a_ii + sum_{j != i} |a_ij| (eq. l1smooth); minv = 1/M.  Flags a
// non-positive or non-finite diagonal or l1 sum as "not SPD".  The block's rows, contiguous in
// CSR, pass through LDS in chunks that the threads load together, each then adding its own
// row's entries in order (a thread walking its row in memory read every line many times: 25 ms
// against 2.4 ms on the 27-point 320^3 matrix).
constexpr int kRowChunk = 2048;

__global__ __launch_bounds__(kBlock) void k_l1_diag(int64_t n, const int32_t* __restrict__ ptr,
                                                    const int32_t* __restrict__ col, const double* __restrict__ val,
                                                    double* __restrict__ minv, int* __restrict__ flag) {
  __shared__ int32_t scol[kRowChunk];
  __shared__ double sval[kRowChunk];
  const int64_t i0 = (int64_t)blockIdx.x * kBlock, i = i0 + threadIdx.x;
  const int64_t i1 = i0 + kBlock < n ? i0 + kBlock : n;
  const int beg = ptr[i0], end = ptr[i1];
  const int p = i < n ? ptr[i] : end, pe = i < n ? ptr[i + 1] : end;
  double d = 0.0, off = 0.0;
  bool has_diag = false;
  for (int b = beg; b < end; b += kRowChunk) {
    const int m = min(kRowChunk, end - b);
    __syncthreads();
    for (int e = threadIdx.x; e < m; e += kBlock) {
      scol[e] = col[b + e];
      sval[e] = val[b + e];
    }
    __syncthreads();
    for (int q = max(p, b); q < min(pe, b + m); ++q) {
      const double v = sval[q - b];
      if (scol[q - b] == i) {
        d += v;
        has_diag = true;
      } else {
        off += fabs(v);
      }
    }
  }
  if (i >= n) return;
  const double m = d + off;
  if (!has_diag || !(d > 0.0) || !(m > 0.0) || m > 1.0e308) flag[F_NOTSPD] = 1;
  minv[i] = 1.0 / m;
}

// width of every slice of R rows = longest row in it
__global__ void k_slice_width(int64_t n, int64_t nslices, int R, const int32_t* __restrict__ ptr,
                              int32_t* __restrict__ w) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= nslices) return;
  int m = 0;
  for (int l = 0; l < R; ++l) {
    const int64_t i = s * R + l;
    if (i >= n) break;
    m = max(m, ptr[i + 1] - ptr[i]);
  }
  w[s] = m;
}

// one thread per (slice, lane): lane l of slice s serves row s R + l / G, entries j = l % G + G t
__global__ void k_ell_fill(int64_t n, int64_t ncols, int64_t nslices, int G, const int32_t* __restrict__ ptr,
                           const int32_t* __restrict__ col, const double* __restrict__ val,
                           const int32_t* __restrict__ sptr, int32_t* __restrict__ ecol, double* __restrict__ eval) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= nslices * kSlice) return;
  const int64_t s = t / kSlice;
  const int lane = (int)(t % kSlice);
  const int64_t i = s * (kSlice / G) + lane / G;
  const int g = lane % G;
  const int base = sptr[s];
  const int steps = (sptr[s + 1] - base) / kSlice;
  int len = 0, p0 = 0;
  if (i < n) {
    p0 = ptr[i];
    len = ptr[i + 1] - p0;
  }
  const int32_t padcol = (i < n && i < ncols) ? (int32_t)i : 0;
  for (int st = 0; st < steps; ++st) {
    const int j = st * G + g;
    const int64_t q = base + (int64_t)st * kSlice + lane;
    if (j < len) {
      ecol[q] = col[p0 + j];
      eval[q] = val[p0 + j];
    } else {
      ecol[q] = padcol;
      eval[q] = 0.0;
    }
  }
}

// Layout of every slice of 64 RPL rows (RPL rows per lane of the kernels), one wavefront per slice,
// its lanes on consecutive entries of the slice's rows (contiguous in CSR, so the loads coalesce; one
// row per lane instead read 20 KB a wavefront through its own cache lines, 33 ms against 5 ms for the
// kinds of the 27-point 320^3 matrix).  The slice's distinct column offsets (col - row, or col -
// anchor[row * astride]) go into an LDS hash set.
//
// TABLES = false: the offsets, sorted, offs[s * 64 + t], their count width[s] (-1 when there are more
// than 64), the longest row lwidth[s], and with kind given the kind of the slice (see Ell): per step
// the lanes must agree on one value up to +0; FULL when every lane holds an entry at every step
// and all of one value (zero included); a differing value ends the search (the first entries of
// a matrix of varying coefficients).
// TABLES = true (uniform slices alone): per step the value and the lane mask (all ones for a full
// step; with two rows per lane of the even rows, then of the odd ones), stride records per slice in
// vtab / mtab, and the hash of offsets, values and masks.
constexpr int kOffHash = 256;
constexpr int kOffEmpty = INT_MIN;

__device__ __forceinline__ unsigned off_slot(int o) { return ((unsigned)o * 2654435761u) & (kOffHash - 1); }

template <bool TABLES, int RPL>
__global__ __launch_bounds__(kWave) void k_slice_layout(
    int64_t n, const int32_t* __restrict__ ptr, const int32_t* __restrict__ col, const double* __restrict__ val,
    const int32_t* anchor, int astride, int32_t* __restrict__ offs, int32_t* __restrict__ width,
    int32_t* __restrict__ lwidth, int32_t* __restrict__ kind, int stride, unsigned long long* __restrict__ vtab,
    unsigned long long* __restrict__ mtab, unsigned long long* __restrict__ hash) {
  __shared__ int set[kOffHash];
  __shared__ int at[kOffHash];  // step of a set entry
  __shared__ int list[kWave];
  constexpr int kRows = kSlice * RPL;
  __shared__ int rp[kRows + 1];
  __shared__ int base[kRows];
  __shared__ unsigned long long sval[kWave], spres[RPL][kWave], snz[RPL][kWave];
  __shared__ int cnt, differ;
  const int64_t s = blockIdx.x;
  const int lane = threadIdx.x;
  if (TABLES && kind[s] == SLICE_DENSE) return;
  for (int k = lane; k < kRows; k += kWave) {
    const int64_t r = s * kRows + k;
    rp[k] = ptr[r < n ? r : n];
    if (k == kRows - 1) rp[kRows] = ptr[r + 1 < n ? r + 1 : n];
    base[k] = r < n ? (anchor ? anchor[r * astride] : (int)r) : 0;
  }
  for (int t = lane; t < kOffHash; t += kWave) set[t] = kOffEmpty;
  if (lane == 0) {
    cnt = 0;
    differ = 0;
  }
  sval[lane] = 0;
  for (int k = 0; k < RPL; ++k) spres[k][lane] = snz[k][lane] = 0;
  __syncthreads();
  const int beg = rp[0], end = rp[kRows];
  auto row_of = [&](int e) {  // the row (of the slice) of entry e
    int lo = 0;
#pragma unroll
    for (int step = kRows / 2; step > 0; step >>= 1)
      if (rp[lo + step] <= e) lo += step;
    return lo;
  };
  auto insert = [&](int o) {
    unsigned h = off_slot(o);
    for (int probe = 0; probe < kOffHash; ++probe) {
      int old = set[h];
      if (old == o) return;
      if (old == kOffEmpty) {
        old = atomicCAS(&set[h], kOffEmpty, o);
        if (old == kOffEmpty) {
          atomicAdd(&cnt, 1);
          return;
        }
        if (old == o) return;
      }
      h = (h + 1) & (kOffHash - 1);
    }
  };
  int c;
  if constexpr (TABLES) {
    c = width[s];
    if (lane < c) {
      list[lane] = offs[s * kSlice + lane];
      insert(list[lane]);
    }
    __syncthreads();
  } else {
    int longest = 0;
    for (int k = lane; k < kRows; k += kWave) longest = max(longest, rp[k + 1] - rp[k]);
    for (int off = 32; off > 0; off >>= 1) longest = max(longest, __shfl_xor(longest, off, kWave));
    if (lane == 0) lwidth[s] = longest;
    for (int e = beg + lane; e < end; e += kWave) {
      if (cnt > kWave) break;  // too many already
      insert(col[e] - base[row_of(e)]);
    }
    __syncthreads();
    c = cnt;
    if (c > kSlice) {
      if (lane == 0) width[s] = -1;
      return;
    }
    // compact (slot order), then an odd-even transposition sort of at most 64 values by the wavefront
    __shared__ int k;
    if (lane == 0) k = 0;
    __syncthreads();
    for (int t = lane; t < kOffHash; t += kWave) {
      const int v = set[t];
      if (v != kOffEmpty) list[atomicAdd(&k, 1)] = v;
    }
    __syncthreads();
    for (int phase = 0; phase < c; ++phase) {
      const int i = 2 * lane + (phase & 1);
      if (i + 1 < c && list[i] > list[i + 1]) {
        const int a = list[i];
        list[i] = list[i + 1];
        list[i + 1] = a;
      }
      __syncthreads();
    }
    if (lane < c) offs[s * kSlice + lane] = list[lane];
    if (lane == 0) width[s] = c;
    if (!kind) return;
  }
  if (lane < c) {  // the step of every offset in the set
    unsigned h = off_slot(list[lane]);
    while (set[h] != list[lane]) h = (h + 1) & (kOffHash - 1);
    at[h] = lane;
  }
  __syncthreads();
  for (int e = beg + lane; e < end; e += kWave) {
    if (!TABLES && differ) break;
    const int row = row_of(e);
    const int o = col[e] - base[row];
    unsigned h = off_slot(o);
    while (set[h] != o) h = (h + 1) & (kOffHash - 1);
    const int t = at[h];
    const unsigned long long bits = (unsigned long long)__double_as_longlong(val[e]);
    const unsigned long long bit = 1ull << (row / RPL);
    atomicOr(&spres[row % RPL][t], bit);
    if (bits) {
      atomicOr(&snz[row % RPL][t], bit);
      unsigned long long old = sval[t];
      if (old == 0) old = atomicCAS(&sval[t], 0ull, bits);
      if (old != 0 && old != bits) differ = 1;
    }
  }
  __syncthreads();
  if (!TABLES && differ) {
    if (lane == 0) kind[s] = SLICE_DENSE;
    return;
  }
  bool whole = true;
  for (int k = 0; k < RPL; ++k)
    whole = whole && spres[k][lane] == ~0ull && snz[k][lane] == snz[0][lane] &&
            (snz[k][lane] == 0 || snz[k][lane] == ~0ull);
  // the halves of 128 rows that use a step's offset
  int bits = 3;
  if constexpr (RPL == 2) {
    const unsigned long long pres = spres[0][lane] | spres[1][lane];
    bits = ((pres & 0xffffffffull) != 0) | ((pres >> 32) != 0) << 1;
  }
  const bool halves = __ballot(lane < c && bits != 3) != 0;
  if constexpr (TABLES) {
    unsigned long long h = 0;
    if (lane < c) {
      if (halves) offs[s * kSlice + lane] = 4 * list[lane] + bits;
      const unsigned long long v = sval[lane];
      vtab[s * stride + lane] = v;
      h = graph::splitmix64(graph::splitmix64(((unsigned long long)lane << 32) + (unsigned)list[lane] * 4 + bits) ^ v);
      for (int k = 0; k < RPL; ++k) {
        const unsigned long long m = whole ? ~0ull : snz[k][lane];
        mtab[(s * RPL + k) * stride + lane] = m;
        h = graph::splitmix64(h ^ m);
      }
    }
    for (int off = 32; off > 0; off >>= 1) h += __shfl_xor(h, off, kWave);
    if (lane == 0) hash[s] = graph::splitmix64(h) | 1;  // 0 marks a free slot
  } else {
    const bool full = __ballot(lane < c && !whole) == 0;
    // triples: a whole slice of consecutive rows whose sorted offsets come in threes
    const bool third = lane < c && (lane % 3 == 0 || list[lane] == list[lane - 1] + 1);
    const bool triples = !anchor && (s + 1) * kRows <= n && c % 3 == 0 && __ballot(lane < c && !third) == 0;
    if (lane == 0)
      kind[s] = halves ? SLICE_HALVES : (full ? SLICE_FULL : SLICE_MASKED) | (triples ? SLICE_TRIPLES : 0);
  }
}

// Equal patterns share one copy: a table of cap (a power of two, at least twice the slices) slots
// keyed by the hash keeps the smallest slice of each key, and a slice whose records equal those of
// that slice takes them over (rep[s]); one that merely has its hash keeps its own.
__global__ void k_pattern_insert(int64_t nslices, const int32_t* __restrict__ kind,
                                 const unsigned long long* __restrict__ hash, unsigned cap,
                                 unsigned long long* __restrict__ keys, int32_t* __restrict__ first) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= nslices || kind[s] == SLICE_DENSE) return;
  unsigned q = (unsigned)hash[s] & (cap - 1);
  // most slices share few patterns: the atomics only where a plain read has not shown the key, or a
  // smaller slice, to be there (on one address they are served one by one)
  for (;;) {
    unsigned long long old = __hip_atomic_load(&keys[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (old == 0) old = atomicCAS(&keys[q], 0ull, hash[s]);
    if (old == 0 || old == hash[s]) break;
    q = (q + 1) & (cap - 1);
  }
  if (__hip_atomic_load(&first[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > (int32_t)s)
    atomicMin(&first[q], (int32_t)s);
}

__global__ void k_pattern_resolve(int64_t nslices, const int32_t* __restrict__ kind,
                                  const unsigned long long* __restrict__ hash, unsigned cap,
                                  const unsigned long long* __restrict__ keys, const int32_t* __restrict__ first,
                                  const int32_t* __restrict__ offs, const int32_t* __restrict__ width, int rpl,
                                  int stride,
                                  const unsigned long long* __restrict__ vtab,
                                  const unsigned long long* __restrict__ mtab, int32_t* __restrict__ rep) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= nslices) return;
  if (kind[s] == SLICE_DENSE) {
    rep[s] = -1;
    return;
  }
  unsigned q = (unsigned)hash[s] & (cap - 1);
  while (keys[q] != hash[s]) q = (q + 1) & (cap - 1);
  const int64_t f = first[q];
  bool same = kind[f] == kind[s] && width[f] == width[s];
  for (int t = 0; same && t < width[s]; ++t)
    same = offs[f * kSlice + t] == offs[s * kSlice + t] && vtab[f * stride + t] == vtab[s * stride + t] &&
           mtab[f * rpl * stride + t] == mtab[s * rpl * stride + t] &&
           mtab[(f * rpl + rpl - 1) * stride + t] == mtab[(s * rpl + rpl - 1) * stride + t];
  rep[s] = same ? (int32_t)f : (int32_t)s;
}

// The kept patterns' steps: one wavefront per slice, lane t writes step t.
__global__ void k_pattern_write(int64_t nslices, const int32_t* __restrict__ rep, const int2* __restrict__ desc,
                                const int32_t* __restrict__ offs, int rpl, int stride,
                                const unsigned long long* __restrict__ vtab,
                                const unsigned long long* __restrict__ mtab, int npat,
                                unsigned long long* __restrict__ pat) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t s = g / kSlice;
  if (s >= nslices || rep[s] != s) return;
  const int2 d = desc[s];
  const int t = (int)(g % kSlice);
  if (t >= (d.y >> 4)) return;
  const int64_t q = d.x + t;
  for (int k = 0; k < rpl; ++k) pat[(int64_t)k * npat + q] = mtab[(s * rpl + k) * stride + t];
  pat[(int64_t)rpl * npat + q] = vtab[s * stride + t];
  reinterpret_cast<int32_t*>(pat + (rpl + 1) * (int64_t)npat)[q] = offs[s * kSlice + t];
}

// Sums over the slices: steps of the aligned and of the packed layout, slices that fit no pattern
// table (width -1), uniform slices, those of them in triples, and the widest slice.
enum SliceStat { ST_ALIGNED = 0, ST_PACKED, ST_OVER, ST_UNIFORM, ST_TRIPLES, ST_WIDEST, ST_COUNT };
__global__ __launch_bounds__(kBlock) void k_slice_stats(int64_t nslices, const int32_t* __restrict__ width,
                                                        const int32_t* __restrict__ lwidth,
                                                        const int32_t* __restrict__ kind,
                                                        unsigned long long* __restrict__ stat) {
  unsigned long long v[ST_COUNT] = {};
  for (int64_t s = (int64_t)blockIdx.x * kBlock + threadIdx.x; s < nslices; s += (int64_t)gridDim.x * kBlock) {
    const int w = width[s];
    if (w < 0) {
      v[ST_OVER] += 1;
      continue;
    }
    v[ST_ALIGNED] += w;
    v[ST_PACKED] += lwidth[s];
    v[ST_UNIFORM] += kind && kind[s] != SLICE_DENSE;
    v[ST_TRIPLES] += kind && (kind[s] & SLICE_TRIPLES);
    v[ST_WIDEST] = max(v[ST_WIDEST], (unsigned long long)w);
  }
  for (int k = 0; k < ST_COUNT; ++k) {
    unsigned long long x = v[k];
    for (int off = 32; off > 0; off >>= 1) {
      const unsigned long long y = __shfl_xor(x, off, kWave);
      x = k == ST_WIDEST ? max(x, y) : x + y;
    }
    if ((threadIdx.x & (kWave - 1)) == 0 && x) {
      if (k == ST_WIDEST)
        atomicMax(&stat[k], x);
      else
        atomicAdd(&stat[k], x);
    }
  }
}

// what a slice stores: its steps as a dense slice (dcnt) or as the representative of a pattern (pcnt)
__global__ void k_slice_store(int64_t nslices, const int32_t* __restrict__ width, const int32_t* __restrict__ kind,
                              const int32_t* __restrict__ rep, int32_t* __restrict__ dcnt,
                              int32_t* __restrict__ pcnt) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= nslices) return;
  const bool dense = kind[s] == SLICE_DENSE;
  dcnt[s] = dense ? width[s] : 0;
  pcnt[s] = !dense && rep[s] == s ? width[s] : 0;
}

__global__ void k_slice_desc(int64_t nslices, const int32_t* __restrict__ width, const int32_t* __restrict__ kind,
                             const int32_t* __restrict__ rep, const int32_t* __restrict__ dbeg,
                             const int32_t* __restrict__ pbeg, int2* __restrict__ desc) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= nslices) return;
  desc[s] = int2{kind[s] == SLICE_DENSE ? dbeg[s] : pbeg[rep[s]], width[s] * 16 + kind[s]};
}

// Offset-aligned fill: lane l of slice s (row r, anchor a = r or anchor[r * astride]) puts, at
// step t, its entry of column a + offs[t] (0 when the row has none), with the steps of a lane in
// pairs: step t at 64 (t - t % 2) + 2 l + t % 2 while t has a partner, an odd last step at 64 t + l.
// With desc only the dense slices are stored.
__global__ void k_ell_fill_aligned(int64_t n, int64_t nslices, const int32_t* __restrict__ ptr,
                                   const int32_t* __restrict__ col, const double* __restrict__ val,
                                   const int32_t* anchor, int astride, const int32_t* __restrict__ offs,
                                   const int32_t* __restrict__ sptr, const int2* __restrict__ desc,
                                   double* __restrict__ eval, int32_t* __restrict__ doff) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= nslices * kSlice) return;
  const int64_t s = t / kSlice;
  const int lane = (int)(t % kSlice);
  const int64_t r = s * kSlice + lane;
  int base, steps;
  if (desc) {
    const int2 d = desc[s];
    if ((d.y & 15) != SLICE_DENSE) return;
    base = d.x * kSlice;
    steps = d.y >> 4;
  } else {
    base = sptr[s];
    steps = (sptr[s + 1] - base) / kSlice;
  }
  int p = 0, pe = 0;
  int64_t a = r;
  if (r < n) {
    p = ptr[r];
    pe = ptr[r + 1];
    if (anchor) a = anchor[r * astride];
  }
  const int paired = steps & ~1;
  for (int st = 0; st < steps; ++st) {
    const int o = offs[s * kSlice + st];
    const int64_t c = a + o;
    double v = 0.0;
    while (p < pe && col[p] < c) ++p;
    if (p < pe && col[p] == c) v = val[p++];
    const int dst = st < paired ? kSlice * (st & ~1) + 2 * lane + (st & 1) : kSlice * st + lane;
    eval[base + dst] = v;
    if (lane == 0) doff[(base >> 6) + st] = o;
  }
}

// Distinct offsets of all slices into table[kOffHash] (empty slots kOffEmpty), their number in *count.
__global__ void k_union_offsets(int64_t nslices, const int32_t* __restrict__ offs, const int32_t* __restrict__ width,
                                int32_t* __restrict__ table, int32_t* __restrict__ count) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t s = g / kSlice;
  const int t = (int)(g % kSlice);
  if (s >= nslices || t >= width[s]) return;
  const int o = offs[s * kSlice + t];
  unsigned h = off_slot(o);
  for (int probe = 0; probe < kOffHash; ++probe) {
    int old = __hip_atomic_load(&table[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (old == o) return;
    if (old == kOffEmpty) {
      if (__hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > kMirrorMaxSteps) return;
      old = atomicCAS(&table[h], kOffEmpty, o);
      if (old == kOffEmpty) {
        atomicAdd(count, 1);
        return;
      }
      if (old == o) return;
    }
    h = (h + 1) & (kOffHash - 1);
  }
}

// bit t of present[s]: slice s has entries of offset sorted[t]
__global__ void k_mirror_present(int64_t nslices, const int32_t* __restrict__ offs, const int32_t* __restrict__ width,
                                 int w, const MirrorStep* __restrict__ steps, int32_t* __restrict__ present) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= nslices) return;
  unsigned m = 0;
  for (int k = 0, t = 0; k < width[s]; ++k) {  // both lists ascend
    while (t < w && steps[t].off != offs[s * kSlice + k]) ++t;
    if (t < w) m |= 1u << t;
  }
  present[s] = (int32_t)m;
}

__global__ void k_fill_int(int n, int32_t v, int32_t* __restrict__ x) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) x[i] = v;
}

// Mirrored diagonals: CHECK = false stores every entry of offset >= 0 (row i of array k at
// val[k stride + pad + i], zeroed beforehand); CHECK = true compares every entry of negative offset
// with the one it mirrors (differ[0] set on other bits) and counts the entries that are not +0 on
// each side (differ[1], differ[2]), which agree when no entry lacks its mirror image.
// Rows pass through LDS as in k_l1_diag.
template <bool CHECK>
__global__ __launch_bounds__(kBlock) void k_mirror(int64_t n, const int32_t* __restrict__ ptr,
                                                   const int32_t* __restrict__ col, const double* __restrict__ cval,
                                                   int nup, const int32_t* __restrict__ up, int64_t stride,
                                                   int64_t pad, double* __restrict__ val,
                                                   unsigned long long* __restrict__ differ) {
  __shared__ int32_t scol[kRowChunk];
  __shared__ double sval[kRowChunk];
  __shared__ int32_t sup[kMirrorMaxSteps];
  const int64_t i0 = (int64_t)blockIdx.x * kBlock, i = i0 + threadIdx.x;
  const int64_t i1 = i0 + kBlock < n ? i0 + kBlock : n;
  const int beg = ptr[i0], end = ptr[i1];
  const int p = i < n ? ptr[i] : end, pe = i < n ? ptr[i + 1] : end;
  if ((int)threadIdx.x < nup) sup[threadIdx.x] = up[threadIdx.x];
  unsigned long long bad = 0, above = 0, below = 0;
  for (int b = beg; b < end; b += kRowChunk) {
    const int m = min(kRowChunk, end - b);
    __syncthreads();
    for (int e = threadIdx.x; e < m; e += kBlock) {
      scol[e] = col[b + e];
      sval[e] = cval[b + e];
    }
    __syncthreads();
    for (int q = max(p, b); q < min(pe, b + m); ++q) {
      const int c = scol[q - b], o = c - (int)i;
      const unsigned long long bits = (unsigned long long)__double_as_longlong(sval[q - b]);
      int k = 0;
      while (k < nup && sup[k] != abs(o)) ++k;
      if (k == nup) continue;  // cannot be: up lists every offset of the matrix
      if (!CHECK && o >= 0) val[k * stride + pad + i] = sval[q - b];
      if (CHECK && o > 0) above += bits != 0;
      if (CHECK && o < 0) {
        below += bits != 0;
        bad |= bits != (unsigned long long)__double_as_longlong(val[k * stride + pad + c]);
      }
    }
  }
  if constexpr (CHECK) {
    for (int off = 32; off > 0; off >>= 1) {
      bad |= __shfl_xor(bad, off, kWave);
      above += __shfl_xor(above, off, kWave);
      below += __shfl_xor(below, off, kWave);
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
      if (bad) differ[0] = 1;
      atomicAdd(&differ[1], above);
      atomicAdd(&differ[2], below);
    }
  }
}

// Dense slices of 128 rows (two rows per lane): step t of row k of the slice at 128 (beg + t) + k, its
// offset with the bits of the halves that use it (doff zero before).  A wavefront serves one half.
__global__ void k_ell_fill_pairs(int64_t n, const int32_t* __restrict__ ptr, const int32_t* __restrict__ col,
                                 const double* __restrict__ val, const int32_t* __restrict__ offs,
                                 const int2* __restrict__ desc, double* __restrict__ eval,
                                 int32_t* __restrict__ doff) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t s = r / (2 * kSlice);
  const int k = (int)(r % (2 * kSlice));
  if (s * 2 * kSlice >= n) return;
  const int2 d = desc[s];
  if ((d.y & 15) != SLICE_DENSE) return;
  int p = r < n ? ptr[r] : 0;
  const int pe = r < n ? ptr[r + 1] : 0;
  for (int st = 0; st < (d.y >> 4); ++st) {
    const int o = offs[s * kSlice + st];
    double v = 0.0;
    while (p < pe && col[p] < r + o) ++p;
    const bool has = p < pe && col[p] == r + o;
    if (has) v = val[p++];
    eval[(int64_t)(d.x + st) * 2 * kSlice + k] = v;
    const int half = k / kSlice, used = __ballot(has) != 0 ? 1 << half : 0;
    if (k % kSlice == 0) atomicAdd(&doff[d.x + st], half == 0 ? 4 * o + used : used);
  }
}

__global__ void k_round_f32(int64_t m, const double* __restrict__ a, float* __restrict__ b) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < m) b[i] = (float)a[i];
}

// FP32 copy of offset-aligned slices: slices of at least kQuadMinSteps steps put each lane's steps in
// quads (step t of lane l at 64 (t - t % 4) + 4 l + t % 4 for t below w - w % 4, then a pair at
// 64 (t - t % 2) + 2 l + t % 2, then a single step at 64 t + l), narrower ones keep the FP64 pairs.
__global__ void k_round_f32_aligned(int64_t nslices, const int32_t* __restrict__ sptr,
                                    const int2* __restrict__ desc, const double* __restrict__ a,
                                    float* __restrict__ b) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t s = g >> 6;
  const int lane = (int)(g & 63);
  if (s >= nslices) return;
  int beg, w;
  if (desc) {
    const int2 d = desc[s];
    if ((d.y & 15) != SLICE_DENSE) return;
    beg = d.x * kSlice;
    w = d.y >> 4;
  } else {
    beg = sptr[s];
    w = (sptr[s + 1] - beg) >> 6;
  }
  const int w2 = w & ~1, w4 = w >= kQuadMinSteps ? (w & ~3) : 0;
  for (int t = 0; t < w; ++t) {
    const int pair = t < w2 ? 64 * (t & ~1) + 2 * lane + (t & 1) : 64 * t + lane;
    const int dst = t < w4 ? 64 * (t & ~3) + 4 * lane + (t & 3) : pair;
    b[beg + dst] = (float)a[beg + pair];
  }
}


// Box aggregates of edge e: row (i, j, k) of problem p -> coarse (i/e, j/e, k/e) of
// problem p; an axis of extent 1 is not coarsened.  For e = 2, children[I*8 + c]
// lists the rows of aggregate I in ascending order (z, then y, then x), -1 padded.
__global__ void k_agg(int64_t n, int nx, int ny, int nz, int e, int cx, int cy, int cz, int32_t* __restrict__ agg) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  const int64_t per = (int64_t)nx * ny * nz;
  const int64_t p = r / per, q = r % per;
  const int i = (int)(q % nx), j = (int)((q / nx) % ny), k = (int)(q / ((int64_t)nx * ny));
  const int ci = nx == 1 ? i : i / e, cj = ny == 1 ? j : j / e, ck = nz == 1 ? k : k / e;
  agg[r] = (int32_t)(p * (int64_t)cx * cy * cz + ci + (int64_t)cx * cj + (int64_t)cx * cy * ck);
}

__global__ void k_children(int64_t nc, int nx, int ny, int nz, int cx, int cy, int cz, int32_t* __restrict__ ch) {
  const int64_t I = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (I >= nc) return;
  const int64_t cper = (int64_t)cx * cy * cz, per = (int64_t)nx * ny * nz;
  const int64_t p = I / cper, q = I % cper;
  const int ci = (int)(q % cx), cj = (int)((q / cx) % cy), ck = (int)(q / ((int64_t)cx * cy));
  const int sx = nx == 1 ? 1 : 2, sy = ny == 1 ? 1 : 2, sz = nz == 1 ? 1 : 2;
  int c = 0;
  for (int dz = 0; dz < sz; ++dz) {
    const int k = ck * sz + dz;
    if (k >= nz) continue;
    for (int dy = 0; dy < sy; ++dy) {
      const int j = cj * sy + dy;
      if (j >= ny) continue;
      for (int dx = 0; dx < sx; ++dx) {
        const int i = ci * sx + dx;
        if (i >= nx) continue;
        ch[I * kMaxChildren + c++] = (int32_t)(p * per + i + (int64_t)nx * j + (int64_t)nx * ny * k);
      }
    }
  }
  for (; c < kMaxChildren; ++c) ch[I * kMaxChildren + c] = -1;
}

// Galerkin row I of P^T A P: sum the entries of the aggregate's rows, mapping
// column j to agg[j].  Columns kept sorted in a small per-thread list
// (insertion), duplicates merged.  Pass 0 counts, pass 1 writes.
constexpr int kRapCap = 64;

template <bool FILL>
__global__ __launch_bounds__(64) void k_rap(int64_t nc, const int32_t* __restrict__ ptr,
                                            const int32_t* __restrict__ col, const double* __restrict__ val,
                                            const int32_t* __restrict__ agg, const int32_t* __restrict__ ch,
                                            int32_t* __restrict__ cnt_or_ptr, int32_t* __restrict__ ccol,
                                            double* __restrict__ cval, int* __restrict__ flag) {
  const int64_t I = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (I >= nc) return;
  int32_t cols[kRapCap];
  double vals[kRapCap];
  int m = 0;
  bool over = false;
  for (int c = 0; c < kMaxChildren; ++c) {
    const int i = ch[I * kMaxChildren + c];
    if (i < 0) break;
    for (int p = ptr[i]; p < ptr[i + 1]; ++p) {
      const int32_t J = agg[col[p]];
      const double v = val[p];
      int pos = m;
      while (pos > 0 && cols[pos - 1] > J) --pos;
      if (pos > 0 && cols[pos - 1] == J) {
        vals[pos - 1] += v;
      } else if (m < kRapCap) {
        for (int t = m; t > pos; --t) {
          cols[t] = cols[t - 1];
          vals[t] = vals[t - 1];
        }
        cols[pos] = J;
        vals[pos] = v;
        ++m;
      } else {
        over = true;
      }
    }
  }
  if (over) flag[F_CAPACITY] = 1;
  if (!FILL) {
    cnt_or_ptr[I] = m;
  } else {
    const int base = cnt_or_ptr[I];
    for (int t = 0; t < m; ++t) {
      ccol[base + t] = cols[t];
      cval[base + t] = vals[t];
    }
  }
}

// entries of the dense matrices, zeroed beforehand; padding rows get a unit diagonal
__global__ void k_to_dense(int64_t total_rows, int64_t nl, int64_t np, const int32_t* __restrict__ ptr,
                           const int32_t* __restrict__ col, const double* __restrict__ val,
                           double* __restrict__ dense, int* __restrict__ flag) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= total_rows) return;
  const int64_t p = r / np, lr = r % np;
  double* row = dense + p * np * np + lr * np;
  if (lr >= nl) {
    row[lr] = 1.0;  // padding: identity
    return;
  }
  const int64_t g = p * nl + lr;
  for (int q = ptr[g]; q < ptr[g + 1]; ++q) {
    const int64_t c = col[q] - p * nl;
    if (c >= 0 && c < nl) {
      row[c] = val[q];
    } else {
      flag[F_NOTSPD] = 1;  // coupling between stacked problems: not block diagonal
    }
  }
}

}  // namespace

int validate_csr(hipStream_t s, int64_t n, int64_t nnz, const int32_t* ptr, const int32_t* col, int* flag) {
  int h[F_NFLAG];
  hipLaunchKernelGGL(k_check_ptr, dim3(grid_for(n + 1)), dim3(kBlock), 0, s, n, nnz, ptr, flag);
  AMGP_HIP(hipGetLastError());
  AMGP_HIP(hipMemcpyAsync(h, flag, sizeof(h), hipMemcpyDeviceToHost, s));
  AMGP_HIP(hipStreamSynchronize(s));
  if (h[F_BADCSR]) return AMG_EINVAL;
  hipLaunchKernelGGL(k_check_col, dim3(grid_for(n)), dim3(kBlock), 0, s, n, ptr, col, flag);
  AMGP_HIP(hipGetLastError());
  AMGP_HIP(hipMemcpyAsync(h, flag, sizeof(h), hipMemcpyDeviceToHost, s));
  AMGP_HIP(hipStreamSynchronize(s));
  return h[F_BADCSR] ? AMG_EINVAL : AMG_OK;
}

int launch_l1_diag(hipStream_t s, int64_t n, const int32_t* ptr, const int32_t* col, const double* val,
                   double* minv, int* flag) {
  hipLaunchKernelGGL(k_l1_diag, dim3(grid_for(n)), dim3(kBlock), 0, s, n, ptr, col, val, minv, flag);
  return hipGetLastError() == hipSuccess ? AMG_OK : AMG_EHIP;
}

// Uniform slices are kept as patterns when they are at least half of the matrix's (a matrix of
// constant coefficients: all but the slices that cross an odd boundary); below that most slices
// stay dense and the plain kernels, which have no pattern path, serve them faster.  Wide triples (27
// points) in FP32 hierarchies below 2^18 rows keep their values too, which the L2 caches hold (time of a step
// of a smoother application, values -> patterns: 40^3 rows 3.3 -> 4.0 us, 56^3 4.0 -> 4.5, 64^3 5.3 -> 4.8,
// 80^3 11.4 -> 7.0; FP64 40^3 4.2 -> 4.3, 48^3 5.3 -> 4.8).
constexpr int kWideTripleSteps = 24;
constexpr int64_t kTriplesMinRows32 = int64_t(1) << 18;
constexpr int64_t kUniformMaxRows = int64_t(1) << 28;  // 32-bit byte offsets of the full slices' gathers

// Mirrored diagonals for the matrix of the given slices when it is large enough to be bound by its
// bytes, its offsets are few and come in pairs, storing half of them takes at most 65% of the dense
// slices' room (a wide pad or many rows at a boundary take more), and it is symmetric in every
// bit; out->mir stays null otherwise.  Smaller levels are bound by latency, where the dense slices'
// two steps per load win: with the 262144 rows of a 64^3 level mirrored its solve took 2.22 instead of
// 2.13 ms.
constexpr int64_t kMirrorMinRows = int64_t(1) << 19;

static int build_mirror(hipStream_t s, int64_t n, const int32_t* ptr, const int32_t* col, const double* val,
                        int64_t nslices, const int32_t* offs, const int32_t* width, int64_t aligned,
                        Ell<double>* out) {
  using graph::DevBuf;
  DevBuf<int32_t> buf;  // table, count, upper offsets
  DevBuf<unsigned long long> differ;
  AMGP_TRY(buf.alloc(kOffHash + 1 + kMirrorMaxSteps));
  AMGP_TRY(differ.alloc(3));
  int32_t *table = buf.p, *count = table + kOffHash, *dup = count + 1;
  hipLaunchKernelGGL(k_fill_int, dim3(1), dim3(kOffHash), 0, s, kOffHash, kOffEmpty, table);
  AMGP_HIP(hipMemsetAsync(count, 0, sizeof(int32_t), s));
  hipLaunchKernelGGL(k_union_offsets, dim3(grid_for(nslices * kSlice)), dim3(kBlock), 0, s, nslices, offs, width, table,
                     count);
  int32_t h[kOffHash + 1];
  AMGP_HIP(hipMemcpyAsync(h, table, sizeof(h), hipMemcpyDeviceToHost, s));
  AMGP_HIP(hipStreamSynchronize(s));
  const int w = h[kOffHash];
  if (w > kMirrorMaxSteps || w % 2 == 0) return AMG_OK;
  std::vector<int32_t> o;
  for (int t = 0; t < kOffHash; ++t)
    if (h[t] != kOffEmpty) o.push_back(h[t]);
  std::sort(o.begin(), o.end());
  if ((int)o.size() != w) return AMG_OK;
  for (int t = 0; t < w; ++t)
    if (o[t] != -o[w - 1 - t]) return AMG_OK;
  const int nup = w / 2 + 1;
  const int64_t pad = (o[w - 1] + 31) / 32 * 32, stride = (pad + n + 31) / 32 * 32;
  if (nup * stride > aligned / 100 * 65) return AMG_OK;
  std::vector<MirrorStep> st(w);
  for (int t = 0; t < w; ++t) {
    const int k = std::abs(t - w / 2);
    st[t] = MirrorStep{k * stride + pad + std::min(o[t], 0), o[t], 0};
  }
  double* v = nullptr;
  if (temp_malloc(&v, sizeof(double) * nup * stride) != hipSuccess) return AMG_ENOMEM;
  unsigned long long d[3] = {1, 0, 0};
  const int rc = [&]() -> int {
    AMGP_HIP(hipMemsetAsync(v, 0, sizeof(double) * nup * stride, s));
    AMGP_HIP(hipMemsetAsync(differ.p, 0, sizeof(d), s));
    AMGP_HIP(hipMemcpyAsync(dup, o.data() + w / 2, sizeof(int32_t) * nup, hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(k_mirror<false>, dim3(grid_for(n)), dim3(kBlock), 0, s, n, ptr, col, val, nup, dup, stride, pad,
                       v, differ.p);
    hipLaunchKernelGGL(k_mirror<true>, dim3(grid_for(n)), dim3(kBlock), 0, s, n, ptr, col, val, nup, dup, stride, pad,
                       v, differ.p);
    AMGP_HIP(hipMemcpyAsync(d, differ.p, sizeof(d), hipMemcpyDeviceToHost, s));
    AMGP_HIP(hipStreamSynchronize(s));
    if (d[0] || d[1] != d[2]) return AMG_OK;
    MirrorStep* m = nullptr;
    if (keep_malloc(&m, sizeof(MirrorStep) * w) != hipSuccess ||
        keep_malloc(&out->doff, sizeof(int32_t) * nslices) != hipSuccess)
      return AMG_ENOMEM;
    AMGP_HIP(hipMemcpyAsync(m, st.data(), sizeof(MirrorStep) * w, hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(k_mirror_present, dim3(grid_for(nslices)), dim3(kBlock), 0, s, nslices, offs, width, w,
                       (const MirrorStep*)m, out->doff);
    AMGP_HIP(hipGetLastError());
    AMGP_HIP(settle(s, &v, sizeof(double) * nup * stride));
    AMGP_HIP(hipStreamSynchronize(s));
    out->mir = m;
    out->nmir = w;
    out->val = v;
    out->dense = nup * stride;
    return AMG_OK;
  }();
  if (!out->mir) dev_free(v);
  return rc;
}

// Patterns of the uniform slices (64 rpl rows each) that k_slice_layout<false, rpl> found, and all
// slices' descriptors.
static int build_patterns(hipStream_t s, int rpl, int64_t n, const int32_t* ptr, const int32_t* col, const double* val,
                          const int32_t* anchor, int astride, int64_t nslices, const int32_t* offs, int32_t* wd,
                          int32_t* kind, int wmax, int64_t uniform, Ell<double>* e) {
  unsigned cap = 64;
  while (cap < 2 * nslices + 2) cap *= 2;  // its slices' room serves two scans of nslices + 1 later
  // per slice and step the value and the masks, per slice the hash; the table's keys, then its slices, and rep
  graph::DevBuf<unsigned long long> tab;
  AMGP_TRY(tab.alloc(nslices * ((1 + rpl) * wmax + 1) + cap + (cap + nslices + 1) / 2));
  unsigned long long *vtab = tab.p, *mtab = vtab + nslices * wmax, *hash = mtab + nslices * rpl * wmax,
                     *keys = hash + nslices;
  int32_t *first = reinterpret_cast<int32_t*>(keys + cap), *rep = first + cap;
  const dim3 grid((unsigned)nslices), each(grid_for(nslices));
  if (rpl == 1)
    hipLaunchKernelGGL((k_slice_layout<true, 1>), grid, dim3(kWave), 0, s, n, ptr, col, val, anchor, astride,
                       const_cast<int32_t*>(offs), wd, nullptr, kind, wmax, vtab, mtab, hash);
  else
    hipLaunchKernelGGL((k_slice_layout<true, 2>), grid, dim3(kWave), 0, s, n, ptr, col, val, anchor, astride,
                       const_cast<int32_t*>(offs), wd, nullptr, kind, wmax, vtab, mtab, hash);
  AMGP_HIP(hipMemsetAsync(keys, 0, sizeof(unsigned long long) * cap, s));
  AMGP_HIP(hipMemsetAsync(first, 0x7f, sizeof(int32_t) * cap, s));
  hipLaunchKernelGGL(k_pattern_insert, each, dim3(kBlock), 0, s, nslices, kind, hash, cap, keys, first);
  hipLaunchKernelGGL(k_pattern_resolve, each, dim3(kBlock), 0, s, nslices, kind, hash, cap, keys, first, offs, wd, rpl,
                     wmax, vtab, mtab, rep);
  // where every slice begins among the stored values or the patterns' steps (the table's slices are
  // done with)
  int32_t *dbeg = first, *pbeg = first + nslices + 1;
  hipLaunchKernelGGL(k_slice_store, each, dim3(kBlock), 0, s, nslices, wd, kind, rep, dbeg, pbeg);
  int rc = AMG_OK;
  e->dense = scan_ptr(s, nslices, dbeg, dbeg, &rc) * kSlice * rpl;
  AMGP_TRY(rc);
  e->npat = scan_ptr(s, nslices, pbeg, pbeg, &rc);
  AMGP_TRY(rc);
  e->patterned = uniform;
  e->rpl = rpl;
  if (keep_malloc(&e->desc, sizeof(int2) * nslices) != hipSuccess ||
      keep_malloc(&e->pat, pattern_bytes(e->npat, rpl)) != hipSuccess)
    return AMG_ENOMEM;
  hipLaunchKernelGGL(k_slice_desc, each, dim3(kBlock), 0, s, nslices, wd, kind, rep, dbeg, pbeg, e->desc);
  hipLaunchKernelGGL(k_pattern_write, dim3(grid_for(nslices * kSlice)), dim3(kBlock), 0, s, nslices, rep, e->desc, offs,
                     rpl, wmax, vtab, mtab, (int)e->npat, e->pat);
  AMGP_HIP(hipGetLastError());
  AMGP_HIP(hipStreamSynchronize(s));  // tab leaves scope
  return AMG_OK;
}

static int slice_stats(hipStream_t s, int64_t nslices, const int32_t* wd, const int32_t* lw, const int32_t* kind,
                       unsigned long long (&st)[ST_COUNT]) {
  graph::DevBuf<unsigned long long> stat;
  AMGP_TRY(stat.alloc(ST_COUNT));
  AMGP_HIP(hipMemsetAsync(stat.p, 0, sizeof(st), s));
  hipLaunchKernelGGL(k_slice_stats, dim3(std::min(256u, grid_for(nslices))), dim3(kBlock), 0, s, nslices, wd, lw, kind,
                     stat.p);
  AMGP_HIP(hipMemcpyAsync(st, stat.p, sizeof(st), hipMemcpyDeviceToHost, s));
  AMGP_HIP(hipStreamSynchronize(s));
  return AMG_OK;
}

// Offset-aligned sliced ELL (one row per lane) when every slice has at most 64 distinct column
// offsets and the layout is at most 10% larger than the packed one; AMG_EINVAL otherwise.
int build_ell_aligned(hipStream_t s, int64_t n, const int32_t* ptr, const int32_t* col, const double* val,
                      Ell<double>* out, const int32_t* anchor, int astride, int64_t ncols, bool any_size,
                      bool single, bool patterns) {
  using graph::DevBuf;
  const int64_t nslices = (n + kSlice - 1) / kSlice;
  // per slice: the sorted offsets (64), their count, the packed width, the kind
  DevBuf<int32_t> buf, buf2;
  AMGP_TRY(buf.alloc(nslices * (kSlice + 3)));
  int32_t *offs = buf.p, *wd = offs + nslices * kSlice, *lw = wd + nslices, *kind = lw + nslices;
  const bool try_uniform = n < kUniformMaxRows && (ncols < 0 ? n : ncols) < kUniformMaxRows;
  hipLaunchKernelGGL((k_slice_layout<false, 1>), dim3((unsigned)nslices), dim3(kWave), 0, s, n, ptr, col, val, anchor,
                     astride, offs, wd, lw, try_uniform ? kind : nullptr, 0, nullptr, nullptr, nullptr);
  unsigned long long st[ST_COUNT];
  AMGP_TRY(slice_stats(s, nslices, wd, lw, try_uniform ? kind : nullptr, st));
  if (st[ST_OVER]) return AMG_EINVAL;
  const int64_t aligned = (int64_t)st[ST_ALIGNED] * kSlice, packed = (int64_t)st[ST_PACKED] * kSlice;
  if ((!any_size && aligned > packed + packed / 10) || aligned >= (int64_t)INT32_MAX) return AMG_EINVAL;
  Ell<double> e;
  e.n = n;
  e.ncols = ncols < 0 ? n : ncols;
  e.anchor = anchor;
  e.astride = astride;
  e.group = 1;
  e.nslices = nslices;
  e.padded = aligned;
  const int rc = [&]() -> int {
    const bool square = !anchor && e.ncols == n;
    const bool wide_triples = aligned >= kWideTripleSteps * n && 2 * (int64_t)st[ST_TRIPLES] >= nslices;
    const bool compact = patterns && !(single && wide_triples && n < kTriplesMinRows32) &&
                         2 * (int64_t)st[ST_UNIFORM] >= nslices;
    if (compact && square && !single && n >= kPairMinRows) {
      // the operator itself: slices of 128 rows, two rows per lane, where half of those are uniform too
      // (not where every second slice of 64 rows has a line's end in it with a value of its own)
      const int64_t ns = (n + 2 * kSlice - 1) / (2 * kSlice);
      AMGP_TRY(buf2.alloc(ns * (kSlice + 3)));
      int32_t *offs2 = buf2.p, *wd2 = offs2 + ns * kSlice, *lw2 = wd2 + ns, *kind2 = lw2 + ns;
      hipLaunchKernelGGL((k_slice_layout<false, 2>), dim3((unsigned)ns), dim3(kWave), 0, s, n, ptr, col, val, anchor,
                         astride, offs2, wd2, lw2, kind2, 0, nullptr, nullptr, nullptr);
      unsigned long long st2[ST_COUNT];
      AMGP_TRY(slice_stats(s, ns, wd2, lw2, kind2, st2));
      if (!st2[ST_OVER] && 2 * (int64_t)st2[ST_UNIFORM] >= ns) {
        e.nslices = ns;
        AMGP_TRY(build_patterns(s, 2, n, ptr, col, val, anchor, astride, ns, offs2, wd2, kind2,
                                std::max(1, (int)st2[ST_WIDEST]), (int64_t)st2[ST_UNIFORM], &e));
        if (keep_malloc(&e.val, sizeof(double) * std::max<int64_t>(e.dense, 1)) != hipSuccess ||
            keep_malloc(&e.doff, sizeof(int32_t) * std::max<int64_t>(e.dense / (2 * kSlice), 1)) != hipSuccess)
          return AMG_ENOMEM;
        AMGP_HIP(hipMemsetAsync(e.doff, 0, sizeof(int32_t) * (e.dense / (2 * kSlice)), s));
        if (e.dense > 0)
          hipLaunchKernelGGL(k_ell_fill_pairs, dim3(grid_for(ns * 2 * kSlice)), dim3(kBlock), 0, s, n, ptr, col, val,
                             offs2, e.desc, e.val, e.doff);
        AMGP_HIP(hipGetLastError());
        AMGP_HIP(hipStreamSynchronize(s));
        return AMG_OK;
      }
    }
    if (compact) {
      AMGP_TRY(build_patterns(s, 1, n, ptr, col, val, anchor, astride, nslices, offs, wd, kind,
                              std::max(1, (int)st[ST_WIDEST]), (int64_t)st[ST_UNIFORM], &e));
    } else {
      if (square && n >= kMirrorMinRows && n < kUniformMaxRows) {
        AMGP_TRY(build_mirror(s, n, ptr, col, val, nslices, offs, wd, aligned, &e));
        if (e.mir) return AMG_OK;
      }
      e.dense = aligned;
      if (keep_malloc(&e.sptr, sizeof(int32_t) * (nslices + 1)) != hipSuccess) return AMG_ENOMEM;
      int rc2 = AMG_OK;
      scan_ptr(s, nslices, wd, e.sptr, &rc2, 1, kSlice);
      AMGP_TRY(rc2);
    }
    if (keep_malloc(&e.val, sizeof(double) * std::max<int64_t>(e.dense, 1)) != hipSuccess ||
        keep_malloc(&e.doff, sizeof(int32_t) * std::max<int64_t>(e.dense / kSlice, 1)) != hipSuccess)
      return AMG_ENOMEM;
    if (e.dense > 0)
      hipLaunchKernelGGL(k_ell_fill_aligned, dim3(grid_for(nslices * kSlice)), dim3(kBlock), 0, s, n, nslices, ptr,
                         col, val, anchor, astride, offs, e.sptr, e.desc, e.val, e.doff);
    AMGP_HIP(hipGetLastError());
    AMGP_HIP(hipStreamSynchronize(s));
    return AMG_OK;
  }();
  if (rc != AMG_OK) {
    hipStreamSynchronize(s);
    free_ell(e);
    return rc;
  }
  *out = e;
  return AMG_OK;
}

int build_ell64(hipStream_t s, int64_t n, const int32_t* ptr, const int32_t* col, const double* val,
                Ell<double>* out, int64_t ncols, int group, bool single) {
  if (ncols < 0) ncols = n;
  if (group == 0) {
    // lanes per row from the mean row length: about four entries or more per lane
    int32_t last = 0;
    AMGP_HIP(hipMemcpyAsync(&last, ptr + n, sizeof(int32_t), hipMemcpyDeviceToHost, s));
    AMGP_HIP(hipStreamSynchronize(s));
    const double mean = (double)last / (double)n;
    group = mean >= 256 ? 64 : mean >= 64 ? 16 : mean >= 16 ? 4 : 1;
    if (group == 4 && n >= kAlignedWideMinRows && ncols == n) {
      // a coarse stencil (27 points on Q1 boxes) on a large level: one row per lane without
      // column indices moves 4 bytes less per entry than four lanes per row with them
      const int rc = build_ell_aligned(s, n, ptr, col, val, out, nullptr, 1, -1, false, single);
      if (rc != AMG_EINVAL) return rc;
    }
  }
  if (group != 1 && group != 4 && group != 16 && group != 64) return AMG_EINVAL;
  if (group == 1 && ncols == n) {
    const int rc = build_ell_aligned(s, n, ptr, col, val, out, nullptr, 1, -1, false, single);
    if (rc != AMG_EINVAL) return rc;  // EINVAL: the slices are not offset-aligned; use the packed layout
  }
  const int R = kSlice / group;
  Ell<double> e;
  e.n = n;
  e.group = group;
  e.nslices = (n + R - 1) / R;
  int32_t* dw = nullptr;
  AMGP_HIP(temp_malloc(&dw, sizeof(int32_t) * e.nslices));
  hipLaunchKernelGGL(k_slice_width, dim3(grid_for(e.nslices)), dim3(kBlock), 0, s, n, e.nslices, R, ptr, dw);
  if (keep_malloc(&e.sptr, sizeof(int32_t) * (e.nslices + 1)) != hipSuccess) {
    dev_free(dw);
    return AMG_ENOMEM;
  }
  int rc = AMG_OK;
  const int64_t acc = scan_ptr(s, e.nslices, dw, e.sptr, &rc, group, kSlice);
  dev_free(dw);
  if (rc != AMG_OK) {
    free_ell(e);
    return rc;
  }
  e.padded = acc;
  if (keep_malloc(&e.col, sizeof(int32_t) * std::max<int64_t>(acc, 1)) != hipSuccess) return AMG_ENOMEM;
  if (keep_malloc(&e.val, sizeof(double) * std::max<int64_t>(acc, 1)) != hipSuccess) return AMG_ENOMEM;
  hipLaunchKernelGGL(k_ell_fill, dim3(grid_for(e.nslices * kSlice)), dim3(kBlock), 0, s, n, ncols, e.nslices, group,
                     ptr, col, val, e.sptr, e.col, e.val);
  AMGP_HIP(hipGetLastError());
  AMGP_HIP(hipStreamSynchronize(s));
  *out = e;
  return AMG_OK;
}

int build_ell32(hipStream_t s, const Ell<double>& a, Ell<float>* out) {
  Ell<float> e;
  e.n = a.n;
  e.ncols = a.ncols;
  e.anchor = a.anchor;
  e.astride = a.astride;
  e.nslices = a.nslices;
  e.padded = a.padded;
  e.group = a.group;
  e.npat = a.npat;
  e.dense = a.dense;
  e.patterned = a.patterned;
  e.nmir = a.nmir;
  const int64_t stored = a.doff ? a.dense : a.padded;
  auto copy = [&](auto** to, const auto* from, int64_t count) -> int {
    if (!from) return AMG_OK;
    if (keep_malloc(to, sizeof(**to) * std::max<int64_t>(count, 1)) != hipSuccess) return AMG_ENOMEM;
    AMGP_HIP(hipMemcpyAsync(*to, from, sizeof(**to) * count, hipMemcpyDeviceToDevice, s));
    return AMG_OK;
  };
  const int rc = [&]() -> int {
    AMGP_TRY(copy(&e.sptr, a.sptr, e.nslices + 1));
    AMGP_TRY(copy(&e.col, a.col, stored));
    AMGP_TRY(copy(&e.doff, a.doff, a.mir ? a.nslices : stored / kSlice));
    AMGP_TRY(copy(&e.mir, a.mir, a.nmir));
    AMGP_TRY(copy(&e.desc, a.desc, e.nslices));
    AMGP_TRY(copy(&e.pat, a.pat, pattern_bytes(e.npat, 1) / 8));
    if (keep_malloc(&e.val, sizeof(float) * std::max<int64_t>(stored, 1)) != hipSuccess) return AMG_ENOMEM;
    if (a.desc) {
      const EllView<double> av = view(a);
      const EllView<float> ev = view(e);
      hipLaunchKernelGGL(k_round_f32, dim3(grid_for(e.npat)), dim3(kBlock), 0, s, e.npat, av.pval(1),
                         const_cast<float*>(ev.pval(1)));
    }
    if (a.doff && !a.mir && stored > 0)
      hipLaunchKernelGGL(k_round_f32_aligned, dim3(grid_for(e.nslices * kSlice)), dim3(kBlock), 0, s, e.nslices,
                         e.sptr, e.desc, a.val, e.val);
    else if (!a.doff || a.mir)
      hipLaunchKernelGGL(k_round_f32, dim3(grid_for(stored)), dim3(kBlock), 0, s, stored, a.val, e.val);
    AMGP_HIP(hipGetLastError());
    return AMG_OK;
  }();
  if (rc != AMG_OK) {
    hipStreamSynchronize(s);
    free_ell(e);
    return rc;
  }
  *out = e;
  return AMG_OK;
}

template <typename T>
static void free_ell_of(Ell<T>& e) {
  dev_free(e.sptr);
  dev_free(e.col);
  dev_free(e.val);
  dev_free(e.doff);
  dev_free(e.desc);
  dev_free(e.pat);
  dev_free(e.mir);
  e = Ell<T>();
}
void free_ell(Ell<double>& e) { free_ell_of(e); }
void free_ell(Ell<float>& e) { free_ell_of(e); }

int launch_aggregates(hipStream_t s, int nx, int ny, int nz, int nbatch, int e, int32_t* agg, int32_t* children,
                      int* cnx, int* cny, int* cnz) {
  if (e < 2 || (children && e != 2)) return AMG_EINVAL;
  const int cx = nx == 1 ? 1 : (nx + e - 1) / e, cy = ny == 1 ? 1 : (ny + e - 1) / e,
            cz = nz == 1 ? 1 : (nz + e - 1) / e;
  const int64_t n = (int64_t)nx * ny * nz * nbatch, nc = (int64_t)cx * cy * cz * nbatch;
  hipLaunchKernelGGL(k_agg, dim3(grid_for(n)), dim3(kBlock), 0, s, n, nx, ny, nz, e, cx, cy, cz, agg);
  if (children)
    hipLaunchKernelGGL(k_children, dim3(grid_for(nc)), dim3(kBlock), 0, s, nc, nx, ny, nz, cx, cy, cz, children);
  *cnx = cx;
  *cny = cy;
  *cnz = cz;
  return hipGetLastError() == hipSuccess ? AMG_OK : AMG_EHIP;
}

int galerkin(hipStream_t s, int64_t n, const int32_t* ptr, const int32_t* col, const double* val,
             const int32_t* agg, int64_t nc, const int32_t* children, int32_t** cptr, int32_t** ccol,
             double** cval, int64_t* cnnz, int* flag) {
  (void)n;
  // the arrays belong to the caller as soon as they exist, also when a later step fails
  int32_t* cnt = nullptr;
  if (temp_malloc(&cnt, sizeof(int32_t) * (nc + 1)) != hipSuccess) return AMG_ENOMEM;
  *cptr = cnt;
  hipLaunchKernelGGL((k_rap<false>), dim3((unsigned)((nc + 63) / 64)), dim3(64), 0, s, nc, ptr, col, val, agg,
                     children, cnt, (int32_t*)nullptr, (double*)nullptr, flag);
  AMGP_HIP(hipGetLastError());
  int hflag[F_NFLAG];
  AMGP_HIP(hipMemcpyAsync(hflag, flag, sizeof(hflag), hipMemcpyDeviceToHost, s));
  AMGP_HIP(hipStreamSynchronize(s));
  if (hflag[F_CAPACITY]) return AMG_ECAPACITY;
  int rc = AMG_OK;
  const int64_t acc = scan_ptr(s, nc, cnt, cnt, &rc);
  if (rc != AMG_OK) return rc;
  if (temp_malloc(ccol, sizeof(int32_t) * std::max<int64_t>(acc, 1)) != hipSuccess) return AMG_ENOMEM;
  if (temp_malloc(cval, sizeof(double) * std::max<int64_t>(acc, 1)) != hipSuccess) return AMG_ENOMEM;
  hipLaunchKernelGGL((k_rap<true>), dim3((unsigned)((nc + 63) / 64)), dim3(64), 0, s, nc, ptr, col, val, agg,
                     children, cnt, *ccol, *cval, flag);
  AMGP_HIP(hipGetLastError());
  AMGP_HIP(hipStreamSynchronize(s));
  *cnnz = acc;
  return AMG_OK;
}

int launch_to_dense(hipStream_t s, int nbatch, int64_t nl, int64_t np, const int32_t* ptr, const int32_t* col,
                    const double* val, double* dense, int* flag) {
  const int64_t rows = (int64_t)nbatch * np;
  AMGP_HIP(hipMemsetAsync(dense, 0, sizeof(double) * rows * np, s));
  hipLaunchKernelGGL(k_to_dense, dim3(grid_for(rows)), dim3(kBlock), 0, s, rows, nl, np, ptr, col, val, dense,
                     flag);
  return hipGetLastError() == hipSuccess ? AMG_OK : AMG_EHIP;
}

}  // namespace amgp
