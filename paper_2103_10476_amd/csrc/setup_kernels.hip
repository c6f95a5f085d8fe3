// Setup kernels: CSR validation, strength of connection, the aggregation graph, parallel
// root selection, aggregation, Sprsfy, filtered matrix with its smoothing diagonal, power
// method, prolongator smoothing, Cnstrnt, transpose.
//
// Every floating-point reduction runs in the order the method's definition fixes (row sums
// sequential in ascending column order from 0), with FMA contraction disabled at compile
// time, so the setup is deterministic and equal to the sequential definition bit for bit.
// Most setup kernels work per entry, or with a few lanes or a wavefront per row; where a row's
// sums are a chain anyway and rows are short (5-30 entries on the fine levels) one thread has the
// row, its entries staged by the block where that pays.  They run once per level and are bound by
// HBM traffic, by chains of dependent loads or by the level's size.
#include <chrono>
#include <climits>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <type_traits>
#include <utility>

#include "kernels.hpp"

namespace sa {

#define SA_ROW_KERNEL_BEGIN(n)                                    \
  const int64_t i64_ = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; \
  if (i64_ >= (n)) return;                                        \
  const int32_t i = (int32_t)i64_;

// ---- one wavefront per row (levels with long rows) ------------------------------------------
// Kernels below with a _w suffix process one row per 64-thread block (one wavefront), lanes
// striding over the row.  Floating-point sums keep the sequential order: terms are staged in
// LDS 64 at a time and lane 0 adds them in ascending entry order from 0.  A term outside the
// summed subset contributes +0.0, which leaves a sum that started from +0.0 unchanged bit for
// bit (such a sum is never -0.0), so the result equals the sequential sum over the subset.
constexpr int kW = 64;
#define SA_WAVE_ROW_BEGIN(n)                        \
  const int32_t i = (int32_t)blockIdx.x;            \
  if (i >= (n)) return;                             \
  const int lane = threadIdx.x;

template <class F>
__device__ inline double wave_seq_sum(int32_t b, int32_t e, F term, double *lds) {
  const int lane = threadIdx.x;
  double acc = 0.0;
  for (int32_t c = b; c < e; c += kW) {
    const int32_t k = c + lane;
    lds[lane] = (k < e) ? term(k) : 0.0;
    __syncthreads();
    if (lane == 0) {
      const int32_t lim = min(kW, e - c);
      for (int32_t q = 0; q < lim; ++q) acc += lds[q];
    }
    __syncthreads();
  }
  if (lane == 0) lds[0] = acc;
  __syncthreads();
  const double r = lds[0];
  __syncthreads();
  return r;
}
__device__ inline int32_t wave_sum_i32(int32_t v) {
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
__device__ inline bool wave_any(bool p) { return __ballot(p) != 0; }

// ---- validation -----------------------------------------------------------------------
// Entry-parallel (a block owns kBlock rows, whose row pointers it stages in LDS and checks
// first; coalesced reads of col and val): bit 1 a row pointer or column out of range or
// columns not ascending, 2 a row without its diagonal entry, 4 a non-finite value, 2048 row
// pointers that do not start at 0 and end at nnz.  dval (may be null) gets the diagonal, which
// a search of its own in 970K rows of 26 entries took 206 us to find again.
__global__ __launch_bounds__(kBlock) void k_validate(int32_t n, int64_t nnz,
                                                     const int32_t *__restrict__ rp,
                                                     const int32_t *__restrict__ col,
                                                     const double *__restrict__ val,
                                                     double *__restrict__ dval, int32_t *err) {
  __shared__ int32_t s_rp[kBlock + 1];
  __shared__ uint8_t s_diag[kBlock];
  const int t = threadIdx.x;
  const int64_t r0 = (int64_t)blockIdx.x * kBlock;
  const int32_t nr = (int32_t)min<int64_t>(kBlock, (int64_t)n - r0);
  if (blockIdx.x == 0 && t == 0 && (rp[0] != 0 || (int64_t)rp[n] != nnz)) atomicOr(err, 2048);
  if (t < nr) s_rp[t] = rp[r0 + t];
  if (t == 0) s_rp[nr] = rp[r0 + nr];
  s_diag[t] = 0;
  __syncthreads();
  // the block's row pointers: within [0, nnz] and not decreasing, else nothing is read
  const bool bad = t < nr && (s_rp[t] < 0 || s_rp[t + 1] < s_rp[t] || (int64_t)s_rp[t + 1] > nnz);
  if (__syncthreads_or(bad)) {
    if (t == 0) atomicOr(err, 1);
    return;
  }
  const int32_t e0 = s_rp[0], e1 = s_rp[nr];
  int32_t flags = 0;
  for (int32_t e = e0 + t; e < e1; e += kBlock) {
    int32_t lo = 0, hi = nr - 1;  // the entry's row: the last r with s_rp[r] <= e
    while (lo < hi) {
      const int32_t mid = (lo + hi + 1) >> 1;
      if (s_rp[mid] <= e) lo = mid;
      else hi = mid - 1;
    }
    const int32_t c = col[e];
    if (c < 0 || c >= n) flags |= 1;
    if (e > s_rp[lo] && c <= col[e - 1]) flags |= 1;
    if (c == (int32_t)r0 + lo) {
      s_diag[lo] = 1;
      if (dval) dval[c] = val[e];
    }
    if (val && !isfinite(val[e])) flags |= 4;
  }
  __syncthreads();
  if (t < nr && !s_diag[t]) flags |= 2;
  if (flags) atomicOr(err, flags);
}

// nnz: the length of col and val (rp[n] is checked against it on the device).
void validate_csr(int32_t n, int64_t nnz, const int32_t *rp, const int32_t *col,
                  const double *val, double *dval, int32_t *err, hipStream_t s) {
  k_validate<<<grid_for(n), kBlock, 0, s>>>(n, nnz, rp, col, val, dval, err);
  SA_LAUNCH_CHECK();
}
__global__ void k_find_diag(int32_t n, const int32_t *rp, const int32_t *col, const double *val,
                            double *dval) {
  SA_ROW_KERNEL_BEGIN(n)
  int32_t lo = rp[i], hi = rp[i + 1] - 1;
  double d = 0.0;
  while (lo <= hi) {
    int32_t mid = (lo + hi) >> 1;
    int32_t c = col[mid];
    if (c == i) {
      d = val[mid];
      break;
    }
    if (c < i) lo = mid + 1;
    else hi = mid - 1;
  }
  dval[i] = d;
}
void find_diag(int32_t n, const int32_t *rp, const int32_t *col, const double *val,
               double *dval, hipStream_t s) {
  if (n <= 0) return;
  k_find_diag<<<grid_for(n), kBlock, 0, s>>>(n, rp, col, val, dval);
  SA_LAUNCH_CHECK();
}

// ---- strength (Sec. 1.1 criterion, evaluated squared) ----------------------------------
// Entry-parallel: block b owns rows [256 b, 256 b + 256), whose entries are one contiguous run;
// consecutive threads take consecutive entries (coalesced loads and mask stores), each finding
// its row by binary search over the block's row pointers in LDS; strong entries are counted per
// row with LDS integer atomics.
__global__ __launch_bounds__(kBlock) void k_strength(int32_t n, const int32_t *__restrict__ rp,
                                                     const int32_t *__restrict__ col,
                                                     const double *__restrict__ val,
                                                     const double *__restrict__ dval, double th2,
                                                     uint8_t *__restrict__ mask,
                                                     int32_t *__restrict__ scount) {
  __shared__ int32_t s_rp[kBlock + 1];
  __shared__ double s_d[kBlock];
  __shared__ int32_t s_cnt[kBlock];
  const int t = threadIdx.x;
  const int64_t r0 = (int64_t)blockIdx.x * kBlock;
  const int32_t nr = (int32_t)min<int64_t>(kBlock, (int64_t)n - r0);
  if (t < nr) {
    s_rp[t] = rp[r0 + t];
    s_d[t] = dval[r0 + t];
  }
  if (t == 0) s_rp[nr] = rp[r0 + nr];  // nr can be kBlock: no thread t == nr
  s_cnt[t] = 0;
  __syncthreads();
  const int32_t e0 = s_rp[0], e1 = s_rp[nr];
  for (int32_t e = e0 + t; e < e1; e += kBlock) {
    int32_t lo = 0, hi = nr - 1;  // the entry's row: the last r with s_rp[r] <= e
    while (lo < hi) {
      const int32_t mid = (lo + hi + 1) >> 1;
      if (s_rp[mid] <= e) lo = mid;
      else hi = mid - 1;
    }
    const int32_t j = col[e];
    uint8_t m = 3;
    if (j != (int32_t)r0 + lo) {
      const double a = val[e];
      const double p = s_d[lo] * dval[j];
      const bool strong = (p > 0.0) && (a * a >= th2 * p);
      m = strong ? 1 : 0;
      if (strong) atomicAdd(&s_cnt[lo], 1);
    }
    mask[e] = m;
  }
  __syncthreads();
  if (t < nr) scount[r0 + t] = s_cnt[t];
}
__global__ __launch_bounds__(kW) void k_strength_w(int32_t n, const int32_t *rp,
                                                   const int32_t *col, const double *val,
                                                   const double *dval, double th2,
                                                   uint8_t *mask, int32_t *scount) {
  SA_WAVE_ROW_BEGIN(n)
  const double di = dval[i];
  int32_t cnt = 0;
  for (int32_t k = rp[i] + lane; k < rp[i + 1]; k += kW) {
    const int32_t j = col[k];
    if (j == i) {
      mask[k] = 3;
      continue;
    }
    const double a = val[k];
    const double p = di * dval[j];
    const bool strong = (p > 0.0) && (a * a >= th2 * p);
    mask[k] = strong ? 1 : 0;
    cnt += strong;
  }
  cnt = wave_sum_i32(cnt);
  if (lane == 0) scount[i] = cnt;
}
void strength(int32_t n, const int32_t *rp, const int32_t *col, const double *val,
              const double *dval, double th2, uint8_t *mask, int32_t *scount, bool wave,
              hipStream_t s) {
  if (n <= 0) return;
  if (wave) k_strength_w<<<(unsigned)n, kW, 0, s>>>(n, rp, col, val, dval, th2, mask, scount);
  else k_strength<<<grid_for(n), kBlock, 0, s>>>(n, rp, col, val, dval, th2, mask, scount);
  SA_LAUNCH_CHECK();
}

// ---- distance-Laplacian weights (Sec. 3.1) -------------------------------------------------
// The strength test can be taken on a Laplacian built from node coordinates instead of on A:
// same pattern, off-diagonal weight w = 1/d^P with d the distance (the squared distance d2
// summed over the coordinates in order from 0; P = 1: 1/sqrt(d2), both correctly rounded;
// P = 2: 1/d2), diagonal Ld[i] = the row's weights summed in ascending column order from 0.
// k_strength then runs on (w, Ld) unchanged: |L_ij| >= theta sqrt(L_ii L_jj) squared is
// w^2 >= theta^2 Ld_i Ld_j.  A zero (or NaN) distance between two connected nodes
// sets err bit `ebit`.
template <int D>
__device__ inline double dist2(const double *__restrict__ xyz, int32_t i, int32_t j) {
  double d2 = 0.0;
#pragma unroll
  for (int k = 0; k < D; ++k) {
    const double t = xyz[(int64_t)i * D + k] - xyz[(int64_t)j * D + k];
    d2 = d2 + t * t;
  }
  return d2;
}
// 8 lanes per row (a thread per row left its loads a chain and its lines to 64 rows: 205K rows of
// 26 entries 164 us, now 29); the row's sum goes through the lanes in entry order.
template <int D, int P>
__global__ __launch_bounds__(kBlock) void k_distance_weights(
    int32_t n, const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
    const double *__restrict__ xyz, double *w, double *Ld, int32_t *err, int32_t ebit) {
  const int lane = threadIdx.x & 7;
  bool bad = false;
  for (int64_t i64 = first_row<8>(); i64 < n; i64 += row_stride<8>()) {  // uniform over the lanes
    const int32_t i = (int32_t)i64;
    const int32_t e = rp[i + 1];
    double s = 0.0;
    for (int32_t k = rp[i]; k < e; k += 8) {
      double wk = 0.0;  // the diagonal's, and past the row: leaves the sum as it is
      if (k + lane < e) {
        const int32_t j = col[k + lane];
        if (j != i) {
          const double d2 = dist2<D>(xyz, i, j);
          bad |= !(d2 > 0.0);
          wk = P == 1 ? 1.0 / sqrt(d2) : 1.0 / d2;
        }
        w[k + lane] = wk;
      }
#pragma unroll
      for (int o = 0; o < 8; ++o) s = s + __shfl(wk, o, 8);
    }
    if (lane == 0) Ld[i] = s;
  }
  if (bad) atomicOr(err, ebit);
}
template <int D>
static void distance_weights_dim(int32_t n, const int32_t *rp, const int32_t *col,
                                 const double *xyz, int32_t power, double *w, double *Ld,
                                 int32_t *err, int32_t ebit, hipStream_t s) {
  if (power == 1)
    k_distance_weights<D, 1><<<grid_rows(n, 8), kBlock, 0, s>>>(n, rp, col, xyz, w, Ld, err,
                                                              ebit);
  else
    k_distance_weights<D, 2><<<grid_rows(n, 8), kBlock, 0, s>>>(n, rp, col, xyz, w, Ld, err,
                                                              ebit);
}
void distance_weights(int32_t n, const int32_t *rp, const int32_t *col, const double *xyz,
                      int32_t dim, int32_t power, double *w, double *Ld, int32_t *err,
                      int32_t ebit, hipStream_t s) {
  if (n <= 0) return;
  if (power != 1 && power != 2) throw Error(SA_ERR_INVALID_ARG, "dist_power");
  switch (dim) {
    case 1: distance_weights_dim<1>(n, rp, col, xyz, power, w, Ld, err, ebit, s); break;
    case 2: distance_weights_dim<2>(n, rp, col, xyz, power, w, Ld, err, ebit, s); break;
    case 3: distance_weights_dim<3>(n, rp, col, xyz, power, w, Ld, err, ebit, s); break;
    default: throw Error(SA_ERR_INVALID_ARG, "coordinate dimension");
  }
  SA_LAUNCH_CHECK();
}

__global__ void k_check_finite(int64_t m, const double *x, int32_t *err, int32_t ebit) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < m && !isfinite(x[i])) atomicOr(err, ebit);
}
void check_finite(const double *x, int64_t m, int32_t *err, int32_t ebit, hipStream_t s) {
  if (m <= 0) return;
  k_check_finite<<<grid_for(m), kBlock, 0, s>>>(m, x, err, ebit);
  SA_LAUNCH_CHECK();
}

// ---- coarse coordinates: aggregate centroids ---------------------------------------------
// Member lists by counting sort (count, scan, scatter, then each list sorted ascending), then
// one thread per aggregate sums its members' coordinates in ascending vertex order from 0
// and divides by the member count.
__global__ void k_count_members(int32_t n, const int32_t *agg, int32_t *cnt) {
  SA_ROW_KERNEL_BEGIN(n)
  if (agg[i] >= 0) atomicAdd(&cnt[agg[i]], 1);
}
__global__ void k_scatter_members(int32_t n, const int32_t *agg, int32_t *pos, int32_t *mem) {
  SA_ROW_KERNEL_BEGIN(n)
  if (agg[i] >= 0) mem[atomicAdd(&pos[agg[i]], 1)] = i;
}
// Member lists of the nc aggregates: mrp[nc+1] offsets into mem[n] (unaggregated vertices
// left out); members in scatter order, or ascending when `sorted`.
void member_lists(int32_t n, const int32_t *agg, int32_t nc, bool sorted, Arena &ar,
                  int32_t **mrp_out, int32_t **mem_out, hipStream_t s) {
  int32_t *cnt = ar.alloc<int32_t>(nc + 1);
  int32_t *mrp = ar.alloc<int32_t>(nc + 1);
  int32_t *mem = ar.alloc<int32_t>(n > 0 ? n : 1);
  fill_i32(cnt, 0, nc + 1, s);
  if (n > 0) {
    k_count_members<<<grid_for(n), kBlock, 0, s>>>(n, agg, cnt);
    SA_LAUNCH_CHECK();
  }
  exclusive_scan_i32(cnt, mrp, nc, s);
  SA_HIP(hipMemcpyAsync(cnt, mrp, sizeof(int32_t) * (nc + 1), hipMemcpyDeviceToDevice, s));
  if (n > 0) {
    k_scatter_members<<<grid_for(n), kBlock, 0, s>>>(n, agg, cnt, mem);
    SA_LAUNCH_CHECK();
  }
  if (sorted) sort_rows(nc, mrp, mem, nullptr, s);
  *mrp_out = mrp;
  *mem_out = mem;
}
__global__ void k_centroids(int32_t nc, int32_t dim, const int32_t *mrp, const int32_t *mem,
                            const double *__restrict__ xyz, double *cxyz) {
  SA_ROW_KERNEL_BEGIN(nc)
  const int32_t b = mrp[i], e = mrp[i + 1];
  for (int k = 0; k < dim; ++k) {
    double s = 0.0;
    for (int32_t q = b; q < e; ++q) s = s + xyz[(int64_t)mem[q] * dim + k];
    cxyz[(int64_t)i * dim + k] = s / (double)(e - b);
  }
}
void aggregate_centroids(int32_t n, const int32_t *agg, int32_t nc, const double *xyz,
                         int32_t dim, double *cxyz, hipStream_t s) {
  if (nc <= 0) return;
  Arena tmp;
  tmp.stream = s;
  int32_t *mrp, *mem;
  member_lists(n, agg, nc, true, tmp, &mrp, &mem, s);
  k_centroids<<<grid_for(nc), kBlock, 0, s>>>(nc, dim, mrp, mem, xyz, cxyz);
  SA_LAUNCH_CHECK();
}

// ---- aggregation graph G = S u S^T ------------------------------------------------------
// The strong entries of 256 rows are one contiguous run of scol, in entry order: the block
// takes its rows' entries 256 at a time and packs the strong ones behind those before.  Each
// also takes its place in its column's list (trank), so the transpose needs no second count.
__global__ __launch_bounds__(kBlock) void k_fill_strong(int32_t n, const int32_t *__restrict__ rp,
                                                        const int32_t *__restrict__ col,
                                                        const uint8_t *__restrict__ mask,
                                                        const int32_t *__restrict__ srp,
                                                        int32_t *__restrict__ scol,
                                                        int32_t *tcnt,
                                                        int32_t *__restrict__ trank) {
  __shared__ int32_t s_n[2][kBlock / 64];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int64_t r0 = (int64_t)blockIdx.x * kBlock;
  const int64_t r1 = min<int64_t>(n, r0 + kBlock);
  const int32_t e0 = rp[r0], e1 = rp[r1];
  int32_t w = srp[r0];
  int h = 0;
  for (int32_t c = e0; c < e1; c += kBlock, h ^= 1) {
    const int32_t e = c + t;
    const uint8_t m = e < e1 ? mask[e] : (uint8_t)0;
    const bool st = m == 1 || m == 2;
    const uint64_t bm = __ballot(st);
    if (lane == 0) s_n[h][wv] = __popcll(bm);
    __syncthreads();  // (the other half's counts are read before this round's barrier)
    int32_t before = 0, all = 0;
#pragma unroll
    for (int q = 0; q < kBlock / 64; ++q) {
      before += q < wv ? s_n[h][q] : 0;
      all += s_n[h][q];
    }
    if (st) {
      const int32_t pos = w + before + __popcll(bm & ((1ull << lane) - 1ull));
      const int32_t j = col[e];
      scol[pos] = j;
      trank[pos] = atomicAdd(&tcnt[j], 1);
    }
    w += all;
  }
}
__global__ __launch_bounds__(kW) void k_fill_strong_w(int32_t n, const int32_t *rp,
                                                      const int32_t *col, const uint8_t *mask,
                                                      const int32_t *srp, int32_t *scol,
                                                      int32_t *tcnt, int32_t *trank) {
  SA_WAVE_ROW_BEGIN(n)
  int32_t w = srp[i];
  for (int32_t c = rp[i]; c < rp[i + 1]; c += kW) {
    const int32_t k = c + lane;
    bool st = false;
    int32_t j = 0;
    if (k < rp[i + 1]) {
      const uint8_t m = mask[k];
      st = (m == 1 || m == 2);
      j = col[k];
    }
    const unsigned long long bm = __ballot(st);
    if (st) {
      const int32_t pos = w + __popcll(bm & ((1ull << lane) - 1ull));
      scol[pos] = j;
      trank[pos] = atomicAdd(&tcnt[j], 1);
    }
    w += __popcll(bm);
  }
}
// Entry-parallel (256 rows per block, an entry's row by binary search in LDS): every entry's
// row goes to its place in its column's list, rp[column] + rank.  VAL: the value too.
template <bool VAL>
__global__ __launch_bounds__(kBlock) void k_scatter_ranked(int32_t n,
                                                           const int32_t *__restrict__ rp,
                                                           const int32_t *__restrict__ col,
                                                           const double *__restrict__ val,
                                                           const int32_t *__restrict__ rank,
                                                           const int32_t *__restrict__ trp,
                                                           int32_t *__restrict__ tcol,
                                                           double *__restrict__ tval) {
  __shared__ int32_t s_rp[kBlock + 1];
  const int t = threadIdx.x;
  const int64_t r0 = (int64_t)blockIdx.x * kBlock;
  const int32_t nr = (int32_t)min<int64_t>(kBlock, (int64_t)n - r0);
  if (t < nr) s_rp[t] = rp[r0 + t];
  if (t == 0) s_rp[nr] = rp[r0 + nr];  // nr can be kBlock: no thread t == nr
  __syncthreads();
  const int32_t e0 = s_rp[0], e1 = s_rp[nr];
  for (int32_t e = e0 + t; e < e1; e += kBlock) {
    int32_t lo = 0, hi = nr - 1;  // the entry's row: the last r with s_rp[r] <= e
    while (lo < hi) {
      const int32_t mid = (lo + hi + 1) >> 1;
      if (s_rp[mid] <= e) lo = mid;
      else hi = mid - 1;
    }
    const int32_t p = trp[col[e]] + rank[e];
    tcol[p] = (int32_t)r0 + lo;
    if (VAL) tval[p] = val[e];
  }
}
__global__ void k_union(int32_t n, const int32_t *arp, const int32_t *acol, const int32_t *brp,
                        const int32_t *bcol, const int32_t *orp, int32_t *ocol, int32_t *ocnt) {
  SA_ROW_KERNEL_BEGIN(n)
  int32_t a = arp[i], ae = arp[i + 1], b = brp[i], be = brp[i + 1];
  int32_t w = orp ? orp[i] : 0;
  int32_t cnt = 0;
  while (a < ae || b < be) {
    int32_t v;
    if (b >= be || (a < ae && acol[a] < bcol[b])) v = acol[a++];
    else if (a >= ae || bcol[b] < acol[a]) v = bcol[b++];
    else {
      v = acol[a++];
      ++b;
    }
    if (ocol) ocol[w + cnt] = v;
    ++cnt;
  }
  if (ocnt) ocnt[i] = cnt;
}

// Levels of at most this many vertices have their roots selected in one workgroup (default of
// SAAMG_MIS_WG_MAX_N).
constexpr int64_t kMisWgMaxN = 4096;

int64_t strength_graph(int32_t n, int64_t nnz_a, const int32_t *rp, const int32_t *col,
                       const uint8_t *mask, const int32_t *scount, bool wave, Arena &ar,
                       int32_t **grp_out, int32_t **gcol_out, int32_t *maxdeg,
                       const ReadAlong &along, hipStream_t s) {
  Arena tmp;
  tmp.stream = s;
  int32_t *srp = tmp.alloc<int32_t>(n + 1);
  exclusive_scan_i32(scount, srp, n, s);
  // S has at most A's entries: no readback of its count
  int32_t *scol = tmp.alloc<int32_t>(nnz_a);
  int32_t *tcnt = tmp.alloc<int32_t>(n + 1);
  fill_i32(tcnt, 0, n + 1, s);
  int32_t *trank = tmp.alloc<int32_t>(nnz_a);
  if (wave) k_fill_strong_w<<<(unsigned)n, kW, 0, s>>>(n, rp, col, mask, srp, scol, tcnt, trank);
  else k_fill_strong<<<grid_for(n), kBlock, 0, s>>>(n, rp, col, mask, srp, scol, tcnt, trank);
  SA_LAUNCH_CHECK();
  int32_t *trp = tmp.alloc<int32_t>(n + 1);
  exclusive_scan_i32(tcnt, trp, n, s);
  int32_t *tcol = tmp.alloc<int32_t>(nnz_a);
  k_scatter_ranked<false><<<grid_for(n), kBlock, 0, s>>>(n, srp, scol, nullptr, trank, trp, tcol,
                                                         nullptr);
  SA_LAUNCH_CHECK();
  RowSort sort;
  sort_rows_begin(n, trp, tcol, nullptr, sort, s);
  constexpr int kAlong = 8;
  int32_t hw[kRowSortWords + kAlong];
  WordRuns runs;
  runs.add(sort.words, kRowSortWords);
  if (along.words > 0) runs.add(along.dev, std::min(along.words, kAlong));
  readback_runs(hw, runs, s);
  if (along.words > 0)
    std::memcpy(along.host, hw + kRowSortWords, 4 * std::min(along.words, kAlong));
  sort_rows_end(sort, hw, s);
  int32_t *gcnt = tmp.alloc<int32_t>(n + 1);
  k_union<<<grid_for(n), kBlock, 0, s>>>(n, srp, scol, trp, tcol, nullptr, nullptr, gcnt);
  SA_LAUNCH_CHECK();
  int32_t *grp = ar.alloc<int32_t>(n + 1);
  exclusive_scan_i32(gcnt, grp, n, s);
  int32_t hg[2] = {0, -1};
  if (n > kMisWgMaxN) {
    int32_t *mx = tmp.alloc<int32_t>(row_max_words(n) + 1);
    row_max(n, grp, mx + 1, mx, s);
    WordRuns last;
    last.add(grp + n, 1);
    last.add(mx, 1);
    readback_runs(hg, last, s);
  } else {
    hg[0] = read1(grp + n, s);
  }
  const int32_t nnzG = hg[0];
  *maxdeg = hg[1];
  int32_t *gcol = ar.alloc<int32_t>(nnzG);
  k_union<<<grid_for(n), kBlock, 0, s>>>(n, srp, scol, trp, tcol, grp, gcol, nullptr);
  SA_LAUNCH_CHECK();
  *grp_out = grp;
  *gcol_out = gcol;
  return nnzG;
}

// ---- root selection: lexicographically-first distance-2 maximal independent set -----------
// In priority order (natural: the index; hashed: a seeded 30-bit hash, ties by index) a vertex
// is a root (IN) when no earlier vertex within distance 2 is one.  A round decides, all at
// once, every undecided vertex whose earlier vertices within distance 2 were all decided in
// earlier rounds: it becomes a root, and the undecided vertices within distance 2 of it
// become OUT.  Both follow from earlier decisions only, so the rounds reproduce the sequential
// greedy choice exactly; at least one vertex (the earliest undecided) is decided per round.
//
// Nothing is re-evaluated until it can change: every undecided vertex watches ONE undecided
// earlier vertex within distance 2, and only when that one is decided does it look over its
// distance-2 ball for another to watch; if there is none, it is a root.  On the 128^3 cube a
// vertex looks 1.1-1.8 times in all and reads ~6 states (the look ends at the first
// undecided earlier vertex), and a round of the 2M-vertex level has ~4,400 looks.  Kernel
// trace of one 128^3 setup: 665 launches of 7-13 us, 6.3 ms (205 of 7.6 us on the 2M-vertex
// level), against 12.5 ms with two neighbourhood-minimum passes per round over byte stamps
// and OUT marks and root decisions in rounds of their own (2 x 410 launches of 4.7 us on that
// level); setup 26.5 -> 20.4 ms.
//
// What bounds a round is the chain of dependent loads: a vertex's state, its watch, that
// one's state, then three of the ball (neighbours with their row ranges, their neighbours,
// those ones' states).  G lanes share a ball (mis_ball).
//
// Visibility on the grid: one launch per round decides and looks at once, so a decision is
// stamped with its round and other vertices take it as undecided until the next launch.  The
// state byte holds 0 undecided, 1 OUT and 2 IN of long ago, and 4 + 2 (r mod 126) + (1 if IN)
// for a decision of round r; every 126 rounds one launch ages all decisions (k_mis_age)
// before their stamps come round again.
//
// The round count reported to the caller counts a root decision and the OUT marks that
// follow from it as a round each, and the round in which nothing is left to decide: with T
// rounds as above it is 2 T - 1, plus 1 if the last of them marked a vertex OUT.
constexpr int kMisStamps = 126;

__device__ inline uint64_t splitmix64_dev(uint64_t seed, uint64_t k) {
  uint64_t z = seed + (k + 1) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
__device__ inline uint64_t stream_key_dev(int stream, int level, int64_t i) {
  return ((uint64_t)stream << 56) | ((uint64_t)level << 40) | (uint64_t)i;
}

// Priority orders.  past(x, v): in a row sorted by index, no entry from x on precedes v.
struct NaturalOrder {
  __device__ int32_t pri(int32_t v) const { return v; }
  __device__ bool before(int32_t x, int32_t pv) const { return x < pv; }
  __device__ bool past(int32_t x, int32_t pv) const { return x >= pv; }
};
struct HashedOrder {
  uint64_t seed;
  int32_t level;
  __device__ uint64_t pri(int32_t v) const {
    return ((splitmix64_dev(seed, stream_key_dev(2, level, v)) >> 34) << 32) | (uint64_t)v;
  }
  __device__ bool before(int32_t x, uint64_t pv) const { return pri(x) < pv; }
  __device__ bool past(int32_t, uint64_t) const { return false; }
};

// Whether other vertices count a state as undecided in the round with stamps c0, c0 | 1.
__device__ __forceinline__ bool mis_open(uint8_t s, uint8_t c0) {
  return s == 0 || (s | 1) == (c0 | 1);
}

template <int G>
__device__ __forceinline__ uint64_t group_ballot(bool p) {
  const uint64_t m = __ballot(p);
  if constexpr (G == 64) return m;
  const int sh = (int)__lane_id() & ~(G - 1);
  return (m >> sh) & ((1ull << (G & 63)) - 1ull);
}

// Row ranges of the strength graph as a look reads them.  On the grid the range of every
// entry's own row is stored beside the entry (gext), which takes a dependent load out of the
// chain; in one workgroup the row pointers are in LDS.
struct EntryRanges {
  const int32_t *__restrict__ gcol;
  const int2 *__restrict__ gext;  // per entry: start and length of that vertex's row
  __device__ void entry(int32_t k, int32_t &u, int32_t &ub, int32_t &ulen) const {
    u = gcol[k];
    const int2 x = gext[k];
    ub = x.x;
    ulen = x.y;
  }
};
struct RowRanges {
  const int32_t *__restrict__ gcol;
  const int32_t *rp;
  __device__ void entry(int32_t k, int32_t &u, int32_t &ub, int32_t &ulen) const {
    u = gcol[k];
    ub = rp[u];
    ulen = rp[u + 1] - ub;
  }
};

// The distance-2 ball of v (row [b, e)) by the G lanes of a group: f(c, last) for eight
// vertices per lane at a time, until it returns true (group-uniform) or the ball is through;
// last: the step that ends the ball.  Lane j takes v's j-th neighbour u (G of them per outer
// step); the lists {u, N[u]} of the lanes are laid end to end and shared out over the lanes,
// so a step's entries are loaded together whatever their rows' lengths.  Positions past the
// end give v itself; a vertex may come more than once.
template <int G, class R, class F>
__device__ __forceinline__ void mis_ball(int32_t v, int32_t b, int32_t e, int j, const R &rows,
                                         F &&f) {
  for (int32_t k0 = b; k0 < e; k0 += G) {  // group-uniform
    int32_t u = v, ub = 0, len = 0;
    if (k0 + j < e) {
      rows.entry(k0 + j, u, ub, len);
      ++len;
    }
    const int32_t end = group_prefix<G>(len, j);  // of the lists' lengths
    const int32_t start = end - len;
    const int32_t total = __shfl(end, G - 1, G);
    for (int32_t p0 = 0; p0 < total; p0 += 8 * G) {  // group-uniform
      int32_t c[8], at[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int32_t p = p0 + i * G + j;
        int s = 0;  // the last list that starts at or before p
#pragma unroll
        for (int step = G / 2; step >= 1; step >>= 1)
          if (__shfl(start, s + step, G) <= p) s += step;
        const int32_t k = p - __shfl(start, s, G);  // 0: u itself, k > 0: entry k - 1
        const int32_t su = __shfl(u, s, G), sb = __shfl(ub, s, G);
        c[i] = p < total ? su : v;
        at[i] = p < total && k > 0 ? sb + k - 1 : -1;
      }
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (at[i] >= 0) c[i] = rows.gcol[at[i]];
      if (f(c, k0 + G >= e && p0 + 8 * G >= total)) return;
    }
  }
}

// A look at v: returns an undecided vertex before it within distance 2 (of those found in the
// same step the one with the largest index, the likeliest to be decided last), or -1 when
// there is none: v is a root then, and its ball's undecided vertices have been marked OUT
// (*out raised if any was).  A ball of one step is marked from the registers that hold it.
template <int G, class R, class O>
__device__ __forceinline__ int32_t mis_look(int32_t v, int32_t b, int32_t e, int j, const R &rows,
                                            uint8_t *st, uint8_t c0, const O &ord, bool *out) {
  const auto pv = ord.pri(v);
  int32_t found = -1;
  bool marked = false;
  auto mark = [&](const int32_t (&c)[8], const uint8_t (&x)[8]) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (x[i] == 0 && c[i] != v) {
        st[c[i]] = c0;
        *out = true;
      }
  };
  int32_t steps = 0;
  mis_ball<G>(v, b, e, j, rows, [&](const int32_t (&c)[8], bool last) {
    uint8_t x[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = st[c[i]];
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (mis_open(x[i], c0) && ord.before(c[i], pv)) found = max(found, c[i]);
    if (group_ballot<G>(found >= 0) != 0) return true;
    if (last && steps == 0) {
      mark(c, x);
      marked = true;
    }
    ++steps;
    return false;
  });
  if (!marked && group_ballot<G>(found >= 0) == 0)
    mis_ball<G>(v, b, e, j, rows, [&](const int32_t (&c)[8], bool) {
      uint8_t x[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) x[i] = st[c[i]];
      mark(c, x);
      return false;
    });
#pragma unroll
  for (int off = G / 2; off >= 1; off >>= 1) found = max(found, __shfl_xor(found, off, G));
  return found;
}

// A vertex without neighbours is decided at once: nothing near it can ever be aggregated, so
// the sequential rule makes it a root whatever its priority (singletons), or it is left out.
// Any other vertex first watches its first earlier neighbour, or (itself as the mark) looks in
// the first round.
template <class O>
__global__ void k_mis_init(int32_t n, const int32_t *__restrict__ grp,
                           const int32_t *__restrict__ gcol, O ord, bool singletons, uint8_t *st,
                           int32_t *watch) {
  SA_ROW_KERNEL_BEGIN(n)
  const int32_t b = grp[i], e = grp[i + 1];
  const auto pv = ord.pri(i);
  int32_t w = i;
  for (int32_t k = b; k < e; ++k) {
    const int32_t u = gcol[k];
    if (ord.before(u, pv)) w = u;
    if (w != i || ord.past(u, pv)) break;
  }
  st[i] = e > b ? 0 : singletons ? 2 : 1;
  watch[i] = w;
}

// Positions for the entries with take[q] of every active lane, counted on from *cnt: one LDS
// atomic per wavefront, slots in lane-major order of the ballots.
template <int Q>
__device__ __forceinline__ void wave_reserve(const bool (&take)[Q], int32_t *cnt,
                                             int32_t (&pos)[Q]) {
  uint32_t total = 0;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const uint64_t m = __ballot(take[q]);
    pos[q] = (int32_t)(total + __builtin_amdgcn_mbcnt_hi(
                                   (uint32_t)(m >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u)));
    total += (uint32_t)__popcll(m);
  }
  if (total == 0) return;  // uniform over the active lanes
  const uint64_t act = __ballot(true);
  int32_t base = 0;
  if ((int)__lane_id() == __ffsll((unsigned long long)act) - 1)
    base = atomicAdd(cnt, (int32_t)total);
  base = __builtin_amdgcn_readfirstlane(base);
#pragma unroll
  for (int q = 0; q < Q; ++q) pos[q] += base;
}

// Vertices per thread from a level size on: fewer workgroups to dispatch per round against
// more looks per workgroup (128^3 setup 20.4 ms, with one vertex per thread on every level
// 20.6 ms, with four from 0 on 21.1 ms; 160^3 39.1 against 40.0 ms).
constexpr int kMisV = 4;
constexpr int64_t kMisVMinN = 524288;

// One round on the grid.  Each thread takes V vertices and reads their states, their watched
// vertices and those vertices' states; the block's vertices whose watched vertex is decided
// go to an LDS list and are looked at by G lanes each.  A block's vertices are runs of kMisRun
// consecutive ones, the grid's block count of runs apart: neighbouring vertices tend to be
// decided together, and their looks are spread over many blocks.
// flags: per round {a root was decided, a vertex was marked OUT}; this launch clears the next
// round's and posts the previous round's to the host word.  A round whose predecessor decided
// nothing exits at once.
constexpr int kMisRun = 16;
template <int G, int V, class O>
__global__ __launch_bounds__(kBlock) void k_mis_round(
    int32_t n, const int32_t *__restrict__ grp, const int32_t *__restrict__ gcol,
    const int2 *__restrict__ gext, uint8_t *st, int32_t *__restrict__ watch, uint8_t c0, O ord,
    const int32_t *prev, int32_t *cur, int32_t *next, uint32_t *hstat, uint32_t tag) {
  __shared__ int32_t lv[kBlock * V], lb[kBlock * V], le[kBlock * V];
  __shared__ int32_t count;
  auto vertex = [&](int q) {
    const int64_t run = (int64_t)(q * (kBlock / kMisRun) + (threadIdx.x / kMisRun)) * gridDim.x +
                        blockIdx.x;
    return run * kMisRun + (threadIdx.x % kMisRun);
  };
  uint8_t s[V];
#pragma unroll
  for (int q = 0; q < V; ++q) {
    const int64_t v = vertex(q);
    s[q] = v < n ? st[v] : (uint8_t)1;
  }
  const bool over = prev && prev[0] == 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    next[0] = 0;
    next[1] = 0;
    if (hstat)
      __hip_atomic_store(hstat, tag | (over ? 2u : prev[1] ? 3u : 1u), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_SYSTEM);
  }
  if (over) return;  // block-uniform
  if (threadIdx.x == 0) count = 0;
  __syncthreads();
  // (a vertex marked OUT by another block in this launch may be listed or not: it is blocked
  // by that root either way)
  int32_t w[V], b[V], e[V], pos[V];
  bool take[V];
#pragma unroll
  for (int q = 0; q < V; ++q) {
    w[q] = -1;
    if (s[q] == 0) {
      const int32_t v = (int32_t)vertex(q);
      w[q] = watch[v];
      b[q] = grp[v];
      e[q] = grp[v + 1];
    }
  }
#pragma unroll
  for (int q = 0; q < V; ++q)
    take[q] = w[q] >= 0 && (w[q] == (int32_t)vertex(q) || !mis_open(st[w[q]], c0));
  wave_reserve<V>(take, &count, pos);
#pragma unroll
  for (int q = 0; q < V; ++q)
    if (take[q]) {
      lv[pos[q]] = (int32_t)vertex(q);
      lb[pos[q]] = b[q];
      le[pos[q]] = e[q];
    }
  __syncthreads();
  const int32_t m = count;
  const EntryRanges rows{gcol, gext};
  auto looks = [&](auto gc) {
    constexpr int L = decltype(gc)::value;
    const int j = threadIdx.x % L;
    for (int32_t i = threadIdx.x / L; i < m; i += kBlock / L) {
      const int32_t v = lv[i];
      bool out = false;
      const int32_t f = mis_look<L>(v, lb[i], le[i], j, rows, st, c0, ord, &out);
      if (j == 0) {
        if (f >= 0) {
          watch[v] = f;
        } else {
          st[v] = c0 | 1;
          cur[0] = 1;
        }
      }
      if (out) cur[1] = 1;
    }
  };
  // up to 4 looks have a wavefront each (fewer steps through a ball)
  if (G == 32 && m <= kBlock / 64) looks(std::integral_constant<int, 64>{});
  else looks(std::integral_constant<int, G>{});
}

// Decisions of earlier rounds lose their stamps (four states per thread).
__global__ void k_mis_age(int32_t nw, uint32_t *st) {
  SA_ROW_KERNEL_BEGIN(nw)
  const uint32_t w = st[i];
  uint32_t o = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t x = (w >> (8 * q)) & 0xffu;
    o |= (x >= 4u ? 1u + (x & 1u) : x) << (8 * q);
  }
  st[i] = o;
}

// ---- root selection in one workgroup --------------------------------------------------------
// On levels of at most kMisWgMaxN vertices all rounds run inside a single workgroup of kMisWg
// threads, with __syncthreads() in place of kernel boundaries; the states, watched vertices and
// row pointers are in LDS, only the neighbour lists are read from memory.  The same polls,
// looks and stamps as on the grid; a round's looks get a wavefront each while they are few,
// else 16 lanes.  result[0] = the reported round count (bit 31: max_rounds reached); the same
// word goes to the host-mapped post.
constexpr int kMisWg = 1024;
// (64^2 grid and 128^3 cube: within 1% of the grid's rounds at this size, with no launches)
constexpr int kMisWgV = 5;            // vertices per thread: levels up to 5120 vertices fit LDS
constexpr int64_t kMisWgLdsMaxN = kMisWgV * kMisWg;

template <class O>
__global__ __launch_bounds__(kMisWg) void k_mis_wg(int32_t n, const int32_t *__restrict__ grp,
                                                   const int32_t *__restrict__ gcol,
                                                   const int32_t *__restrict__ gwatch,
                                                   uint8_t *gst, O ord, int32_t max_rounds,
                                                   int32_t *result, uint32_t *hpost) {
  __shared__ int32_t rp[kMisWgLdsMaxN + 1], watch[kMisWgLdsMaxN];
  __shared__ uint8_t st[kMisWgLdsMaxN];
  __shared__ uint16_t list[kMisWgLdsMaxN];
  __shared__ int32_t count[2], root[2], mark[2];
  const int tid = threadIdx.x;
  for (int32_t i = tid; i < n; i += kMisWg) {
    rp[i] = grp[i];
    watch[i] = gwatch[i];
    st[i] = gst[i];
  }
  if (tid == 0) {
    rp[n] = grp[n];
    count[0] = count[1] = root[0] = root[1] = mark[0] = mark[1] = 0;
  }
  __syncthreads();
  const RowRanges rows{gcol, rp};
  int32_t T = 0;  // rounds that decided something
  bool out_last = false, err = false;
  for (int32_t r = 0;; ++r) {  // workgroup-uniform
    const uint8_t c0 = (uint8_t)(4 + 2 * (r % kMisStamps));
    const int h = r & 1;  // this round's counters; the other round's are cleared in this one
    if (r > 0 && r % kMisStamps == 0) {
      for (int32_t i = tid; i < n; i += kMisWg)
        if (st[i] >= 4) st[i] = 1 + (st[i] & 1);
      __syncthreads();
    }
    bool take[kMisWgV];
    int32_t pos[kMisWgV];
#pragma unroll
    for (int q = 0; q < kMisWgV; ++q) {
      const int32_t v = q * kMisWg + tid;
      take[q] = false;
      if (v < n && st[v] == 0) {
        const int32_t w = watch[v];
        take[q] = w == v || !mis_open(st[w], c0);
      }
    }
    wave_reserve<kMisWgV>(take, &count[h], pos);
#pragma unroll
    for (int q = 0; q < kMisWgV; ++q)
      if (take[q]) list[pos[q]] = (uint16_t)(q * kMisWg + tid);
    __syncthreads();
    const int32_t m = count[h];
    if (tid == 0) count[h ^ 1] = root[h ^ 1] = mark[h ^ 1] = 0;
    auto looks = [&](auto gc) {
      constexpr int G = decltype(gc)::value;
      const int j = tid % G;
      for (int32_t i = tid / G; i < m; i += kMisWg / G) {
        const int32_t v = list[i];
        bool out = false;
        const int32_t f = mis_look<G>(v, rp[v], rp[v + 1], j, rows, st, c0, ord, &out);
        if (j == 0) {
          if (f >= 0) {
            watch[v] = f;
          } else {
            st[v] = c0 | 1;
            root[h] = 1;
          }
        }
        if (out) mark[h] = 1;
      }
    };
    if (m <= 2 * (kMisWg / 64)) looks(std::integral_constant<int, 64>{});
    else looks(std::integral_constant<int, 16>{});
    __syncthreads();
    if (root[h] == 0) break;
    ++T;
    out_last = mark[h] != 0;
    if (r >= max_rounds) {
      err = true;
      break;
    }
  }
  for (int32_t i = tid; i < n; i += kMisWg) gst[i] = st[i];
  if (tid == 0) {
    const uint32_t used = T > 0 ? 2u * (uint32_t)T - 1u + (out_last ? 1u : 0u) : 0u;
    const uint32_t word = used | (err ? 1u << 31 : 0u);
    result[0] = (int32_t)word;
    if (hpost)
      __hip_atomic_store(hpost, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// Beside each entry of the graph the start and length of that vertex's own row.
__global__ void k_mis_ranges(int64_t nnz, const int32_t *__restrict__ grp,
                             const int32_t *__restrict__ gcol, int2 *gext) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nnz) return;
  const int32_t u = gcol[k];
  const int32_t b = grp[u];
  gext[k] = make_int2(b, grp[u + 1] - b);
}

// Largest row length of a CSR (two-stage maximum, no contended atomics).
__global__ void k_rowlen_max_stage(int32_t n, const int32_t *rp, int32_t *part) {
  __shared__ int32_t sh[kBlock];
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  sh[threadIdx.x] = (i < n) ? rp[i + 1] - rp[i] : 0;
  __syncthreads();
  for (int w = kBlock / 2; w >= 1; w >>= 1) {
    if ((int)threadIdx.x < w) sh[threadIdx.x] = max(sh[threadIdx.x], sh[threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}
__global__ void k_max_i32(int32_t n, const int32_t *a, int32_t *out) {
  __shared__ int32_t sh[kBlock];
  int32_t m = 0;
  for (int32_t i = threadIdx.x; i < n; i += blockDim.x) m = max(m, a[i]);
  sh[threadIdx.x] = m;
  __syncthreads();
  for (int w = kBlock / 2; w >= 1; w >>= 1) {
    if ((int)threadIdx.x < w) sh[threadIdx.x] = max(sh[threadIdx.x], sh[threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = sh[0];
}
int32_t row_max_words(int32_t n) { return n > 0 ? (int32_t)grid_for(n) : 0; }
void row_max(int32_t n, const int32_t *rp, int32_t *part, int32_t *out, hipStream_t s) {
  const unsigned nb = grid_for(n);
  k_rowlen_max_stage<<<nb, kBlock, 0, s>>>(n, rp, part);
  k_max_i32<<<1, kBlock, 0, s>>>((int32_t)nb, part, out);
  SA_LAUNCH_CHECK();
}
int32_t max_row_length(int32_t n, const int32_t *rp, hipStream_t s) {
  if (n <= 0) return 0;
  const int32_t nb = row_max_words(n);
  int32_t *part = (int32_t *)dev_alloc(sizeof(int32_t) * (nb + 1), s);
  row_max(n, rp, part, part + nb, s);
  const int32_t m = read1(part + nb, s);
  dev_free(part, s);
  return m;
}

// IN states: 2, or a stamp with its lowest bit set.
__device__ __forceinline__ bool mis_in(uint8_t s) { return s == 2 || (s >= 4 && (s & 1) != 0); }

__global__ void k_roots(int32_t n, const uint8_t *st, int32_t *isr) {
  SA_ROW_KERNEL_BEGIN(n)
  isr[i] = mis_in(st[i]) ? 1 : 0;
}
__global__ void k_agg_phase1(int32_t n, const int32_t *grp, const int32_t *gcol,
                             const uint8_t *st,
                             const int32_t *rid, int32_t *agg1, uint8_t *is_root,
                             int32_t *root_vertex) {
  SA_ROW_KERNEL_BEGIN(n)
  int32_t a = -1;
  const bool root = mis_in(st[i]);
  if (root) {
    a = rid[i];
    root_vertex[a] = i;
  } else {
    for (int32_t k = grp[i]; k < grp[i + 1]; ++k) {
      const int32_t u = gcol[k];
      if (mis_in(st[u])) {
        a = rid[u];
        break;
      }
    }
  }
  agg1[i] = a;
  is_root[i] = root ? 1 : 0;
}
// Leftover vertices join the phase-1 aggregate with the most strong connections to them,
// ties to the smaller aggregate number (a total order on the candidates: the choice does not
// depend on the order they are looked at in).
// Rows of up to R entries: the neighbours' phase-1 aggregates are loaded once, in one batch
// (-1 past the end of the row), and counted in registers.
template <int R>
__device__ __forceinline__ int32_t agg_join_regs(int32_t b, int32_t e,
                                                 const int32_t *__restrict__ gcol,
                                                 const int32_t *__restrict__ agg1) {
  int32_t g[R], c[R];
#pragma unroll
  for (int q = 0; q < R; ++q) g[q] = gcol[min(b + q, e - 1)];
#pragma unroll
  for (int q = 0; q < R; ++q) c[q] = (b + q < e) ? agg1[g[q]] : -1;
  int32_t best = -1, bestc = 0;
#pragma unroll
  for (int k = 0; k < R; ++k) {
    if (c[k] < 0) continue;
    int32_t cnt = 0;
#pragma unroll
    for (int q = 0; q < R; ++q) cnt += (c[q] == c[k]);
    if (cnt > bestc || (cnt == bestc && c[k] < best)) {
      best = c[k];
      bestc = cnt;
    }
  }
  return best;
}

// Rows of more than 32 neighbours are left to k_agg_phase2_w (wide).
__global__ void k_agg_phase2(int32_t n, const int32_t *grp, const int32_t *gcol,
                             const int32_t *agg1, int32_t *agg) {
  SA_ROW_KERNEL_BEGIN(n)
  int32_t a = agg1[i];
  const int32_t b = grp[i], e = grp[i + 1];
  if (a < 0 && e > b) {
    if (e - b > 32) return;
    a = e - b <= 8 ? agg_join_regs<8>(b, e, gcol, agg1) : agg_join_regs<32>(b, e, gcol, agg1);
  }
  agg[i] = a;
}
// A wavefront per vertex: its neighbours' aggregates 64 at a time against 64 at a time of the
// same row, through the lanes, so a vertex of d neighbours costs d^2 / 64 steps of one
// instruction each (a thread per vertex: 1,600 vertices of up to 600 neighbours 114 us, now
// 14 for the pass over the others and 4).
__global__ __launch_bounds__(kBlock) void k_agg_phase2_w(int32_t n,
                                                         const int32_t *__restrict__ grp,
                                                         const int32_t *__restrict__ gcol,
                                                         const int32_t *__restrict__ agg1,
                                                         int32_t *__restrict__ agg) {
  const int lane = threadIdx.x & 63;
  for (int64_t i = first_row<64>(); i < n; i += row_stride<64>()) {  // wave-uniform
    const int32_t b = grp[i], e = grp[i + 1];
    if (e - b <= 32 || agg1[i] >= 0) continue;
    int32_t best = INT_MAX, bestc = 0;
    for (int32_t k0 = b; k0 < e; k0 += 64) {
      const int32_t c = k0 + lane < e ? agg1[gcol[k0 + lane]] : -1;
      int32_t cnt = 0;
      for (int32_t q0 = b; q0 < e; q0 += 64) {
        const int32_t o = q0 + lane < e ? agg1[gcol[q0 + lane]] : -1;
        const int32_t len = min(64, e - q0);
        for (int32_t l = 0; l < len; ++l)
          cnt += __builtin_amdgcn_readlane(o, l) == c ? 1 : 0;
      }
      if (c >= 0 && (cnt > bestc || (cnt == bestc && c < best))) {
        best = c;
        bestc = cnt;
      }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      const int32_t oc = __shfl_xor(bestc, off, 64), ob = __shfl_xor(best, off, 64);
      if (oc > bestc || (oc == bestc && ob < best)) {
        best = ob;
        bestc = oc;
      }
    }
    if (lane == 0) agg[i] = bestc > 0 ? best : -1;
  }
}

template <class O>
static int32_t aggregate_impl(int32_t n, int64_t nnzG, const int32_t *grp, const int32_t *gcol,
                              int32_t maxdeg, O ord, bool singletons, int32_t *agg,
                              uint8_t *is_root, Arena &ar, int32_t **root_vertex,
                              int32_t *rounds_out, hipStream_t s) {
  Arena tmp;
  tmp.stream = s;
  uint8_t *st = tmp.alloc<uint8_t>(((int64_t)n + 15) & ~(int64_t)15);  // padded for word reads
  int32_t *watch = tmp.alloc<int32_t>(n);
  // levels up to wg_max_n vertices run every round in one workgroup
  int64_t wg_max_n = kMisWgMaxN;
  if (const char *e = std::getenv("SAAMG_MIS_WG_MAX_N")) wg_max_n = std::atoll(e);
  const bool one_wg = nnzG > 0 && n <= std::min(wg_max_n, kMisWgLdsMaxN);
  k_mis_init<O><<<grid_for(n), kBlock, 0, s>>>(n, grp, gcol, ord, singletons, st, watch);
  SA_LAUNCH_CHECK();
  // Rounds are launched back to back, at most kAhead past the last round whose outcome the
  // host has seen.  The launch of round r+1 posts round r's outcome into a pinned status ring
  // (slot r mod kRing, tagged with r); the first round that decided nothing ends the
  // selection, and the rounds still queued behind it exit at once.  Device flags live in a
  // ring of the same size: round r clears slot r+1 and raises slot r.  If a status
  // word is not seen within spin_ns (20 ms; the environment variable SAAMG_STATUS_SPIN_NS
  // overrides it, 0 taking the fallback at every wait), the stream is synchronised and the
  // device flags read instead, so the outcome never depends on the host mapping alone.
  constexpr int kRing = 256, kAhead = 6;
  int64_t spin_ns = 20000000;
  if (const char *e = std::getenv("SAAMG_STATUS_SPIN_NS")) spin_ns = std::atoll(e);
  // every round before the last decides at least one vertex, so this bound is never reached
  const int64_t cap = (int64_t)n + 2 + 2 * kAhead;
  int32_t *flags = tmp.alloc<int32_t>(2 * kRing);
  fill_i32(flags, 0, 2 * kRing, s);
  volatile uint32_t *hs = (volatile uint32_t *)pinned_status(sizeof(uint32_t) * kRing);
  for (int q = 0; q < kRing; ++q) hs[q] = ~0u;
  uint32_t *hs_dev = nullptr;
  SA_HIP(hipHostGetDevicePointer((void **)&hs_dev, (void *)hs, 0));
  // lanes per look: the longest row's neighbours in one step where 64 lanes hold them.  8 on
  // every level took the 128^3 setup from 20.7 to 25.3 ms; 64 on every level but those of
  // rows up to 8 took the 100^3 27-point cube's from 17.8 to 19.2 ms
  if (!one_wg && maxdeg < 0) maxdeg = max_row_length(n, grp, s);
  int2 *gext = nullptr;
  if (!one_wg && nnzG > 0) {
    gext = tmp.alloc<int2>(nnzG);
    k_mis_ranges<<<grid_for(nnzG), kBlock, 0, s>>>(nnzG, grp, gcol, gext);
    SA_LAUNCH_CHECK();
  }
  // large levels: kMisV vertices per thread, fewer workgroups to dispatch per round;
  // SAAMG_MIS_V_MIN_N overrides the level size from which they are used
  int64_t v_min_n = kMisVMinN;
  if (const char *e = std::getenv("SAAMG_MIS_V_MIN_N")) v_min_n = std::atoll(e);
  const bool many = n >= v_min_n;
  const unsigned g = grid_for(n, many ? kBlock * kMisV : kBlock);
  auto launch_round = [&](int64_t r) {
    const uint8_t c0 = (uint8_t)(4 + 2 * (r % kMisStamps));
    if (r > 0 && r % kMisStamps == 0) {
      const int32_t nw = (int32_t)ceil_div(n, 4);
      k_mis_age<<<grid_for(nw), kBlock, 0, s>>>(nw, (uint32_t *)st);
    }
    const bool first = r == 0;
    const int32_t *prev = first ? nullptr : flags + 2 * ((r - 1) & (kRing - 1));
    int32_t *cur = flags + 2 * (r & (kRing - 1));
    int32_t *next = flags + 2 * ((r + 1) & (kRing - 1));
    uint32_t *post = first ? nullptr : hs_dev + ((r - 1) & (kRing - 1));
    const uint32_t tag = (uint32_t)(r - 1) << 2;
    auto go = [&](auto gc, auto vc) {
      constexpr int G = decltype(gc)::value, V = decltype(vc)::value;
      k_mis_round<G, V, O><<<g, kBlock, 0, s>>>(n, grp, gcol, gext, st, watch, c0, ord, prev,
                                                cur, next, post, tag);
    };
    using I1 = std::integral_constant<int, 1>;
    using IV = std::integral_constant<int, kMisV>;
    auto lanes = [&](auto gc) {
      if (many) go(gc, IV{});
      else go(gc, I1{});
    };
    if (maxdeg <= 8) lanes(std::integral_constant<int, 8>{});
    else if (maxdeg <= 32) lanes(std::integral_constant<int, 32>{});
    else lanes(std::integral_constant<int, 64>{});
    SA_LAUNCH_CHECK();
  };
  int64_t launched = 0, seen = 0;  // rounds launched; rounds whose outcome is known
  bool out_last = false;           // the last round seen marked a vertex OUT
  int32_t used = 0;
  auto finish_at = [&](int64_t r) {  // round r decided nothing
    used = r > 0 ? (int32_t)(2 * r - 1 + (out_last ? 1 : 0)) : 0;
  };
  bool done = nnzG == 0;
  int32_t *wg_result = nullptr;
  if (one_wg) {
    wg_result = tmp.alloc<int32_t>(1);
    const int32_t max_rounds = n + 2;
    k_mis_wg<O><<<1, kMisWg, 0, s>>>(n, grp, gcol, watch, st, ord, max_rounds, wg_result, hs_dev);
    SA_LAUNCH_CHECK();
    done = true;
  }
  auto wait_from = std::chrono::steady_clock::now();
  while (!done) {
    // round `seen`'s status is posted by the launch of round seen+1
    if (launched >= seen + 2) {
      const uint32_t v = hs[seen & (kRing - 1)];
      if ((v & ~3u) == ((uint32_t)seen << 2) && (v & 3u) != 0 && v != ~0u) {
        if ((v & 3u) == 2u) {
          finish_at(seen);
          done = true;
        } else {
          out_last = (v & 3u) == 3u;
          ++seen;
        }
        wait_from = std::chrono::steady_clock::now();
        continue;
      }
    }
    if (launched < seen + kAhead) {
      if (launched >= cap) throw Error(SA_ERR_COARSEN_STALLED, "root selection did not end");
      launch_round(launched++);
      continue;
    }
    if (beside_step()) continue;
    const auto now = std::chrono::steady_clock::now();
    if (std::chrono::duration_cast<std::chrono::nanoseconds>(now - wait_from).count() <
        spin_ns)
      continue;
    // status not seen in time: every launched round's flags are final when the readback's
    // copy runs (after them on the stream)
    int32_t hf[2 * kRing];
    readback(hf, flags, sizeof(hf), s);
    for (; seen < launched && !done; ++seen) {
      const int32_t *f = hf + 2 * (seen & (kRing - 1));
      if (f[0] == 0) {
        finish_at(seen);
        done = true;
      } else {
        out_last = f[1] != 0;
      }
    }
    if (done) break;
    wait_from = std::chrono::steady_clock::now();
  }
  int32_t *isr = tmp.alloc<int32_t>(n + 1);
  k_roots<<<grid_for(n), kBlock, 0, s>>>(n, st, isr);
  SA_LAUNCH_CHECK();
  int32_t *rid = tmp.alloc<int32_t>(n + 1);
  exclusive_scan_i32(isr, rid, n, s);
  const int32_t nc = read1(rid + n, s);  // returns once the stream's work so far is done
  if (one_wg) {
    // the workgroup's outcome, posted to the host-mapped word (read back if it is not seen)
    uint32_t v = hs[0];
    if (v == ~0u) v = (uint32_t)read1(wg_result, s);
    if (v >> 31) throw Error(SA_ERR_COARSEN_STALLED, "root selection did not end");
    used = (int32_t)v;
  }
  if (rounds_out) *rounds_out = used;
  int32_t *rv = ar.alloc<int32_t>(nc > 0 ? nc : 1);
  int32_t *agg1 = tmp.alloc<int32_t>(n);
  k_agg_phase1<<<grid_for(n), kBlock, 0, s>>>(n, grp, gcol, st, rid, agg1, is_root, rv);
  SA_LAUNCH_CHECK();
  k_agg_phase2<<<grid_for(n), kBlock, 0, s>>>(n, grp, gcol, agg1, agg);
  if (maxdeg > 32 || maxdeg < 0)
    k_agg_phase2_w<<<grid_rows(n, 64), kBlock, 0, s>>>(n, grp, gcol, agg1, agg);
  SA_LAUNCH_CHECK();
  *root_vertex = rv;
  return nc;
}

int32_t aggregate(int32_t n, int64_t nnzG, const int32_t *grp, const int32_t *gcol,
                  int32_t maxdeg, int32_t order, uint64_t seed, int32_t level, bool singletons,
                  int32_t *agg, uint8_t *is_root, Arena &ar, int32_t **root_vertex, int32_t *rounds,
                  hipStream_t s) {
  if (order == 0)
    return aggregate_impl(n, nnzG, grp, gcol, maxdeg, NaturalOrder{}, singletons, agg, is_root, ar,
                          root_vertex, rounds, s);
  return aggregate_impl(n, nnzG, grp, gcol, maxdeg, HashedOrder{seed, level}, singletons, agg,
                        is_root, ar, root_vertex, rounds, s);
}

// ---- Sprsfy (Sec. 2.5) --------------------------------------------------------------------
constexpr int32_t kSprsfyShort = 32;   // root rows up to this length: one thread per aggregate
constexpr int32_t kSprsfyLds = 4096;   // longer root rows (up to this): one block per aggregate
// ... unless the non-root members' rows hold more than this many entries in all: a thread
// scans them once per candidate, so such aggregates also take the block path
constexpr int32_t kSprsfyMemberWork = 128;
constexpr int32_t kSprsfySmall = 64;   // block path with LDS for root rows up to this length
// One thread per aggregate J with root r.  Candidates: aggregates reached by r's weak
// connections but by none of its strong ones, J excluded.  For a candidate c, a single strong
// connection from a non-root member of J into c is dropped with its transpose.  Decisions read
// "strong" as mask 1 or 2, so concurrent drops by other aggregates do not change them; the
// result depends neither on member order nor on the order in which aggregates are taken.
// Aggregates with a long root row or heavy members are listed for k_sprsfy_block: those with
// root rows up to kSprsfySmall in heavy[0, nc) (count nheavy[0]), those up to kSprsfyLds in
// heavy[nc, 2nc) (count nheavy[1]), longer ones for k_sprsfy_long in heavy[2nc, 3nc) (count
// nheavy[2]).
__global__ void k_sprsfy(int32_t nc, const int32_t *rp, const int32_t *col, uint8_t *mask,
                         const int32_t *agg, const int32_t *root_vertex, const int32_t *mrp,
                         const int32_t *mem, int32_t *heavy, int32_t *nheavy) {
  const int64_t J64 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (J64 >= nc) return;
  const int32_t J = (int32_t)J64;
  const int32_t r = root_vertex[J];
  const int32_t rb = rp[r], re = rp[r + 1];
  bool long_row = re - rb > kSprsfyShort;
  int32_t w = 0;  // entries in the non-root members' rows
  for (int32_t m = mrp[J]; m < mrp[J + 1] && !long_row; ++m) {
    const int32_t v = mem[m];
    if (v != r) w += rp[v + 1] - rp[v];
  }
  if (long_row || w > kSprsfyMemberWork) {
    // root rows up to kSprsfySmall: the small-LDS list; up to kSprsfyLds: the second list;
    // longer ones: the third
    const int which = re - rb > kSprsfyLds ? 2 : re - rb > kSprsfySmall ? 1 : 0;
    heavy[which * (int64_t)nc + atomicAdd(nheavy + which, 1)] = J;
    return;
  }
  for (int32_t k = rb; k < re; ++k) {
    const int32_t u0 = col[k];
    if (u0 == r || mask[k] != 0) continue;  // weak connections of the root only
    const int32_t c = agg[u0];
    if (c < 0 || c == J) continue;
    bool first = true, strong_reached = false;
    for (int32_t q = rb; q < re; ++q) {
      const int32_t uq = col[q];
      if (uq == r || agg[uq] != c) continue;
      const uint8_t mq = mask[q];
      if (mq == 1 || mq == 2) strong_reached = true;
      else if (q < k) first = false;  // an earlier weak connection already reached c
    }
    if (!first || strong_reached) continue;
    // count strong connections from non-root members of J into c
    int32_t count = 0, ev = -1, vv = -1;
    for (int32_t m = mrp[J]; m < mrp[J + 1] && count < 2; ++m) {
      const int32_t v = mem[m];
      if (v == r) continue;
      for (int32_t q = rp[v]; q < rp[v + 1]; ++q) {
        const int32_t u = col[q];
        if (u == v) continue;
        const uint8_t mq = mask[q];
        if ((mq == 1 || mq == 2) && agg[u] == c) {
          ++count;
          ev = q;
          vv = v;
        }
      }
    }
    if (count != 1) continue;
    mask[ev] = 2;
    const int32_t u = col[ev];
    int32_t lo = rp[u], hi = rp[u + 1] - 1;
    while (lo <= hi) {
      const int32_t mid = (lo + hi) >> 1;
      const int32_t cm = col[mid];
      if (cm == vv) {
        if (mask[mid] == 1) mask[mid] = 2;
        break;
      }
      if (cm < vv) lo = mid + 1;
      else hi = mid - 1;
    }
  }
}

// The aggregates k_sprsfy lists (a long root row or heavy members), one block each: the root
// row's (aggregate, strong) pairs are sorted in LDS; a candidate is an aggregate reached only
// through weak entries (not J, not unaggregated).  Strong entries of the non-root members are
// counted per candidate (binary search in the sorted candidate list); a count of 1 drops that
// entry and its transpose.  Same decisions as k_sprsfy.
__device__ inline void bitonic_u64_blk(uint64_t *a, int32_t L) {
  for (int32_t k = 2; k <= L; k <<= 1) {
    for (int32_t j = k >> 1; j > 0; j >>= 1) {
      for (int32_t idx = threadIdx.x; idx < L; idx += blockDim.x) {
        const int32_t ixj = idx ^ j;
        if (ixj > idx) {
          const uint64_t x = a[idx], y = a[ixj];
          const bool up = (idx & k) == 0;
          if ((x > y) == up) {
            a[idx] = y;
            a[ixj] = x;
          }
        }
      }
      __syncthreads();
    }
  }
}
template <int CAP>
__global__ __launch_bounds__(kBlock) void k_sprsfy_block(const int32_t *heavy,
                                                         const int32_t *rp,
                                                         const int32_t *col, uint8_t *mask,
                                                         const int32_t *agg,
                                                         const int32_t *root_vertex,
                                                         const int32_t *mrp,
                                                         const int32_t *mem) {
  __shared__ uint64_t pairs[CAP];
  __shared__ int32_t cand[CAP];
  __shared__ int32_t cnt[CAP];
  __shared__ int32_t edge[CAP];
  __shared__ int32_t s_nc;
  const int32_t J = heavy[blockIdx.x];
  const int32_t r = root_vertex[J];
  const int32_t rb = rp[r], re = rp[r + 1];
  const int32_t len = re - rb;
  if (len > CAP) return;  // never: k_sprsfy lists longer root rows for k_sprsfy_long
  int32_t L = 1;
  while (L < len) L <<= 1;
  // key = (aggregate + 1) << 1 | strong ; entries that cannot be candidates sort first as 0
  for (int32_t q = threadIdx.x; q < L; q += blockDim.x) {
    uint64_t key = ~0ull;
    if (q < len) {
      const int32_t k = rb + q;
      const int32_t u = col[k];
      const int32_t c = (u == r) ? -1 : agg[u];
      const uint8_t m = mask[k];
      const bool strong = (m == 1 || m == 2);
      key = (c < 0) ? 0ull : (((uint64_t)(c + 1) << 1) | (strong ? 1u : 0u));
    }
    pairs[q] = key;
  }
  if (threadIdx.x == 0) s_nc = 0;
  __syncthreads();
  bitonic_u64_blk(pairs, L);
  // run heads: first entry of each aggregate; candidate if no strong entry in its run
  for (int32_t q = threadIdx.x; q < len; q += blockDim.x) {
    const uint64_t x = pairs[q];
    if (x == 0ull || x == ~0ull) continue;
    const int32_t c = (int32_t)(x >> 1) - 1;
    const bool head = q == 0 || (pairs[q - 1] >> 1) != (x >> 1);
    if (!head) continue;
    int32_t t = q;
    bool strong = false;
    while (t < len && (pairs[t] >> 1) == (x >> 1)) strong |= (pairs[t++] & 1) != 0;
    if (!strong && c != J) {
      const int32_t slot = atomicAdd(&s_nc, 1);
      cand[slot] = c;
    }
  }
  __syncthreads();
  const int32_t ncand = s_nc;
  if (ncand == 0) return;  // block-uniform
  // sort the candidate list (small) for binary search
  for (int32_t q = threadIdx.x; q < L; q += blockDim.x)
    pairs[q] = q < ncand ? (uint64_t)(uint32_t)cand[q] : ~0ull;
  __syncthreads();
  bitonic_u64_blk(pairs, L);
  for (int32_t q = threadIdx.x; q < ncand; q += blockDim.x) {
    cand[q] = (int32_t)pairs[q];
    cnt[q] = 0;
    edge[q] = -1;
  }
  __syncthreads();
  // one wavefront per member (4 members at a time), lanes over the member's row
  for (int32_t mm = mrp[J] + (int32_t)(threadIdx.x >> 6); mm < mrp[J + 1]; mm += kBlock / 64) {
    const int32_t v = mem[mm];
    if (v == r) continue;
    for (int32_t k = rp[v] + (int32_t)(threadIdx.x & 63); k < rp[v + 1]; k += 64) {
      const int32_t u = col[k];
      if (u == v) continue;
      const uint8_t m = mask[k];
      if (!(m == 1 || m == 2)) continue;
      const int32_t c = agg[u];
      if (c < 0) continue;
      int32_t lo = 0, hi = ncand - 1;
      while (lo <= hi) {
        const int32_t mid = (lo + hi) >> 1;
        if (cand[mid] == c) {
          atomicAdd(&cnt[mid], 1);
          edge[mid] = k;
          break;
        }
        if (cand[mid] < c) lo = mid + 1;
        else hi = mid - 1;
      }
    }
  }
  __syncthreads();
  for (int32_t q = threadIdx.x; q < ncand; q += blockDim.x) {
    if (cnt[q] != 1) continue;
    const int32_t ev = edge[q];
    mask[ev] = 2;
    const int32_t u = col[ev];
    // the row holding ev: search the members for the one whose row range contains it
    int32_t vv = -1;
    for (int32_t mm = mrp[J]; mm < mrp[J + 1]; ++mm) {
      const int32_t v = mem[mm];
      if (ev >= rp[v] && ev < rp[v + 1]) {
        vv = v;
        break;
      }
    }
    int32_t lo = rp[u], hi = rp[u + 1] - 1;
    while (lo <= hi) {
      const int32_t mid = (lo + hi) >> 1;
      const int32_t cm = col[mid];
      if (cm == vv) {
        if (mask[mid] == 1) mask[mid] = 2;
        break;
      }
      if (cm < vv) lo = mid + 1;
      else hi = mid - 1;
    }
  }
}

// Aggregates whose root row is longer than kSprsfyLds, one block each: k_sprsfy's decisions
// from global memory, the root row's entries shared out over the block's threads.  The thread
// holding a candidate's first weak entry decides that candidate (the others skip it as not
// first), so each candidate is decided once, as in k_sprsfy, for any row length.
__global__ __launch_bounds__(kBlock) void k_sprsfy_long(const int32_t *list, const int32_t *rp,
                                                        const int32_t *col, uint8_t *mask,
                                                        const int32_t *agg,
                                                        const int32_t *root_vertex,
                                                        const int32_t *mrp,
                                                        const int32_t *mem) {
  const int32_t J = list[blockIdx.x];
  const int32_t r = root_vertex[J];
  const int32_t rb = rp[r], re = rp[r + 1];
  for (int32_t k = rb + (int32_t)threadIdx.x; k < re; k += blockDim.x) {
    const int32_t u0 = col[k];
    if (u0 == r || mask[k] != 0) continue;  // weak connections of the root only
    const int32_t c = agg[u0];
    if (c < 0 || c == J) continue;
    bool first = true, strong_reached = false;
    for (int32_t q = rb; q < re && first && !strong_reached; ++q) {
      const int32_t uq = col[q];
      if (uq == r || agg[uq] != c) continue;
      const uint8_t mq = mask[q];
      if (mq == 1 || mq == 2) strong_reached = true;
      else if (q < k) first = false;  // an earlier weak connection already reached c
    }
    if (!first || strong_reached) continue;
    int32_t count = 0, ev = -1, vv = -1;
    for (int32_t m = mrp[J]; m < mrp[J + 1] && count < 2; ++m) {
      const int32_t v = mem[m];
      if (v == r) continue;
      for (int32_t q = rp[v]; q < rp[v + 1]; ++q) {
        const int32_t u = col[q];
        if (u == v) continue;
        const uint8_t mq = mask[q];
        if ((mq == 1 || mq == 2) && agg[u] == c) {
          ++count;
          ev = q;
          vv = v;
        }
      }
    }
    if (count != 1) continue;
    mask[ev] = 2;
    const int32_t u = col[ev];
    int32_t lo = rp[u], hi = rp[u + 1] - 1;
    while (lo <= hi) {
      const int32_t mid = (lo + hi) >> 1;
      const int32_t cm = col[mid];
      if (cm == vv) {
        if (mask[mid] == 1) mask[mid] = 2;
        break;
      }
      if (cm < vv) lo = mid + 1;
      else hi = mid - 1;
    }
  }
}

void sprsfy(int32_t n, const int32_t *rp, const int32_t *col, uint8_t *mask, const int32_t *agg,
            const int32_t *root_vertex, int32_t nc, hipStream_t s) {
  if (nc <= 0) return;
  Arena tmp;
  tmp.stream = s;
  int32_t *mrp, *mem;
  member_lists(n, agg, nc, false, tmp, &mrp, &mem, s);  // decisions ignore member order
  // words: heavy aggregates with root rows [0] up to kSprsfySmall, [1] up to kSprsfyLds,
  // [2] longer; heavy holds the three lists at offsets 0, nc and 2 nc
  int32_t *words = tmp.alloc<int32_t>(3);
  int32_t *heavy = tmp.alloc<int32_t>(3 * (int64_t)nc);
  fill_i32(words, 0, 3, s);
  k_sprsfy<<<grid_for(nc), kBlock, 0, s>>>(nc, rp, col, mask, agg, root_vertex, mrp, mem,
                                           heavy, words);
  SA_LAUNCH_CHECK();
  int32_t nh[3];
  readback(nh, words, sizeof(nh), s);
  if (nh[0] > 0)
    k_sprsfy_block<kSprsfySmall><<<(unsigned)nh[0], kBlock, 0, s>>>(
        heavy, rp, col, mask, agg, root_vertex, mrp, mem);
  if (nh[1] > 0)
    k_sprsfy_block<kSprsfyLds><<<(unsigned)nh[1], kBlock, 0, s>>>(
        heavy + nc, rp, col, mask, agg, root_vertex, mrp, mem);
  if (nh[2] > 0)
    k_sprsfy_long<<<(unsigned)nh[2], kBlock, 0, s>>>(heavy + 2 * (int64_t)nc, rp, col, mask,
                                                     agg, root_vertex, mrp, mem);
  SA_LAUNCH_CHECK();
}

// ---- filtered matrix (Sec. 1.1 plain lumping; Sec. 2.3 Algorithm 2) and its diagonal -----
// Kept entries per row (the diagonal and the strong entries), entry-parallel like k_strength.
__global__ __launch_bounds__(kBlock) void k_lump_count(int32_t n, const int32_t *__restrict__ rp,
                                                       const int32_t *__restrict__ col,
                                                       const uint8_t *__restrict__ mask,
                                                       int32_t *__restrict__ cnt) {
  __shared__ int32_t s_rp[kBlock + 1];
  __shared__ int32_t s_cnt[kBlock];
  const int t = threadIdx.x;
  const int64_t r0 = (int64_t)blockIdx.x * kBlock;
  const int32_t nr = (int32_t)min<int64_t>(kBlock, (int64_t)n - r0);
  if (t < nr) s_rp[t] = rp[r0 + t];
  if (t == 0) s_rp[nr] = rp[r0 + nr];  // nr can be kBlock: no thread t == nr
  s_cnt[t] = 0;
  __syncthreads();
  const int32_t e0 = s_rp[0], e1 = s_rp[nr];
  for (int32_t e = e0 + t; e < e1; e += kBlock) {
    const uint8_t m = mask[e];
    if (m == 1 || m == 3) {  // strong, or the diagonal
      int32_t lo = 0, hi = nr - 1;
      while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (s_rp[mid] <= e) lo = mid;
        else hi = mid - 1;
      }
      atomicAdd(&s_cnt[lo], 1);
    }
  }
  __syncthreads();
  if (t < nr) cnt[r0 + t] = s_cnt[t];
}

// One row of the filtered matrix and its smoothing diagonal.  A's row i is read at
// col/val/mask[k - ko] for k in [b, e); the filtered row is written at acol/aval[w - wo] for
// w from o (its row pointer) on -- global arrays (offsets 0), or the same LDS copy of the row,
// whose kept entries move to its front (eight entries are read before any of them is written).
__device__ __forceinline__ void lump_row(int32_t i, int32_t b, int32_t e, const int32_t *col,
                                         const double *val, const uint8_t *mask, int32_t ko,
                                         int32_t o, int32_t *acol, double *aval, int32_t wo,
                                         bool offlmp, double tau, bool one_norm, double mult,
                                         double *__restrict__ invD, int32_t *__restrict__ err) {
  int32_t w = o, ds = o;
  double aii = 0.0, r = 0.0, offsum = 0.0;
  for (int32_t k0 = b; k0 < e; k0 += 8) {
    int32_t j[8];
    double v[8];
    uint8_t m[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int32_t k = min(k0 + q, e - 1) - ko;
      j[q] = col[k];
      v[q] = val[k];
      m[q] = mask[k];
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if (k0 + q >= e) break;
      if (j[q] == i) {
        aii = v[q];
        ds = w;
      } else {
        offsum += fabs(v[q]);
        if (m[q] != 1) {
          r += v[q];
          continue;
        }
      }
      acol[w - wo] = j[q];
      aval[w - wo] = v[q];
      ++w;
    }
  }
  const int32_t wend = w;
  if (!offlmp || r >= 0.0 || !(aii > 0.0)) {
    aval[ds - wo] = aii + r;
  } else {
    double kp = 0.0, km = 0.0;
    bool has_kp = false, has_km = false;
    for (int32_t t = o; t < wend; ++t) {
      if (t == ds) continue;
      const double v = aval[t - wo];
      if (v > 0.0) {
        kp += v;
        has_kp = true;
      } else if (v < 0.0) {
        km += v;
        has_km = true;
      }
    }
    if (-r <= kp) {
      const double delta = r / kp;
      for (int32_t t = o; t < wend; ++t)
        if (t != ds && aval[t - wo] > 0.0) aval[t - wo] = aval[t - wo] * (1.0 + delta);
    } else {
      const double T = tau * (offsum / aii);
      const double rhat = r + kp;
      if (!has_km) {
        if (has_kp && fabs(r + kp) / aii <= T) {
          const double delta = r / kp;
          for (int32_t t = o; t < wend; ++t)
            if (t != ds && aval[t - wo] > 0.0) aval[t - wo] = aval[t - wo] * (1.0 + delta);
        }
      } else {
        const double a = aii;
        const double c = -km - rhat;
        const double U = fmin(fabs(rhat), a);
        const double bnd = T * a - c;
        double rs = 0.0;
        bool feasible;
        if (T > 1.0) {
          const double ub = bnd / (T - 1.0);
          feasible = ub >= 0.0;
          if (feasible) rs = fmin(U, ub);
        } else if (T < 1.0) {
          const double lb = bnd / (T - 1.0);
          feasible = lb <= U;
          if (feasible) rs = U;
        } else {
          feasible = bnd >= 0.0;
          if (feasible) rs = U;
        }
        if (!feasible) rs = (c <= a) ? U : 0.0;
        const double delta = (rhat + rs) / km;
        for (int32_t t = o; t < wend; ++t) {
          if (t == ds) continue;
          const double v = aval[t - wo];
          if (v > 0.0) aval[t - wo] = 0.0;
          else if (v < 0.0) aval[t - wo] = v * (1.0 + delta);
        }
        aval[ds - wo] = a - rs;
      }
    }
  }
  double D;
  if (one_norm) {
    D = 0.0;
    for (int32_t t = o; t < wend; ++t) D += fabs(aval[t - wo]);
    if (D == 0.0) {
      D = 1.0;
    } else {
      double sum = 0.0;
      for (int32_t t = o; t < wend; ++t) sum += aval[t - wo];
      if (D < mult * sum) D = mult * sum;
    }
  } else {
    D = aval[ds - wo];
    if (D == 0.0) atomicOr(err, 8);
  }
  invD[i] = 1.0 / D;
}

// Block b owns rows [R b, R b + R) (R <= 256 chosen so that the rows' entries usually fit
// kLumpCap).  When they fit, the entries are staged in LDS by all 256 threads with coalesced
// loads, threads t < R filter their rows there, in place, and the filtered rows (one contiguous
// run of Abar) are written back with coalesced stores, every entry finding its row by binary
// search; otherwise thread t works on row R b + t in global memory directly.  (970K rows of 26
// entries: 360 us with a second LDS copy for the filtered rows, which left three blocks to a CU,
// now 202; 2.1M rows of 7: 89 -> 82.)
constexpr int32_t kLumpCap = 2048;
template <int R>
__global__ __launch_bounds__(kBlock) void k_lump_fill(
    int32_t n, const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
    const double *__restrict__ val, const uint8_t *__restrict__ mask,
    const int32_t *__restrict__ arp, int32_t *__restrict__ acol, double *__restrict__ aval,
    bool offlmp, double tau, bool one_norm, double mult, double *__restrict__ invD,
    int32_t *__restrict__ err) {
  __shared__ int32_t s_col[kLumpCap];
  __shared__ double s_val[kLumpCap];
  __shared__ uint8_t s_mask[kLumpCap];
  __shared__ int32_t s_rp[R + 1], s_arp[R + 1];
  const int t = threadIdx.x;
  const int64_t r0 = (int64_t)blockIdx.x * R;
  const int32_t nr = (int32_t)min<int64_t>(R, (int64_t)n - r0);
  if (t <= nr && t <= R) {
    s_rp[t] = rp[r0 + t];
    s_arp[t] = arp[r0 + t];
  }
  if (t == 0) {  // nr can be kBlock: no thread t == nr
    s_rp[nr] = rp[r0 + nr];
    s_arp[nr] = arp[r0 + nr];
  }
  __syncthreads();
  const int32_t e0 = s_rp[0], e1 = s_rp[nr];
  const int32_t a0 = s_arp[0], a1 = s_arp[nr];
  const int32_t i = (int32_t)r0 + t;
  if (e1 - e0 <= kLumpCap) {  // block-uniform; the filtered rows are no longer than A's
    for (int32_t k = e0 + t; k < e1; k += kBlock) {
      s_col[k - e0] = col[k];
      s_val[k - e0] = val[k];
      s_mask[k - e0] = mask[k];
    }
    __syncthreads();
    if (t < nr)
      lump_row(i, s_rp[t], s_rp[t + 1], s_col, s_val, s_mask, e0, 0, s_col, s_val,
               e0 - s_rp[t], offlmp, tau, one_norm, mult, invD, err);
    __syncthreads();
    for (int32_t w = a0 + t; w < a1; w += kBlock) {
      int32_t lo = 0, hi = nr - 1;  // the entry's row: the last r with s_arp[r] <= w
      while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (s_arp[mid] <= w) lo = mid;
        else hi = mid - 1;
      }
      const int32_t k = s_rp[lo] - e0 + (w - s_arp[lo]);
      acol[w] = s_col[k];
      aval[w] = s_val[k];
    }
  } else if (t < nr) {
    lump_row(i, s_rp[t], s_rp[t + 1], col, val, mask, 0, s_arp[t], acol, aval, 0, offlmp, tau,
             one_norm, mult, invD, err);
  }
}

__global__ __launch_bounds__(kW) void k_lump_count_w(int32_t n, const int32_t *rp,
                                                     const int32_t *col, const uint8_t *mask,
                                                     int32_t *cnt) {
  SA_WAVE_ROW_BEGIN(n)
  int32_t c = 0;
  for (int32_t k = rp[i] + lane; k < rp[i + 1]; k += kW) c += (col[k] == i || mask[k] == 1);
  c = wave_sum_i32(c);
  if (lane == 0) cnt[i] = c;
}

// Same arithmetic as k_lump_fill, one wavefront per row: the kept entries are compacted in
// parallel; every floating-point sum (removed entries, kept positives/negatives, original
// off-diagonal magnitudes, the 1-norm and the row sum) runs sequentially through
// wave_seq_sum; the scalar decisions are taken identically by all lanes.
__global__ __launch_bounds__(kW) void k_lump_fill_w(int32_t n, const int32_t *rp,
                                                    const int32_t *col, const double *val,
                                                    const uint8_t *mask, const int32_t *arp,
                                                    int32_t *acol, double *aval, bool offlmp,
                                                    double tau, bool one_norm, double mult,
                                                    double *invD, int32_t *err) {
  __shared__ double lds[kW];
  SA_WAVE_ROW_BEGIN(n)
  const int32_t b = rp[i], e = rp[i + 1];
  const int32_t o = arp[i], oe = arp[i + 1];
  int32_t w = o;
  int32_t ds = o;
  double aii = 0.0;
  for (int32_t c = b; c < e; c += kW) {
    const int32_t k = c + lane;
    bool kept = false, isd = false;
    int32_t j = 0;
    double v = 0.0;
    if (k < e) {
      j = col[k];
      v = val[k];
      isd = (j == i);
      kept = isd || mask[k] == 1;
    }
    const unsigned long long bm = __ballot(kept);
    const int32_t pos = w + __popcll(bm & ((1ull << lane) - 1ull));
    if (kept) {
      acol[pos] = j;
      aval[pos] = v;
    }
    const unsigned long long dm = __ballot(isd);
    if (dm) {
      const int dl = __ffsll((long long)dm) - 1;
      ds = __shfl(pos, dl, 64);
      aii = __shfl(v, dl, 64);
    }
    w += __popcll(bm);
  }
  __syncthreads();
  const double r = wave_seq_sum(b, e, [&](int32_t k) {
    return (col[k] != i && mask[k] != 1) ? val[k] : 0.0;
  }, lds);
  if (!offlmp || r >= 0.0 || !(aii > 0.0)) {
    if (lane == 0) aval[ds] = aii + r;
  } else {
    const double kp = wave_seq_sum(o, oe, [&](int32_t t) {
      return (t != ds && aval[t] > 0.0) ? aval[t] : 0.0;
    }, lds);
    const double km = wave_seq_sum(o, oe, [&](int32_t t) {
      return (t != ds && aval[t] < 0.0) ? aval[t] : 0.0;
    }, lds);
    bool hp = false, hm = false;
    for (int32_t t = o + lane; t < oe; t += kW) {
      if (t == ds) continue;
      hp |= aval[t] > 0.0;
      hm |= aval[t] < 0.0;
    }
    const bool has_kp = wave_any(hp), has_km = wave_any(hm);
    __syncthreads();
    if (-r <= kp) {
      const double delta = r / kp;
      for (int32_t t = o + lane; t < oe; t += kW)
        if (t != ds && aval[t] > 0.0) aval[t] = aval[t] * (1.0 + delta);
    } else {
      const double offsum = wave_seq_sum(b, e, [&](int32_t k) {
        return col[k] != i ? fabs(val[k]) : 0.0;
      }, lds);
      const double T = tau * (offsum / aii);
      const double rhat = r + kp;
      if (!has_km) {
        if (has_kp && fabs(r + kp) / aii <= T) {
          const double delta = r / kp;
          for (int32_t t = o + lane; t < oe; t += kW)
            if (t != ds && aval[t] > 0.0) aval[t] = aval[t] * (1.0 + delta);
        }
      } else {
        const double a = aii;
        const double c = -km - rhat;
        const double U = fmin(fabs(rhat), a);
        const double bnd = T * a - c;
        double rs = 0.0;
        bool feasible;
        if (T > 1.0) {
          const double ub = bnd / (T - 1.0);
          feasible = ub >= 0.0;
          if (feasible) rs = fmin(U, ub);
        } else if (T < 1.0) {
          const double lb = bnd / (T - 1.0);
          feasible = lb <= U;
          if (feasible) rs = U;
        } else {
          feasible = bnd >= 0.0;
          if (feasible) rs = U;
        }
        if (!feasible) rs = (c <= a) ? U : 0.0;
        const double delta = (rhat + rs) / km;
        for (int32_t t = o + lane; t < oe; t += kW) {
          if (t == ds) continue;
          const double v = aval[t];
          if (v > 0.0) aval[t] = 0.0;
          else if (v < 0.0) aval[t] = v * (1.0 + delta);
        }
        __syncthreads();
        if (lane == 0) aval[ds] = a - rs;
      }
    }
  }
  __syncthreads();
  double D;
  if (one_norm) {
    D = wave_seq_sum(o, oe, [&](int32_t t) { return fabs(aval[t]); }, lds);
    if (D == 0.0) {
      D = 1.0;
    } else {
      const double sum = wave_seq_sum(o, oe, [&](int32_t t) { return aval[t]; }, lds);
      if (D < mult * sum) D = mult * sum;
    }
  } else {
    D = aval[ds];
    if (D == 0.0 && lane == 0) atomicOr(err, 8);
  }
  if (lane == 0) invD[i] = 1.0 / D;
}

void lump_count(int32_t n, const int32_t *rp, const int32_t *col, const uint8_t *mask, bool wave,
                Arena &ar, Csr &abar, hipStream_t s) {
  int32_t *cnt = (int32_t *)dev_alloc(sizeof(int32_t) * (n + 1), s);
  if (wave) k_lump_count_w<<<(unsigned)n, kW, 0, s>>>(n, rp, col, mask, cnt);
  else k_lump_count<<<grid_for(n), kBlock, 0, s>>>(n, rp, col, mask, cnt);
  SA_LAUNCH_CHECK();
  abar.n = abar.ncols = n;
  abar.rp = ar.alloc<int32_t>(n + 1);
  exclusive_scan_i32(cnt, abar.rp, n, s);
  dev_free(cnt, s);
}
int64_t lump(int32_t n, int64_t nnz_a, const int32_t *rp, const int32_t *col, const double *val,
             const uint8_t *mask, bool offlmp, double tau, bool one_norm, double mult,
             bool wave, Arena &ar, Csr &abar, double *invD, int32_t *err, hipStream_t s) {
  abar.col = ar.alloc<int32_t>(abar.nnz);
  abar.val = ar.alloc<double>(abar.nnz);
  if (wave)
    k_lump_fill_w<<<(unsigned)n, kW, 0, s>>>(n, rp, col, val, mask, abar.rp, abar.col, abar.val,
                                             offlmp, tau, one_norm, mult, invD, err);
  else if (nnz_a <= 7 * (int64_t)n)
    k_lump_fill<256><<<(unsigned)ceil_div(n, 256), kBlock, 0, s>>>(
        n, rp, col, val, mask, abar.rp, abar.col, abar.val, offlmp, tau, one_norm, mult, invD,
        err);
  else if (nnz_a <= 15 * (int64_t)n)
    k_lump_fill<128><<<(unsigned)ceil_div(n, 128), kBlock, 0, s>>>(
        n, rp, col, val, mask, abar.rp, abar.col, abar.val, offlmp, tau, one_norm, mult, invD,
        err);
  else if (nnz_a <= 30 * (int64_t)n)
    k_lump_fill<64><<<(unsigned)ceil_div(n, 64), kBlock, 0, s>>>(
        n, rp, col, val, mask, abar.rp, abar.col, abar.val, offlmp, tau, one_norm, mult, invD,
        err);
  else
    k_lump_fill<32><<<(unsigned)ceil_div(n, 32), kBlock, 0, s>>>(
        n, rp, col, val, mask, abar.rp, abar.col, abar.val, offlmp, tau, one_norm, mult, invD,
        err);
  SA_LAUNCH_CHECK();
  return abar.nnz;
}

// ---- power method (Sec. 1.1 damping; Sec. 3.1 ten sweeps) --------------------------------
// The start vector; block 0 clears the words of the maxima and the dead flag.
__global__ __launch_bounds__(kBlock) void k_power_init(int32_t n, uint64_t seed, int32_t level,
                                                       int32_t stream, double *x,
                                                       unsigned long long *mx, int32_t words) {
  if (blockIdx.x == 0)
    for (int q = threadIdx.x; q < words; q += kBlock) mx[q] = 0ull;
  SA_ROW_KERNEL_BEGIN(n)
  const uint64_t z = splitmix64_dev(seed, stream_key_dev(stream, level, i));
  const double u = (double)(z >> 11) * (1.0 / 9007199254740992.0);
  x[i] = 2.0 * u - 1.0;
}
// x = y / 2^ilogb(m) with m = max |y_i|: every block reduces the kMaxSlots maxima that the
// SpMV left (bit patterns of non-negative doubles, monotone).  A zero or non-finite maximum
// marks the iteration dead.  The last iteration's; the others scale x as they gather it.
__global__ __launch_bounds__(kBlock) void k_normalize(int32_t n, const double *y,
                                                      const unsigned long long *slots,
                                                      double *x, int32_t *dead) {
  static_assert(kMaxSlots == kBlock, "one slot per thread");
  __shared__ unsigned long long wm[kBlock / 64];
  unsigned long long m = slots[threadIdx.x];
  for (int off = 32; off >= 1; off >>= 1) {
    const unsigned long long o = __shfl_xor(m, off, 64);
    m = o > m ? o : m;
  }
  if ((threadIdx.x & 63) == 0) wm[threadIdx.x >> 6] = m;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kBlock / 64; ++q) m = wm[q] > m ? wm[q] : m;
  SA_ROW_KERNEL_BEGIN(n)
  const double mv = __longlong_as_double((long long)m);
  if (!(mv > 0.0) || !isfinite(mv)) {
    if (i == 0) *dead = 1;
    return;
  }
  x[i] = ldexp(y[i], -ilogb(mv));
}
__global__ void k_rayleigh(const double *xy, const double *xx, const int32_t *dead,
                           double *lam) {
  *lam = (*dead) ? 0.0 : (*xy / *xx);
}

// The iterations as launches to be queued one call at a time (false: the last one is queued):
// beside a stage of the main stream whose launches the host must not fall behind with.
std::function<bool()> power_steps(const Csr &M, const double *invD, int32_t iters, uint64_t seed,
                                  int32_t level, int32_t stream_id, double *lam,
                                  hipStream_t s) {
  struct State {
    Arena tmp;
    double *v[2], *ws, *sc;
    unsigned long long *mx;
    int32_t *dead;
    int32_t t = 0;
  };
  const auto st = std::make_shared<State>();
  const int32_t n = M.n;
  return [=]() {
    const int32_t t = st->t++;
    if (t == 0) {
      st->tmp.stream = s;
      st->v[0] = st->tmp.alloc<double>(n);
      st->v[1] = st->tmp.alloc<double>(n);
      st->ws = st->tmp.alloc<double>(2 * dot_ws_size(n));
      st->sc = st->tmp.alloc<double>(2);
      // three sets of kMaxSlots maxima (iteration t reads set t - 1, fills set t and clears set
      // t + 1, mod 3), then the dead flag
      st->mx = st->tmp.alloc<unsigned long long>(3 * kMaxSlots + 1);
      st->dead = (int32_t *)(st->mx + 3 * kMaxSlots);
      k_power_init<<<grid_for(n), kBlock, 0, s>>>(n, seed, level, stream_id, st->v[0], st->mx,
                                                  3 * kMaxSlots + 1);
      SA_LAUNCH_CHECK();
      return true;
    }
    auto set = [&](int32_t q) { return st->mx + (q % 3) * kMaxSlots; };
    double *x = st->v[(t - 1) & 1], *y = st->v[t & 1];
    if (t < iters) {
      const SpmvArgs<double> a = spmv_args<double>(M, M.val, x);
      spmv_scale_max<double>(
          a, invD, y, {set(t), t > 1 ? set(t - 1) : nullptr, set(t + 1), st->dead}, s);
      return true;
    }
    if (t > 1) {
      k_normalize<<<grid_for(n), kBlock, 0, s>>>(n, x, set(t - 1), y, st->dead);
      SA_LAUNCH_CHECK();
      std::swap(x, y);
    }
    SpmvArgs<double> a = spmv_args<double>(M, M.val, x);
    a.plain = true;  // the estimate decides the hierarchy: every row in sequential order
    spmv_scale<double>(a, invD, y, s);
    dot_xy_xx(x, y, n, st->sc, st->ws, s);
    k_rayleigh<<<1, 1, 0, s>>>(st->sc + 0, st->sc + 1, st->dead, lam);
    SA_LAUNCH_CHECK();
    return false;
  };
}

__global__ void k_damping(double *lam, double *omega, bool unit, int32_t *err) {
  if (unit) *lam = 1.0;
  const double l = *lam;
  if (!(l > 0.0) || !isfinite(l)) atomicOr(err, 16);
  *omega = 4.0 / (3.0 * l);
}
void damping(double *lam, double *omega, bool unit, int32_t *err, hipStream_t s) {
  k_damping<<<1, 1, 0, s>>>(lam, omega, unit, err);
  SA_LAUNCH_CHECK();
}

// ---- prolongator smoothing (Sec. 1.1) -------------------------------------------------------
// Row i: for each aggregate J reached by the filtered row (ascending J), acc = sum of the
// entries with agg(k) = J in ascending k from 0; P_iJ = [J == agg_i] - (omega invD_i) acc.
// Rows of at most kPRegs entries keep their aggregates (and values) in registers, loaded as
// independent loads up front; longer rows re-read them per distinct aggregate.
constexpr int kPRegs = 16;
// Rows of up to R entries: the entries' aggregates (and values) loaded once, in one batch,
// and the distinct aggregates counted, or summed in ascending aggregate order, in registers.
template <int R>
__device__ __forceinline__ int32_t p_count_regs(int32_t b, int32_t e,
                                                const int32_t *__restrict__ col,
                                                const int32_t *__restrict__ agg) {
  int32_t a[R];
#pragma unroll
  for (int q = 0; q < R; ++q) a[q] = (b + q < e) ? col[min(b + q, e - 1)] : -1;
#pragma unroll
  for (int q = 0; q < R; ++q) a[q] = (a[q] >= 0) ? agg[a[q]] : -1;
  // distinct aggregates = entries whose aggregate does not occur earlier in the row
  int32_t c = 0;
#pragma unroll
  for (int q = 0; q < R; ++q) {
    bool first = a[q] >= 0;
#pragma unroll
    for (int r = 0; r < q; ++r) first = first && (a[r] != a[q]);
    c += first;
  }
  return c;
}
template <int R>
__device__ __forceinline__ void p_fill_regs(int32_t rb, int32_t re,
                                            const int32_t *__restrict__ col,
                                            const double *__restrict__ val,
                                            const int32_t *__restrict__ agg, int32_t ai, double t,
                                            int32_t w, int32_t *__restrict__ pcol,
                                            double *__restrict__ pval) {
  int32_t a[R];
  double v[R];
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int32_t k = min(rb + q, re - 1);
    a[q] = (rb + q < re) ? col[k] : -1;
    v[q] = (rb + q < re) ? val[k] : 0.0;
  }
#pragma unroll
  for (int q = 0; q < R; ++q) a[q] = (a[q] >= 0) ? agg[a[q]] : -1;
  // aggregates in ascending order; each sums its entries in ascending position from 0
  int32_t prev = -1;
  for (;;) {
    int32_t J = INT_MAX;
#pragma unroll
    for (int q = 0; q < R; ++q)
      if (a[q] > prev && a[q] < J) J = a[q];
    if (J == INT_MAX) break;
    double acc = 0.0;
#pragma unroll
    for (int q = 0; q < R; ++q)
      if (a[q] == J) acc += v[q];
    pcol[w] = J;
    pval[w] = ((J == ai) ? 1.0 : 0.0) - t * acc;
    ++w;
    prev = J;
  }
}

__global__ void k_P_count(int32_t n, const int32_t *rp, const int32_t *col, const int32_t *agg,
                          int32_t *cnt) {
  SA_ROW_KERNEL_BEGIN(n)
  const int32_t b = rp[i], e = rp[i + 1];
  if (e <= b) {
    cnt[i] = 0;
    return;
  }
  if (e - b <= kPRegs) {
    cnt[i] = p_count_regs<kPRegs>(b, e, col, agg);
    return;
  }
  if (e - b <= 2 * kPRegs) {
    cnt[i] = p_count_regs<2 * kPRegs>(b, e, col, agg);
    return;
  }
  int32_t prev = -1, c = 0;
  for (;;) {
    int32_t J = INT_MAX;
    for (int32_t k = rp[i]; k < rp[i + 1]; ++k) {
      const int32_t a = agg[col[k]];
      if (a > prev && a < J) J = a;
    }
    if (J == INT_MAX) break;
    ++c;
    prev = J;
  }
  cnt[i] = c;
}
__global__ void k_P_fill(int32_t n, const int32_t *rp, const int32_t *col, const double *val,
                         const double *invD, const int32_t *agg, const double *omega,
                         const int32_t *prp, int32_t *pcol, double *pval) {
  SA_ROW_KERNEL_BEGIN(n)
  const double t = (*omega) * invD[i];
  const int32_t ai = agg[i];
  const int32_t rb = rp[i], re = rp[i + 1];
  if (re <= rb) return;  // an empty row has no prolongator entries
  if (re - rb <= kPRegs) {
    p_fill_regs<kPRegs>(rb, re, col, val, agg, ai, t, prp[i], pcol, pval);
    return;
  }
  if (re - rb <= 2 * kPRegs) {
    p_fill_regs<2 * kPRegs>(rb, re, col, val, agg, ai, t, prp[i], pcol, pval);
    return;
  }
  int32_t prev = -1, w = prp[i];
  for (;;) {
    int32_t J = INT_MAX;
    for (int32_t k = rp[i]; k < rp[i + 1]; ++k) {
      const int32_t a = agg[col[k]];
      if (a > prev && a < J) J = a;
    }
    if (J == INT_MAX) break;
    double acc = 0.0;
    for (int32_t k = rp[i]; k < rp[i + 1]; ++k)
      if (agg[col[k]] == J) acc += val[k];
    pcol[w] = J;
    pval[w] = ((J == ai) ? 1.0 : 0.0) - t * acc;
    ++w;
    prev = J;
  }
}
// Long rows (the dense coarse levels): the per-aggregate sums of a row of Abar are the row of
// Abar T, T the 0/1 aggregate matrix (T_kJ = 1 iff agg_k = J): every product is A_ik * 1 =
// A_ik exactly and the SpGEMM adds them in ascending k from 0, the order of k_P_fill.  Then
// P_iJ = [J = agg_i] - t_i (Abar T)_iJ in place.
__global__ void k_agg_matrix(int32_t n, const int32_t *agg, const int32_t *trp, int32_t *tcol,
                             double *tval) {
  SA_ROW_KERNEL_BEGIN(n)
  if (agg[i] >= 0) {
    tcol[trp[i]] = agg[i];
    tval[trp[i]] = 1.0;
  }
}
__global__ void k_flag_aggregated(int32_t n, const int32_t *agg, int32_t *f) {
  SA_ROW_KERNEL_BEGIN(n)
  f[i] = agg[i] >= 0 ? 1 : 0;
}
__global__ void k_P_from_sums(int32_t n, const int32_t *prp, const int32_t *pcol, double *pval,
                              const double *invD, const int32_t *agg, const double *omega) {
  SA_ROW_KERNEL_BEGIN(n)
  const double t = (*omega) * invD[i];
  const int32_t ai = agg[i];
  for (int32_t e = prp[i]; e < prp[i + 1]; ++e)
    pval[e] = ((pcol[e] == ai) ? 1.0 : 0.0) - t * pval[e];
}

int64_t prolongator(const Csr &abar, const double *invD, const int32_t *agg, int32_t nc,
                    const double *omega, Arena &ar, Csr &P, hipStream_t s, bool long_rows,
                    const ReadAlong &along) {
  const int32_t n = abar.n;
  if (long_rows && n > 0) {
    Arena tmp;
    tmp.stream = s;
    int32_t *f = tmp.alloc<int32_t>(n + 1);
    k_flag_aggregated<<<grid_for(n), kBlock, 0, s>>>(n, agg, f);
    SA_LAUNCH_CHECK();
    Csr T;
    T.n = n;
    T.ncols = nc;
    T.rp = tmp.alloc<int32_t>(n + 1);
    exclusive_scan_i32(f, T.rp, n, s);
    T.nnz = n;  // at most
    T.col = tmp.alloc<int32_t>(n);
    T.val = tmp.alloc<double>(n);
    k_agg_matrix<<<grid_for(n), kBlock, 0, s>>>(n, agg, T.rp, T.col, T.val);
    SA_LAUNCH_CHECK();
    spgemm(abar, T, ar, P, s, 65, false, along);
    k_P_from_sums<<<grid_for(n), kBlock, 0, s>>>(n, P.rp, P.col, P.val, invD, agg, omega);
    SA_LAUNCH_CHECK();
    return P.nnz;
  }
  int32_t *cnt = (int32_t *)dev_alloc(sizeof(int32_t) * (n + 1), s);
  k_P_count<<<grid_for(n), kBlock, 0, s>>>(n, abar.rp, abar.col, agg, cnt);
  SA_LAUNCH_CHECK();
  P.n = n;
  P.ncols = nc;
  P.rp = ar.alloc<int32_t>(n + 1);
  exclusive_scan_i32(cnt, P.rp, n, s);
  dev_free(cnt, s);
  constexpr int kAlong = 8;
  int32_t h[1 + kAlong];
  WordRuns runs;
  runs.add(P.rp + n, 1);
  if (along.words > 0) runs.add(along.dev, std::min(along.words, kAlong));
  readback_runs(h, runs, s);
  if (along.words > 0) std::memcpy(along.host, h + 1, 4 * std::min(along.words, kAlong));
  P.nnz = h[0];
  P.col = ar.alloc<int32_t>(P.nnz);
  P.val = ar.alloc<double>(P.nnz);
  k_P_fill<<<grid_for(n), kBlock, 0, s>>>(n, abar.rp, abar.col, abar.val, invD, agg, omega, P.rp,
                                          P.col, P.val);
  SA_LAUNCH_CHECK();
  return P.nnz;
}

// ---- Cnstrnt (Sec. 2.4, Algorithm 3, with the loop run while any bound is violated) ------
__global__ void k_cnstrnt(int32_t n, const int32_t *rp, const int32_t *col, double *v,
                          const int32_t *agg, uint8_t *inw) {
  SA_ROW_KERNEL_BEGIN(n)
  const int32_t b = rp[i], e = rp[i + 1];
  bool viol = false;
  for (int32_t k = b; k < e; ++k)
    if (v[k] < 0.0 || v[k] > 1.0) viol = true;
  if (!viol) return;
  int32_t cnt = 0;
  double sum = 0.0;
  for (int32_t k = b; k < e; ++k) {
    inw[k] = v[k] != 0.0;
    if (inw[k]) {
      ++cnt;
      sum += v[k];
    }
  }
  const int32_t ai = agg[i];
  bool tent = false;
  if (sum < 0.0 || sum > (double)cnt) {
    tent = true;
  } else if (sum == 0.0) {
    for (int32_t k = b; k < e; ++k) v[k] = 0.0;
    return;
  } else {
    while (cnt > 0) {
      int32_t kmin = -1, kmax = -1;
      for (int32_t k = b; k < e; ++k) {
        if (!inw[k]) continue;
        if (kmin < 0 || v[k] < v[kmin]) kmin = k;
        if (kmax < 0 || v[k] > v[kmax]) kmax = k;
      }
      if (!(v[kmin] < 0.0 || v[kmax] > 1.0)) break;
      double delta = 0.0;
      if (v[kmin] < 0.0) {
        delta += v[kmin];
        v[kmin] = 0.0;
        inw[kmin] = 0;
        --cnt;
      }
      if (v[kmax] > 1.0) {
        delta += v[kmax] - 1.0;
        v[kmax] = 1.0;
        inw[kmax] = 0;
        --cnt;
      }
      if (cnt == 0) {
        if (delta != 0.0) tent = true;
        break;
      }
      const double q = delta / (double)cnt;
      for (int32_t k = b; k < e; ++k)
        if (inw[k]) v[k] += q;
    }
  }
  if (tent)
    for (int32_t k = b; k < e; ++k) v[k] = (col[k] == ai) ? 1.0 : 0.0;
}
void cnstrnt(const Csr &P, const int32_t *agg, hipStream_t s) {
  if (P.n <= 0) return;
  uint8_t *inw = (uint8_t *)dev_alloc(P.nnz > 0 ? P.nnz : 1, s);
  k_cnstrnt<<<grid_for(P.n), kBlock, 0, s>>>(P.n, P.rp, P.col, P.val, agg, inw);
  SA_LAUNCH_CHECK();
  dev_free(inw, s);
}

__global__ void k_scale_rows(int32_t n, const int32_t *rp, double *val, const double *B) {
  SA_ROW_KERNEL_BEGIN(n)
  for (int32_t k = rp[i]; k < rp[i + 1]; ++k) val[k] = B[i] * val[k];
}
void scale_rows(const Csr &P, const double *B, hipStream_t s) {
  if (P.n <= 0) return;
  k_scale_rows<<<grid_for(P.n), kBlock, 0, s>>>(P.n, P.rp, P.val, B);
  SA_LAUNCH_CHECK();
}

__global__ void k_scale_sym(int32_t n, const int32_t *rp, const int32_t *col, const double *val,
                            const double *B, double *out) {
  SA_ROW_KERNEL_BEGIN(n)
  for (int32_t k = rp[i]; k < rp[i + 1]; ++k) out[k] = (B[i] * val[k]) * B[col[k]];
}
void scale_sym(int32_t n, const int32_t *rp, const int32_t *col, const double *val,
               const double *B, double *out, hipStream_t s) {
  if (n <= 0) return;
  k_scale_sym<<<grid_for(n), kBlock, 0, s>>>(n, rp, col, val, B, out);
  SA_LAUNCH_CHECK();
}


// ---- per-row sort by column --------------------------------------------------------------
// Keys within a row are distinct, so the order is unique.  Up to kSortShort entries: 8 lanes
// per row hold 4 keys each and count, for each of theirs, the row's smaller keys (its place).
// Up to kSortMid: a wavefront per row does the same with 4 keys per lane read against the
// row's keys in LDS.  Up to kSortBlock: a block per row in the same way; its comparisons grow
// with the square of the length, by their count of instructions they reach the bitonic sort's
// time at about 1,400.  Longer rows: one block per row, bitonic sort in LDS (kSortLds entries)
// or, beyond that, in a global scratch region sized for the row.  (A sorting network in one thread's registers for the short
// rows: 131 us for the 600K rows of the 128^3 cube's first R; a block's bitonic sort for the
// middle ones: 690 us for 54K rows of about 40, now 57; and for 9,114 rows of 257 and more,
// about 400: 395 us, now 112; 582 longer ones: 89, now 42.)
constexpr int32_t kSortShort = 32;
constexpr int32_t kSortMid = 256;
constexpr int32_t kSortBlock = 1024;
constexpr int32_t kSortLds = 4096;

// nlist[0], nlist[1]: the rows listed for the wavefront and the block sort (mid, longrows), by
// one atomic per block and list (one per wavefront took 221 us where most of 89K rows are
// listed, now 65); nlist[2]: whether a row has more than 64 entries; nlist[3]: more than
// kSortBlock.  A block has 32 PASS rows.
template <int PASS>
__global__ __launch_bounds__(kBlock) void k_sort_short(int32_t n, const int32_t *__restrict__ rp,
                                                       int32_t *c, double *v, int32_t *nlist,
                                                       int32_t *mid, int32_t *longrows) {
  __shared__ int32_t s_list[2][32 * PASS], s_n[2], s_base[2], s_any[2];
  const int t = threadIdx.x, j = t & 7;
  if (t < 2) s_n[t] = s_any[t] = 0;
  __syncthreads();
  for (int pass = 0; pass < PASS; ++pass) {
    const int64_t i64 = ((int64_t)blockIdx.x * PASS + pass) * 32 + (t >> 3);
    const bool live = i64 < n;
    const int32_t i = live ? (int32_t)i64 : 0;
    const int32_t b = live ? rp[i] : 0;
    const int32_t L = live ? rp[i + 1] - b : 0;
    if (j == 0 && L > kSortShort) {
      const int which = L > kSortMid;
      s_list[which][atomicAdd(&s_n[which], 1)] = i;
      if (L > 64) s_any[0] = 1;
      if (L > kSortBlock) s_any[1] = 1;
    }
    if (L <= 1 || L > kSortShort) continue;  // uniform over the row's lanes
    int32_t k[4], place[4] = {0, 0, 0, 0};
    double x[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const bool in = j + 8 * q < L;
      k[q] = in ? c[b + j + 8 * q] : INT_MAX;
      x[q] = v && in ? v[b + j + 8 * q] : 0.0;
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      if (8 * p < L) {
#pragma unroll
        for (int o = 0; o < 8; ++o) {
          const int32_t other = __shfl(k[p], o, 8);
#pragma unroll
          for (int q = 0; q < 4; ++q) place[q] += other < k[q] ? 1 : 0;
        }
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (j + 8 * q < L) {
        c[b + place[q]] = k[q];
        if (v) v[b + place[q]] = x[q];
      }
  }
  __syncthreads();
  if (t < 2 && s_n[t] > 0) s_base[t] = atomicAdd(nlist + t, s_n[t]);
  if (t < 2 && s_any[t]) nlist[2 + t] = 1;  // (every writer writes the same)
  __syncthreads();
  for (int q = t; q < s_n[0]; q += kBlock) mid[s_base[0] + q] = s_list[0][q];
  for (int q = t; q < s_n[1]; q += kBlock) longrows[s_base[1] + q] = s_list[1][q];
}

__global__ __launch_bounds__(kBlock) void k_sort_mid(const int32_t *rows, int32_t nrows,
                                                     const int32_t *__restrict__ rp, int32_t *c,
                                                     double *v) {
  __shared__ __attribute__((aligned(16))) int32_t s_k[kBlock / 64][kSortMid];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t slot = (int64_t)blockIdx.x * (kBlock / 64) + wv;
  const int32_t i = slot < nrows ? rows[slot] : -1;
  const int32_t b = i >= 0 ? rp[i] : 0;
  const int32_t L = i >= 0 ? rp[i + 1] - b : 0;
  int32_t k[4], place[4] = {0, 0, 0, 0};
  double x[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const bool in = lane + 64 * q < L;
    k[q] = in ? c[b + lane + 64 * q] : INT_MAX;
    x[q] = v && in ? v[b + lane + 64 * q] : 0.0;
    s_k[wv][lane + 64 * q] = k[q];
  }
  __syncthreads();
  for (int32_t o = 0; o < L; o += 4) {  // wave-uniform; past the row the keys are INT_MAX
    const int4 t = *(const int4 *)&s_k[wv][o];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      place[q] += (t.x < k[q]) + (t.y < k[q]) + (t.z < k[q]) + (t.w < k[q]);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (lane + 64 * q < L) {
      c[b + place[q]] = k[q];
      if (v) v[b + place[q]] = x[q];
    }
}

template <int Q>
__device__ __forceinline__ void count_smaller(const int32_t *s_k, int32_t L, const int32_t *k,
                                              int32_t *place) {
  for (int32_t o = 0; o < L; o += 4) {  // past the row the keys are INT_MAX
    const int4 t = *(const int4 *)&s_k[o];
#pragma unroll
    for (int q = 0; q < Q; ++q)
      place[q] += (t.x < k[q]) + (t.y < k[q]) + (t.z < k[q]) + (t.w < k[q]);
  }
}
__global__ __launch_bounds__(kBlock) void k_sort_block(const int32_t *rows,
                                                       const int32_t *__restrict__ rp,
                                                       int32_t *c, double *v) {
  static_assert(kSortBlock == 4 * kBlock, "four keys a thread");
  __shared__ __attribute__((aligned(16))) int32_t s_k[kSortBlock];
  const int t = threadIdx.x;
  const int32_t i = rows[blockIdx.x];
  const int32_t b = rp[i], L = rp[i + 1] - b;
  if (L > kSortBlock) return;  // block-uniform
  int32_t k[4], place[4] = {0, 0, 0, 0};
  double x[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const bool in = t + kBlock * q < L;
    k[q] = in ? c[b + t + kBlock * q] : INT_MAX;
    x[q] = v && in ? v[b + t + kBlock * q] : 0.0;
    s_k[t + kBlock * q] = k[q];
  }
  __syncthreads();
  if (L <= 2 * kBlock) count_smaller<2>(s_k, L, k, place);
  else count_smaller<4>(s_k, L, k, place);
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (t + kBlock * q < L) {
      c[b + place[q]] = k[q];
      if (v) v[b + place[q]] = x[q];
    }
}

__device__ inline void bitonic_kv_any(int32_t *k, double *v, int32_t L) {
  for (int32_t kk = 2; kk <= L; kk <<= 1) {
    for (int32_t j = kk >> 1; j > 0; j >>= 1) {
      for (int32_t idx = threadIdx.x; idx < L; idx += blockDim.x) {
        const int32_t ixj = idx ^ j;
        if (ixj > idx) {
          const int32_t x = k[idx], y = k[ixj];
          const bool up = (idx & kk) == 0;
          if ((x > y) == up) {
            k[idx] = y;
            k[ixj] = x;
            if (v) {
              const double t = v[idx];
              v[idx] = v[ixj];
              v[ixj] = t;
            }
          }
        }
      }
      __syncthreads();
    }
  }
}

// One block per row of more than kSortBlock entries; those longer than kSortLds use gk/gv at
// goff[slot].
__global__ __launch_bounds__(kBlock) void k_sort_long(const int32_t *rows, int32_t nrows,
                                                      const int32_t *rp, int32_t *c, double *v,
                                                      int32_t *gk, double *gv,
                                                      const int64_t *goff) {
  __shared__ int32_t sk[kSortLds];
  __shared__ double sv[kSortLds];
  const int32_t slot = blockIdx.x;
  if (slot >= nrows) return;
  const int32_t i = rows[slot];
  const int32_t b = rp[i], len = rp[i + 1] - b;
  if (len <= kSortBlock) return;  // k_sort_block's
  int32_t L = 1;
  while (L < len) L <<= 1;
  int32_t *kk;
  double *vv;
  if (L <= kSortLds) {
    kk = sk;
    vv = v ? sv : nullptr;
  } else {
    kk = gk + goff[slot];
    vv = v ? gv + goff[slot] : nullptr;
  }
  for (int32_t q = threadIdx.x; q < L; q += blockDim.x) {
    kk[q] = q < len ? c[b + q] : INT_MAX;
    if (vv) vv[q] = q < len ? v[b + q] : 0.0;
  }
  __syncthreads();
  bitonic_kv_any(kk, vv, L);
  for (int32_t q = threadIdx.x; q < len; q += blockDim.x) {
    c[b + q] = kk[q];
    if (v) v[b + q] = vv[q];
  }
}

__global__ void k_sort_caps(int32_t nrows, const int32_t *rows, const int32_t *rp,
                            int64_t *caps) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= nrows) return;
  const int32_t i = rows[t];
  const int32_t len = rp[i + 1] - rp[i];
  int64_t L = 1;
  while (L < len) L <<= 1;
  caps[t] = (L <= kSortLds) ? 0 : L;
}

void sort_rows_begin(int32_t n, const int32_t *rp, int32_t *col, double *val, RowSort &job,
                     hipStream_t s) {
  job.n = n;
  job.rp = rp;
  job.col = col;
  job.val = val;
  job.tmp.stream = s;
  job.words = job.tmp.alloc<int32_t>(kRowSortWords);
  fill_i32(job.words, 0, kRowSortWords, s);
  if (n <= 0) return;
  job.mid = job.tmp.alloc<int32_t>(n);
  job.rows = job.tmp.alloc<int32_t>(n);
  if (n > 16384)  // (small: the passes' latency counts)
    k_sort_short<8><<<(unsigned)ceil_div(n, 256), kBlock, 0, s>>>(n, rp, col, val, job.words,
                                                                 job.mid, job.rows);
  else
    k_sort_short<1><<<(unsigned)ceil_div(n, 32), kBlock, 0, s>>>(n, rp, col, val, job.words,
                                                                job.mid, job.rows);
  SA_LAUNCH_CHECK();
}
void sort_rows_end(RowSort &job, const int32_t *words, hipStream_t s) {
  if (words[0] > 0) {
    k_sort_mid<<<(unsigned)ceil_div(words[0], kBlock / 64), kBlock, 0, s>>>(
        job.mid, words[0], job.rp, job.col, job.val);
    SA_LAUNCH_CHECK();
  }
  const int32_t nl = words[1];
  if (nl > 0) {
    k_sort_block<<<(unsigned)nl, kBlock, 0, s>>>(job.rows, job.rp, job.col, job.val);
    SA_LAUNCH_CHECK();
  }
  if (words[3] != 0) {  // a listed row has more than kSortBlock entries
    Arena &tmp = job.tmp;
    int64_t *caps = tmp.alloc<int64_t>(nl + 1);
    int64_t *goff = tmp.alloc<int64_t>(nl + 1);
    k_sort_caps<<<grid_for(nl), kBlock, 0, s>>>(nl, job.rows, job.rp, caps);
    SA_LAUNCH_CHECK();
    exclusive_scan_i64(caps, goff, nl, s);
    const int64_t gtot = read1(goff + nl, s);
    int32_t *gk = tmp.alloc<int32_t>(gtot > 0 ? gtot : 1);
    double *gv = tmp.alloc<double>(gtot > 0 ? gtot : 1);
    k_sort_long<<<(unsigned)nl, kBlock, 0, s>>>(job.rows, nl, job.rp, job.col, job.val, gk, gv,
                                                goff);
    SA_LAUNCH_CHECK();
  }
  job.tmp.release();
}
void sort_rows(int32_t n, const int32_t *rp, int32_t *col, double *val, hipStream_t s) {
  if (n <= 0) return;
  RowSort job;
  sort_rows_begin(n, rp, col, val, job, s);
  int32_t words[kRowSortWords];
  readback(words, job.words, sizeof(words), s);
  sort_rows_end(job, words, s);
}

// ---- transpose with values ---------------------------------------------------------------
// Every entry takes its place in its column's list as it is counted (rank), so the scatter
// needs no atomics of its own.  (3.4M entries: count 114 us, scatter 80; a thread per row of
// P scattering with an atomic per entry 178 us, and 600 us for 4.8M entries in 26-entry rows.)
__global__ void k_count_cols(int64_t nnz, const int32_t *col, int32_t *cnt, int32_t *rank) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < nnz) rank[e] = atomicAdd(&cnt[col[e]], 1);
}
void transpose(const Csr &P, Arena &ar, Csr &R, RowSort &sort, hipStream_t s) {
  const int32_t m = P.ncols;
  Arena tmp;
  tmp.stream = s;
  int32_t *cnt = tmp.alloc<int32_t>(m + 1);
  int32_t *rank = tmp.alloc<int32_t>(P.nnz);
  fill_i32(cnt, 0, m + 1, s);
  if (P.nnz > 0) {
    k_count_cols<<<grid_for(P.nnz), kBlock, 0, s>>>(P.nnz, P.col, cnt, rank);
    SA_LAUNCH_CHECK();
  }
  R.n = m;
  R.ncols = P.n;
  R.nnz = P.nnz;
  R.rp = ar.alloc<int32_t>(m + 1);
  exclusive_scan_i32(cnt, R.rp, m, s);
  R.col = ar.alloc<int32_t>(P.nnz);
  R.val = ar.alloc<double>(P.nnz);
  if (P.n > 0) {
    k_scatter_ranked<true><<<grid_for(P.n), kBlock, 0, s>>>(P.n, P.rp, P.col, P.val, rank, R.rp,
                                                            R.col, R.val);
    SA_LAUNCH_CHECK();
  }
  sort_rows_begin(m, R.rp, R.col, R.val, sort, s);
}

__global__ void k_inv_diag(int32_t n, const double *d, double *inv, int32_t *err) {
  SA_ROW_KERNEL_BEGIN(n)
  if (!(d[i] > 0.0)) atomicOr(err, 32);
  inv[i] = 1.0 / d[i];
}
void inv_diag(int32_t n, const double *dval, double *invD, int32_t *err, hipStream_t s) {
  if (n <= 0) return;
  k_inv_diag<<<grid_for(n), kBlock, 0, s>>>(n, dval, invD, err);
  SA_LAUNCH_CHECK();
}

}  // namespace sa
