// Sparse matrix-matrix product C = X*Y for the Galerkin operator (Sec. 1.1), in Gustavson
// order: every output entry C_ij accumulates X_ik*Y_kj over the row's entries k in ascending
// order, from 0.  No floating-point atomics: each output row's products are either ordered by
// (column, position), every run of equal columns summed in order by one lane, or added X entry
// by X entry, in order, to per-column accumulators of one wavefront.  Output rows are sorted;
// cancellations stay stored.
//
// Rows are binned by their product count T:
//   T <= 64      8, 16 or 32 lanes per row (8, 4 or 2 rows per wavefront), two products per
//                lane, sorted as below (k_esc_group);
//   T <= 1024    one wavefront per row, all products (2, 4, 8 or 16 per lane) sorted by
//                (column, position) in registers, each run added in order and written at its
//                rank (k_esc_sort), while 32 bits hold column and position;
//   T > 1024     a wavefront or a block per row, sums in LDS at the rank of their column
//                in the row (k_esc_rows);
//   otherwise    (wide keys; column windows of more than 8 tiles) one wavefront per row, sums
//                in an LDS hash table (k_esc_table) of 512 or 2048 slots, and a dense
//                accumulator in global memory for rows of more than 1536 distinct columns.
// Results go to per-row slots at the row's product offset (room for T >= distinct entries)
// and are compacted into CSR afterwards.
#include <algorithm>
#include <climits>
#include <cstdlib>
#include <cstring>

#include <mutex>

#include "kernels.hpp"

namespace sa {

constexpr int kWave = 64;
constexpr int kChunk = 1024;  // products per block-level chunk

// Bins by product count: <= 16, <= 32, <= 64 (rows sharing wavefronts), <= 128, <= 256, <= 512,
// <= 1024 (a wavefront per row, all products sorted at once), <= 2048, <= 8192, <= 32768, longer
// (sums in LDS).
constexpr int kBins = 11;
__device__ __forceinline__ int bin_of(int64_t T) {
  return T <= 16     ? 0
         : T <= 32   ? 1
         : T <= 64   ? 2
         : T <= 128  ? 3
         : T <= 256  ? 4
         : T <= 512  ? 5
         : T <= 1024 ? 6
         : T <= 2048 ? 7
         : T <= 8192 ? 8
         : T <= 32768 ? 9
                     : 10;
}

// A block lists its rows per bin: counted in LDS, each non-empty bin's share reserved with one
// global atomic (the order inside a list is immaterial: rows are independent).
__device__ __forceinline__ void bin_row(bool live, int32_t i, int64_t T, int32_t m,
                                        int32_t *lists, int32_t *counters) {
  __shared__ int32_t s_cnt[kBins], s_base[kBins];
  if (threadIdx.x < kBins) s_cnt[threadIdx.x] = 0;
  __syncthreads();
  const int bin = bin_of(T);
  int32_t local = 0;
  if (live) local = atomicAdd(&s_cnt[bin], 1);
  __syncthreads();
  if (threadIdx.x < kBins && s_cnt[threadIdx.x] > 0)
    s_base[threadIdx.x] = atomicAdd(&counters[threadIdx.x], s_cnt[threadIdx.x]);
  __syncthreads();
  if (live) lists[(int64_t)bin * m + s_base[bin] + local] = i;
}

// The rows' product counts, G lanes per row, four rows of a group at a time so that their loads
// go out together, and the rows' places in their bins' lists (a block has 256 rows: one atomic
// per bin and block).
template <int G>
__global__ __launch_bounds__(kBlock) void k_count_products(int32_t m,
                                                           const int32_t *__restrict__ xrp,
                                                           const int32_t *__restrict__ xcol,
                                                           const int32_t *__restrict__ yrp,
                                                           int64_t *__restrict__ cnt,
                                                           int32_t *lists, int32_t *counters) {
  constexpr int R = kBlock / G, U = 4;  // rows at once, rows per group and step
  __shared__ int32_t s_rp[kBlock + 1];
  __shared__ int64_t s_t[kBlock];
  const int t = threadIdx.x, lane = t % G;
  const int64_t r0 = (int64_t)blockIdx.x * kBlock;
  const int32_t nr = (int32_t)min<int64_t>(kBlock, (int64_t)m - r0);
  if (t <= nr) s_rp[t] = xrp[r0 + t];
  if (t == 0) s_rp[nr] = xrp[r0 + nr];  // nr can be kBlock: no thread t == nr
  __syncthreads();
  for (int32_t q = t / G; q < nr; q += U * R) {  // uniform over the group
    int32_t b[U], e[U], k[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int32_t r = q + u * R;
      b[u] = r < nr ? s_rp[r] + lane : 0;
      e[u] = r < nr ? s_rp[r + 1] : 0;
      k[u] = b[u] < e[u] ? xcol[b[u]] : -1;
    }
    int64_t sum[U];
#pragma unroll
    for (int u = 0; u < U; ++u) sum[u] = k[u] >= 0 ? yrp[k[u] + 1] - yrp[k[u]] : 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      for (int32_t c = b[u] + G; c < e[u]; c += G) {
        const int32_t j = xcol[c];
        sum[u] += yrp[j + 1] - yrp[j];
      }
#pragma unroll
      for (int off = G / 2; off >= 1; off >>= 1) sum[u] += __shfl_xor(sum[u], off, G);
      if (lane == 0 && q + u * R < nr) s_t[q + u * R] = sum[u];
    }
  }
  __syncthreads();
  const bool live = t < nr;
  if (live) cnt[r0 + t] = s_t[t];
  bin_row(live, live ? (int32_t)(r0 + t) : 0, live ? s_t[t] : 0, m, lists, counters);
}
// A wavefront per row (rows of more than 64 entries among them), binned by a launch of its own.
__global__ __launch_bounds__(kBlock) void k_count_products_w(int32_t m,
                                                             const int32_t *__restrict__ xrp,
                                                             const int32_t *__restrict__ xcol,
                                                             const int32_t *__restrict__ yrp,
                                                             int64_t *__restrict__ cnt) {
  const int64_t i = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / kWave;
  if (i >= m) return;  // uniform over the row's lanes
  const int lane = threadIdx.x % kWave;
  const int32_t end = xrp[i + 1];
  int64_t sum = 0;
  for (int32_t e = xrp[i] + lane; e < end; e += kWave) {
    const int32_t k = xcol[e];
    sum += yrp[k + 1] - yrp[k];
  }
#pragma unroll
  for (int off = kWave / 2; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, kWave);
  if (lane == 0) cnt[i] = sum;
}
// The products before each entry of the listed rows (a wavefront per row), for k_esc_dense.
__global__ __launch_bounds__(kWave) void k_row_prefix(const int32_t *rows, const int32_t *xrp,
                                                      const int32_t *xcol, const int32_t *yrp,
                                                      int32_t *xpref) {
  const int lane = threadIdx.x;
  const int32_t i = rows[blockIdx.x], end = xrp[i + 1];
  int32_t base = 0;
  for (int32_t c = xrp[i]; c < end; c += kWave) {
    const int32_t e = c + lane;
    int32_t len = 0;
    if (e < end) {
      const int32_t k = xcol[e];
      len = yrp[k + 1] - yrp[k];
    }
    const int32_t incl = group_prefix<64>(len, lane);
    if (e < end) xpref[e] = base + incl - len;
    base += __builtin_amdgcn_readlane(incl, 63);
  }
}

// ---- rows in a dense accumulator (the last resort) -------------------------------------------
__device__ inline int32_t find_entry(const int32_t *xpref, int32_t xb, int32_t xe, int32_t p) {
  // last e in [xb, xe) with xpref[e] <= p (entries with no products share a prefix value;
  // the last one holding p is the one whose Y row contains it).
  int32_t lo = xb, hi = xe - 1;
  while (lo < hi) {
    const int32_t mid = (lo + hi + 1) >> 1;
    if (xpref[mid] <= p) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

__device__ inline void bitonic_u64(uint64_t *a, int32_t L) {
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

__device__ inline int32_t next_pow2(int32_t x) {
  int32_t p = 1;
  while (p < x) p <<= 1;
  return p;
}

// Loads products c0 .. c0+L-1 of row i into sk (column << 32 | position) / sv and sorts sk;
// after it, equal columns are adjacent in position (= Gustavson) order.
__device__ inline void load_sorted_chunk(int32_t c0, int32_t L, int32_t xb, int32_t xe,
                                         const int32_t *xpref, const int32_t *xcol,
                                         const double *xval, const int32_t *yrp,
                                         const int32_t *ycol, const double *yval, uint64_t *sk,
                                         double *sv) {
  const int32_t Lp = next_pow2(L);
  for (int32_t q = threadIdx.x; q < Lp; q += blockDim.x) {
    if (q < L) {
      const int32_t p = c0 + q;
      const int32_t e = find_entry(xpref, xb, xe, p);
      const int32_t k = xcol[e];
      const int32_t yy = yrp[k] + (p - xpref[e]);
      sk[q] = ((uint64_t)(uint32_t)ycol[yy] << 32) | (uint32_t)q;
      sv[q] = xval[e] * yval[yy];
    } else {
      sk[q] = ~0ull;
    }
  }
  __syncthreads();
  bitonic_u64(sk, Lp);
}

__device__ inline uint32_t key_of(uint64_t x) { return (uint32_t)(x >> 32); }

// Rows with more distinct columns than the large LDS table takes and windows beyond the tile
// limit: a dense accumulator of ncols entries per block in global
// memory (first touch starts from 0, adds in position order as above); the result is
// extracted in column order by a block-wide scan of the touched flags.
__global__ __launch_bounds__(kBlock) void k_esc_dense(
    const int32_t *rows, int32_t nrows, const int32_t *xrp, const int32_t *xcol,
    const double *xval, const int32_t *xpref, const int32_t *yrp, const int32_t *ycol,
    const double *yval, int32_t ncols, const int64_t *poff, int32_t *ocol, double *oval,
    int32_t *ucnt, double *dacc, int32_t *dflag) {
  __shared__ uint64_t sk[kChunk];
  __shared__ double sv[kChunk];
  __shared__ int32_t s_scan[kBlock];
  __shared__ int32_t s_base;
  const int tid = threadIdx.x;
  double *acc = dacc + (int64_t)blockIdx.x * ncols;
  int32_t *flag = dflag + (int64_t)blockIdx.x * ncols;
  for (int32_t slot = blockIdx.x; slot < nrows; slot += gridDim.x) {
    const int32_t i = rows[slot];
    const int32_t xb = xrp[i], xe = xrp[i + 1];
    const int64_t base = poff[i];
    const int32_t T = (int32_t)(poff[i + 1] - base);
    for (int32_t q = tid; q < ncols; q += kBlock) flag[q] = 0;
    __syncthreads();
    for (int32_t c0 = 0; c0 < T; c0 += kChunk) {
      const int32_t L = min(kChunk, T - c0);
      load_sorted_chunk(c0, L, xb, xe, xpref, xcol, xval, yrp, ycol, yval, sk, sv);
      for (int32_t r = tid; r < L; r += kBlock) {
        const uint32_t key = key_of(sk[r]);
        if (r > 0 && key_of(sk[r - 1]) == key) continue;
        double a = flag[key] ? acc[key] : 0.0;
        for (int32_t q = r; q < L && key_of(sk[q]) == key; ++q) a += sv[(uint32_t)sk[q]];
        acc[key] = a;
        flag[key] = 1;
      }
      __syncthreads();
    }
    if (tid == 0) s_base = 0;
    __syncthreads();
    for (int32_t c0 = 0; c0 < ncols; c0 += kBlock) {
      const int32_t c = c0 + tid;
      const int32_t f = (c < ncols) ? flag[c] : 0;
      s_scan[tid] = f;
      __syncthreads();
      for (int off = 1; off < kBlock; off <<= 1) {
        const int32_t add = (tid >= off) ? s_scan[tid - off] : 0;
        __syncthreads();
        s_scan[tid] += add;
        __syncthreads();
      }
      if (f) {
        const int32_t pos = s_base + s_scan[tid] - 1;
        ocol[base + pos] = c;
        oval[base + pos] = acc[c];
      }
      __syncthreads();
      if (tid == kBlock - 1) s_base += s_scan[kBlock - 1];
      __syncthreads();
    }
    if (tid == 0) ucnt[i] = s_base;
    __syncthreads();
  }
}

// One wavefront's LDS operations complete in its program order: between its lanes only the
// compiler has to keep that order.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// ---- wavefront-per-row bins (T > 64) ------------------------------------------------------
// A wavefront goes over the products X_ik Y_kj of a row in Gustavson order, 64 to a step
// (product p0 + 64 d + lane in step d), S steps' loads issued together: f gets each step's X
// entry (ed, numbering the chunk's non-empty Y rows; -1 past the end) and that of its last
// product, the columns and, with VALS, the products; it returns false to stop.  The X entries
// are taken 64 at a time (chunks first, first + stride, ...).  Each non-empty Y row sets the
// bit of its first product in its step's 64-bit word, and a lane's entry is the number of bits
// up to its own: the words of S steps are one LDS atomic per entry, whatever the row lengths.
// With clip, only the products with columns cA <= j < cB (Y's rows are sorted).
struct ProductStage {
  uint64_t start[8];
  int32_t off[64];
  double a[64];
};
// [b, e) to the entries with columns cA <= j < cB: both ends searched at once.
__device__ __forceinline__ void clip_cols(const int32_t *ycol, int32_t &b, int32_t &e,
                                          int32_t cA, int32_t cB) {
  int32_t h1 = e, l2 = b;
  while (b < h1 || l2 < e) {
    const int32_t m1 = (b + h1) >> 1, m2 = (l2 + e) >> 1;
    const int32_t c1 = b < h1 ? ycol[m1] : cA, c2 = l2 < e ? ycol[m2] : cB;
    if (c1 < cA) b = m1 + 1;
    else h1 = m1;
    if (c2 < cB) l2 = m2 + 1;
    else e = m2;
  }
}
template <int S, bool VALS, typename F>
__device__ __forceinline__ void row_products(ProductStage &st, int lane, int32_t xb, int32_t xe,
                                             int32_t first, int32_t stride, bool clip,
                                             int32_t cA, int32_t cB, const int32_t *xcol,
                                             const double *xval, const int32_t *yrp,
                                             const int32_t *ycol, const double *yval, F f) {
  static_assert(S <= 8, "a start word per step");
  // the next chunk's Y row bounds and the one after's X entries are loaded a chunk ahead
  const int32_t hop = 64 * stride;
  int32_t e0 = xb + 64 * first;
  auto entry = [&](int32_t e, int32_t &k, double &a) {
    k = -1;
    a = 0.0;
    if (e < xe) {
      k = xcol[e];
      if (VALS) a = xval[e];
    }
  };
  auto bounds = [&](int32_t k, int32_t &b, int32_t &e) {
    b = e = 0;
    if (k >= 0) {
      b = yrp[k];
      e = yrp[k + 1];
    }
  };
  int32_t k1, k2, yb1, ye1;
  double a1, a2;
  entry(e0 + lane, k1, a1);
  entry(e0 + hop + lane, k2, a2);
  bounds(k1, yb1, ye1);
  int32_t at = 0;  // the chunk's first position
  for (; e0 < xe; e0 += hop) {
    int32_t ys = yb1, ye = ye1;
    const double a = a1;
    a1 = a2;
    bounds(k2, yb1, ye1);
    entry(e0 + 2 * hop + lane, k2, a2);
    if (clip) clip_cols(ycol, ys, ye, cA, cB);
    const int32_t len = ye - ys;
    const int32_t incl = group_prefix<64>(len, lane);
    const int32_t tot = __builtin_amdgcn_readlane(incl, 63);
    const int32_t ex = incl - len;  // this entry's first product within the chunk
    const unsigned long long some = __ballot(len > 0);
    wave_sync();  // the previous chunk's reads come before
    if (len > 0) {
      const int32_t g = __popcll(some & ((1ull << lane) - 1ull));
      st.off[g] = ys - ex;
      if (VALS) st.a[g] = a;
    }
    int32_t seen = 0;  // entries that start before the step
    for (int32_t g0 = 0; g0 < tot; g0 += 64 * S) {
      if (lane < S) st.start[lane] = 0;
      wave_sync();
      if (len > 0 && ex >= g0 && ex < g0 + 64 * S)
        atomicOr((unsigned long long *)&st.start[(ex - g0) >> 6], 1ull << ((ex - g0) & 63));
      wave_sync();
      uint32_t wl[S], wh[S];
#pragma unroll
      for (int d = 0; d < S; ++d) {
        wl[d] = (uint32_t)st.start[d];
        wh[d] = (uint32_t)(st.start[d] >> 32);
      }
      int32_t ed[S], last[S], qd[S];
#pragma unroll
      for (int d = 0; d < S; ++d) {
        const uint64_t w = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)wh[d]) << 32 |
                           (uint32_t)__builtin_amdgcn_readfirstlane((int)wl[d]);
        const uint64_t up = w >> 1;  // bits 1 .. lane of w are those below `lane` of this
        const int32_t g = __builtin_amdgcn_mbcnt_hi(
            (uint32_t)(up >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)up, seen - 1 + (int)(w & 1)));
        seen += __popcll(w);
        last[d] = seen - 1;
        const int32_t p = g0 + 64 * d + lane;
        ed[d] = p < tot ? g : -1;
        qd[d] = p < tot ? st.off[g] + p : 0;  // lanes past the end load Y's first entry
      }
      int32_t cd[S];
      double vd[S];
#pragma unroll
      for (int d = 0; d < S; ++d) {
        cd[d] = ycol[qd[d]];
        if (VALS) vd[d] = yval[qd[d]];
      }
      if (VALS) {
#pragma unroll
        for (int d = 0; d < S; ++d)
          if (ed[d] >= 0) vd[d] = st.a[ed[d]] * vd[d];
      }
      if (!f(at + g0, ed, last, cd, vd)) return;
    }
    at += tot;
  }
}

// Both values of a pair of lanes (lane, lane ^ J), in either order.  J = 1, 2: a quad permutation
// (DPP); J = 4, 8: a row shift by J toward the lower lanes (row_shl, lane i reads i + J) for the
// lower lanes of a pair, one toward the higher lanes for the others (by bank masks); J = 16, 32: a
// swap of rows of 16 or of 32.
struct Pair {
  uint32_t a, b;
};
template <int J>
__device__ __forceinline__ Pair xor_pair(uint32_t v) {
  if constexpr (J == 1) {
    return {v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, false)};  // [1,0,3,2]
  } else if constexpr (J == 2) {
    return {v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, false)};  // [2,3,0,1]
  } else if constexpr (J == 4 || J == 8) {
    constexpr int low = J == 4 ? 0x5 : 0x3;  // banks (of 4 lanes) of the pairs' lower lanes
    const int x = __builtin_amdgcn_update_dpp((int)v, (int)v, 0x100 + J, 0xF, low, false);
    return {v, (uint32_t)__builtin_amdgcn_update_dpp(x, (int)v, 0x110 + J, 0xF, 0xF ^ low, false)};
  } else if constexpr (J == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return {r[0], r[1]};
  } else {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return {r[0], r[1]};
  }
}
// The smaller of a and b where e is 0, the larger where it is all ones (one median of three).
__device__ __forceinline__ uint32_t pick(uint32_t a, uint32_t b, uint32_t e) {
  return max(min(a, b), min(max(a, b), e));
}
// 0 in the lanes that keep the smaller of a pair (lane, lane ^ J), all ones in the others.
template <int J>
__device__ __forceinline__ uint32_t upper_of(int lane) {
  return (lane & J) ? ~0u : 0u;
}
// Value of lane (lane ^ M), M = 2^m - 1, the partner in a merge's first step (1, 3: quad
// permutations; 7, 15: the mirrors within 8 and 16 lanes; 31, 63: the mirror and row swaps).
template <int M>
__device__ __forceinline__ uint32_t flip_lane(uint32_t v, int lane) {
  if constexpr (M == 1)
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, false);  // [1,0,3,2]
  else if constexpr (M == 3)
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x1B, 0xF, 0xF, false);  // [3,2,1,0]
  else if constexpr (M == 7)
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, false);  // half mirror
  else if constexpr (M == 15)
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xF, 0xF, false);  // row mirror
  else if constexpr (M == 31) {
    const Pair p = xor_pair<16>(flip_lane<15>(v, lane));
    return (lane & 16) ? p.a : p.b;
  } else {
    const Pair p = xor_pair<32>(flip_lane<31>(v, lane));
    return (lane & 32) ? p.a : p.b;
  }
}
// Ascending bitonic sort of N keys, element gl * P + q in k[q] of the gl-th of N / P lanes (a
// power of two, aligned; other groups sort their own).  Merges start by comparing mirrored
// elements, so every comparison puts the smaller key at the lower index: within a lane a
// minimum and a maximum, across lanes a minimum or a maximum by a bit of the lane.
template <int P, int J>
__device__ __forceinline__ void sort_halves(uint32_t (&k)[P], int lane) {
  if constexpr (J >= P) {
    constexpr int L = J / P;
    const uint32_t up = upper_of<L>(lane);
#pragma unroll
    for (int q = 0; q < P; ++q) {
      const Pair p = xor_pair<L>(k[q]);
      k[q] = pick(p.a, p.b, up);
    }
  } else {
#pragma unroll
    for (int q = 0; q < P; ++q)
      if ((q & J) == 0) {
        const uint32_t x = k[q], y = k[q | J];
        k[q] = min(x, y);
        k[q | J] = max(x, y);
      }
  }
  if constexpr (J > 1) sort_halves<P, J / 2>(k, lane);
}
template <int P, int N = 64 * P, int K = 2>
__device__ __forceinline__ void sort_keys(uint32_t (&k)[P], int lane) {
  if constexpr (K <= P) {
#pragma unroll
    for (int q = 0; q < P; ++q) {
      const int o = q ^ (K - 1);
      if (q < o) {
        const uint32_t x = k[q], y = k[o];
        k[q] = min(x, y);
        k[o] = max(x, y);
      }
    }
  } else {
    constexpr int L = K / P;
    const uint32_t up = upper_of<L / 2>(lane);
    uint32_t o[P];
#pragma unroll
    for (int q = 0; q < P; ++q) o[q] = flip_lane<L - 1>(k[P - 1 - q], lane);
#pragma unroll
    for (int q = 0; q < P; ++q) k[q] = pick(k[q], o[q], up);
  }
  if constexpr (K > 2) sort_halves<P, K / 4>(k, lane);
  if constexpr (K < N) sort_keys<P, N, K * 2>(k, lane);
}

// ---- G lanes per row (T <= 2 G), 64/G rows per wavefront -------------------------------------
// A wavefront takes 64/G rows, G lanes each, two products per lane: short rows share a
// wavefront instead of leaving most of its lanes idle, and the more rows a wavefront holds,
// the more of their (dependent) loads are in flight together.  Per row: the X entries G at a
// time, each non-empty Y row's first product a bit of the chunk's word, a product's entry the
// bits up to its own; the (column, position) keys sorted in registers (sort_keys); and each
// run of equal columns added in position order by the lane that holds its first key.  The chunk
// loop runs to the longest X row of the wavefront.  The ranks by comparing every pair of
// products in LDS, before, made the instructions the bound: 524K rows of 33..64 products 372 us,
// now 190, 477K of 17..32 150 -> 92; 1.6M of at most 16 210 -> 161, where the chain of loads is.
template <int G>
__global__ __launch_bounds__(kWave) void k_esc_group(
    const int32_t *rows, int32_t nrows, const int32_t *xrp, const int32_t *xcol,
    const double *xval, const int32_t *yrp, const int32_t *ycol, const double *yval,
    const int64_t *poff, int32_t *ocol, double *oval, int32_t *ucnt) {
  constexpr int N = 2 * G;  // products of one row at most
  constexpr int B = G == 8 ? 4 : G == 16 ? 5 : 6;
  constexpr uint32_t kNone = ~0u;
  static_assert(N == 1 << B, "a position per key");
  __shared__ uint32_t s_k[2 * kWave];
  __shared__ double s_v[2 * kWave];
  __shared__ unsigned long long s_start[kWave / G];
  __shared__ int32_t s_off[kWave];
  __shared__ double s_a[kWave];
  const int lane = threadIdx.x;
  const int gl = lane % G, gb = lane - gl;  // lane in the group, the group's first lane
  const int pb = gb * 2;                    // the row's product slots
  // consecutive rows share the Y rows of their neighbours: each XCD takes a contiguous run of
  // the bin's rows (bins list rows roughly in row order), so those reads hit its L2
  const int64_t r64 = (int64_t)xcd_block(blockIdx.x, gridDim.x) * (kWave / G) + lane / G;
  const bool live = r64 < nrows;
  const int32_t i = live ? rows[r64] : 0;
  const int64_t base = live ? poff[i] : 0;
  const int32_t xb = live ? xrp[i] : 0, xe = live ? xrp[i + 1] : 0;
  int32_t nch = (xe - xb + G - 1) / G;  // chunks of this row; the wavefront runs the most
  for (int off = 32; off >= G; off >>= 1) nch = max(nch, __shfl_xor(nch, off, kWave));
  // expansion in Gustavson order: position = products of earlier X entries + offset in Y row
  int32_t filled = 0;
  for (int32_t c = 0; c < nch; ++c) {
    const int32_t e = xb + c * G + gl;
    int32_t len = 0, ys = 0;
    double a = 0.0;
    if (e < xe) {
      const int32_t k = xcol[e];
      a = xval[e];
      ys = yrp[k];
      len = yrp[k + 1] - ys;
    }
    const int32_t incl = group_prefix<G>(len, gl);
    const int32_t tot = __shfl(incl, G - 1, G), ex = incl - len;
    const unsigned long long some = __ballot(len > 0) >> gb & ((1ull << G) - 1ull);
    if (gl == 0) s_start[lane / G] = 0;
    wave_sync();  // (the previous chunk's reads come before, too)
    if (len > 0) {
      const int g = __popcll(some & ((1ull << gl) - 1ull));
      s_off[gb + g] = ys - ex;
      s_a[gb + g] = a;
      atomicOr(&s_start[lane / G], 1ull << ex);
    }
    wave_sync();
    const unsigned long long w = s_start[lane / G];
    int32_t g[2], cu[2];
    double yu[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int32_t p = gl + u * G;
      g[u] = gb + __popcll(w & ((2ull << p) - 1ull)) - 1;
      const int32_t q = p < tot ? s_off[g[u]] + p : 0;  // lanes past the end load Y's first entry
      cu[u] = ycol[q];
      yu[u] = yval[q];
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int32_t p = gl + u * G;
      if (p < tot) {
        s_k[pb + filled + p] = (uint32_t)cu[u] << B | (uint32_t)(filled + p);
        s_v[pb + filled + p] = s_a[g[u]] * yu[u];
      }
    }
    filled += tot;
  }
  for (int32_t p = filled + gl; p < N; p += G) s_k[pb + p] = kNone;
  wave_sync();
  uint32_t k[2] = {s_k[pb + gl], s_k[pb + G + gl]};
  sort_keys<2, N>(k, lane);
  double v[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) v[q] = k[q] == kNone ? 0.0 : s_v[pb + (k[q] & (N - 1))];
  wave_sync();
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    s_k[pb + 2 * gl + q] = k[q];
    s_v[pb + 2 * gl + q] = v[q];
  }
  const uint32_t below = (uint32_t)__shfl_up((int)k[1], 1, 64);
  const bool h0 = k[0] != kNone && (gl == 0 || (below >> B) != (k[0] >> B));
  const bool h1 = k[1] != kNone && (k[0] >> B) != (k[1] >> B);
  const int32_t nh = (int)h0 + (int)h1;
  const int32_t incl = group_prefix<G>(nh, gl);
  wave_sync();
  int32_t at = incl - nh;  // rank of the lane's next run
  if (h0 && (h1 || k[1] == kNone)) {  // a run of one
    ocol[base + at] = (int32_t)(k[0] >> B);
    oval[base + at] = 0.0 + v[0];
    ++at;
  }
  if (h1 || (h0 && k[1] != kNone)) {  // the lane's last run may go on in the next lanes' keys
    const uint32_t col = k[1] >> B;
    double sum = 0.0;
    if (!h1) sum += v[0];
    sum += v[1];
    for (int32_t r = 2 * gl + 2; r < N; ++r) {
      const uint32_t kr = s_k[pb + r];
      if (kr == kNone || (kr >> B) != col) break;
      sum += s_v[pb + r];
    }
    ocol[base + at] = (int32_t)col;
    oval[base + at] = sum;
  }
  if (live && gl == G - 1) ucnt[i] = incl;
}

// Products at their Gustavson positions p go to LDS as keys (column << B | p) and values; the
// keys are sorted in registers (P per lane); then each run of equal columns is added in
// position order by the lane that holds its first key: through that lane's registers, then on
// through LDS.  Runs are written at their rank.  The whole sort is 21 exchanges between lanes
// per key, most of them register moves (DPP), whatever the number of 64-product steps, and
// nothing has to be looked up or extracted afterwards: what bounds it is the row's chain of
// loads (X entries, their Y rows, the products) and, from 512 products on, the sort's own
// instructions (two to a key and exchange: a move and a median of three; 854 us in the first line
// below with a minimum, a maximum and a choice).  893K rows of 65..128 products: 739 us, against
// 2,130 with 64 products per step sorted and added to a hash table; 178K rows of 456 products
// 440 us against 2,800 with a 256-thread block sorting in LDS; R (A P) with 52K rows of
// 257..512: 141 us against 553 with the products added X entry by X entry to the rank of their
// column in the row.
template <int P>
__global__ __launch_bounds__(64) void k_esc_sort(
    const int32_t *rows, int32_t nrows, const int32_t *xrp, const int32_t *xcol,
    const double *xval, const int32_t *yrp, const int32_t *ycol, const double *yval,
    const int64_t *poff, int32_t *ocol, double *oval, int32_t *ucnt) {
  constexpr int N = 64 * P;
  constexpr int B = P == 2 ? 7 : P == 4 ? 8 : P == 8 ? 9 : 10;
  constexpr uint32_t kNone = ~0u;
  static_assert(N == 1 << B, "a position per key");
  __shared__ uint32_t s_k[N];
  __shared__ double s_v[N];
  __shared__ ProductStage st;
  const int lane = threadIdx.x;
  const int32_t slot = xcd_block(blockIdx.x, gridDim.x);
  if (slot >= nrows) return;  // block-uniform
  const int32_t i = rows[slot];
  const int64_t base = poff[i];
  const int32_t T = (int32_t)(poff[i + 1] - base);
  constexpr int S = P < 8 ? P : 8;
  row_products<S, true>(
      st, lane, xrp[i], xrp[i + 1], 0, 1, false, 0, 0, xcol, xval, yrp, ycol, yval,
      [&](int32_t p0, const int32_t (&ed)[S], const int32_t (&)[S], const int32_t (&cd)[S],
          const double (&vd)[S]) {
#pragma unroll
        for (int d = 0; d < S; ++d)
          if (ed[d] >= 0) {
            const int32_t p = p0 + 64 * d + lane;
            s_k[p] = ((uint32_t)cd[d] << B) | (uint32_t)p;
            s_v[p] = vd[d];
          }
        return true;
      });
  for (int32_t p = T + lane; p < N; p += 64) s_k[p] = kNone;
  __syncthreads();
  uint32_t k[P];
#pragma unroll
  for (int q = 0; q < P; ++q) k[q] = s_k[64 * q + lane];
  sort_keys<P>(k, lane);
  double v[P];
#pragma unroll
  for (int q = 0; q < P; ++q) v[q] = k[q] == kNone ? 0.0 : s_v[k[q] & (N - 1)];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < P; ++q) {
    s_k[lane * P + q] = k[q];
    s_v[lane * P + q] = v[q];
  }
  const uint32_t below = (uint32_t)__shfl_up((int)k[P - 1], 1, 64);
  bool head[P];
  int32_t nh = 0;
#pragma unroll
  for (int q = 0; q < P; ++q) {
    const uint32_t prev = q > 0 ? k[q > 0 ? q - 1 : 0] : below;
    head[q] = k[q] != kNone && ((lane == 0 && q == 0) || (prev >> B) != (k[q] >> B));
    nh += head[q];
  }
  int32_t incl = nh;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int32_t t = __shfl_up(incl, off, 64);
    if (lane >= off) incl += t;
  }
  __syncthreads();
  int32_t w = incl - nh;  // rank of the lane's next run
  bool open = false;
  double sum = 0.0;
  uint32_t col = 0;
#pragma unroll
  for (int q = 0; q < P; ++q) {
    if (head[q]) {
      if (open) {
        ocol[base + w] = (int32_t)col;
        oval[base + w] = sum;
        ++w;
      }
      open = true;
      col = k[q] >> B;
      sum = 0.0;
    }
    if (open && k[q] != kNone) sum += v[q];
  }
  if (open) {  // the lane's last run may go on in the next lanes' keys
    for (int32_t r = (lane + 1) * P; r < N && s_k[r] != kNone && (s_k[r] >> B) == col; ++r)
      sum += s_v[r];
    ocol[base + w] = (int32_t)col;
    oval[base + w] = sum;
  }
  if (lane == 63) ucnt[i] = incl;
}

// ---- sums in LDS, by the column's rank in the row (more than 1024 products) ------------------
// The columns of one Y row are distinct, so the adds of one X entry never meet, and the adds of
// successive entries are LDS atomics of one wavefront, which the LDS executes in the
// wavefront's order: every output entry receives its products in ascending k, from 0, and no
// add waits for the one before it.
__device__ __forceinline__ void lds_fadd(double *p, double v) {
  __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
constexpr int32_t kFewEntries = 16;
// The products of S steps added at their places x[d] < 2^bits of acc.  A step of a few X
// entries: one add per entry.  More: the lanes of equal places are found bit by bit with
// ballots, and the k-th product of every place is added k-th.
template <int S>
__device__ __forceinline__ void add_products(const int32_t (&ed)[S], const int32_t (&last)[S],
                                             const int32_t (&x)[S], int bits,
                                             const double (&vd)[S], double *acc) {
#pragma unroll
  for (int d = 0; d < S; ++d) {
    const int32_t g0 = __builtin_amdgcn_readfirstlane(ed[d]);
    if (g0 < 0) continue;  // wave-uniform: past the end
    if (last[d] - g0 < kFewEntries) {
      for (int32_t g = g0; g <= last[d]; ++g) {
        if (ed[d] == g) lds_fadd(&acc[x[d]], vd[d]);
        __builtin_amdgcn_wave_barrier();
      }
    } else {
      const bool live = ed[d] >= 0;
      unsigned long long same = __ballot(live);
      for (int b = 0; b < bits; ++b) {
        const bool one = (x[d] >> b) & 1;
        const unsigned long long ones = __ballot(one);
        same &= one ? ones : ~ones;
      }
      const int32_t k = (int32_t)__builtin_amdgcn_mbcnt_hi(
          (uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0));
      for (int32_t r = 0; __ballot(live && k >= r); ++r) {
        if (live && k == r) lds_fadd(&acc[x[d]], vd[d]);
        __builtin_amdgcn_wave_barrier();
      }
    }
  }
}
constexpr __device__ int log2_up(int32_t n) { return n > 1 ? 32 - __builtin_clz(n - 1) : 0; }

// A block of NW wavefronts per row.  The row's column window [first, last column] is taken in
// tiles of W columns: the columns that occur are marked in a bitmap, whose words carry the
// number of columns before them, and a product finds its sum at its column's rank.  The
// tile's columns are cut at bitmap words into ranges of at most RD ranks, one wavefront to a
// range, each going over the products of its range alone (searched in the sorted Y rows).
// Windows of more than maxw columns are listed in ovf[].  A rank needs 8 bytes of LDS per
// distinct column and a quarter byte per window column, where sums over the whole window (8
// bytes each) left five wavefronts to a CU: A P of 176K rows, 2,100 products over 74 columns
// each, 3,890 -> 1,480 us (250 G products/s); R (A P), 15.5K rows of 19K products, 1,650 ->
// 910; 18K rows of 570 entries or more with 2.5 products each, 1,140 -> 550, where 64
// products at a time were sorted.  What bounds it is the chain of loads and LDS operations of
// each 512 products (2 us a wavefront) where rows are few, the instructions of the adds where
// they are many.
constexpr int32_t kRowWhole = 2048;  // output columns
struct RowLists {  // the lists of several bins one after the other
  const int32_t *list[4];
  int32_t end[4];
};
template <int NW, int RD>
__global__ __launch_bounds__(64 * NW) void k_esc_rows(
    RowLists rows, const int32_t *xrp, const int32_t *xcol,
    const double *xval, const int32_t *yrp, const int32_t *ycol, const double *yval,
    const int64_t *poff, int32_t *ocol, double *oval, int32_t *ucnt, int32_t ncols, int32_t W,
    int64_t maxw, int32_t *ovf, int32_t *novf) {
  constexpr int S = 8;
  extern __shared__ double lds_dyn[];
  __shared__ ProductStage s_st[NW];
  __shared__ int32_t s_lo[NW], s_hi[NW], s_total;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int32_t slot = blockIdx.x;
  if (slot >= rows.end[3]) return;  // block-uniform
  int bin = 0;
  while (slot >= rows.end[bin]) ++bin;
  const int32_t i = rows.list[bin][slot - (bin > 0 ? rows.end[bin - 1] : 0)];
  double *acc = lds_dyn + wave * RD;
  uint2 *word = reinterpret_cast<uint2 *>(lds_dyn + NW * RD);
  ProductStage &st = s_st[wave];
  const int64_t base = poff[i];
  const int32_t xb = xrp[i], xe = xrp[i + 1];
  const bool whole = ncols <= kRowWhole;  // a few words: no search for the window
  int32_t lo = whole ? 0 : INT_MAX, hi = whole ? ncols - 1 : -1;
  for (int32_t e = xb + (int32_t)threadIdx.x; e < xe && !whole; e += 64 * NW) {
    const int32_t k = xcol[e];
    const int32_t b = yrp[k], en = yrp[k + 1];
    if (b < en) {
      lo = min(lo, ycol[b]);
      hi = max(hi, ycol[en - 1]);
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    lo = min(lo, __shfl_xor(lo, off, 64));
    hi = max(hi, __shfl_xor(hi, off, 64));
  }
  if (NW > 1) {
    if (lane == 0) {
      s_lo[wave] = lo;
      s_hi[wave] = hi;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NW; ++q) {
      lo = min(lo, s_lo[q]);
      hi = max(hi, s_hi[q]);
    }
  }
  if ((int64_t)hi - lo >= maxw) {  // block-uniform
    if (threadIdx.x == 0) ovf[atomicAdd(novf, 1)] = i;
    return;
  }
  int32_t at = 0;  // the row's columns before the tile
  for (int64_t tile = lo; tile <= hi; tile += W) {
    const int32_t cA = (int32_t)tile, cB = (int32_t)min((int64_t)hi + 1, tile + W);
    const int32_t nw = (cB - cA + 31) >> 5;
    const bool tiles = hi - lo >= W;
    __syncthreads();  // the previous tile's words are read
    for (int32_t w = threadIdx.x; w < nw; w += 64 * NW) word[w].x = 0;
    __syncthreads();
    row_products<S, false>(
        st, lane, xb, xe, wave, NW, tiles, cA, cB, xcol, xval, yrp, ycol, yval,
        [&](int32_t, const int32_t (&ed)[S], const int32_t (&)[S], const int32_t (&cd)[S],
            const double (&)[S]) {
          uint32_t b[S];
#pragma unroll
          for (int d = 0; d < S; ++d) b[d] = ed[d] >= 0 ? word[(cd[d] - cA) >> 5].x : ~0u;
#pragma unroll
          for (int d = 0; d < S; ++d) {
            const uint32_t bit = 1u << ((cd[d] - cA) & 31);
            if (!(b[d] & bit)) atomicOr(&word[(cd[d] - cA) >> 5].x, bit);
          }
          return true;
        });
    __syncthreads();
    if (wave == 0) {
      int32_t before = 0;
      for (int32_t w0 = 0; w0 < nw; w0 += 64) {
        const int32_t n = w0 + lane < nw ? __popc(word[w0 + lane].x) : 0;
        const int32_t incl = group_prefix<64>(n, lane);
        if (w0 + lane < nw) word[w0 + lane].y = (uint32_t)(before + incl - n);
        before += __builtin_amdgcn_readlane(incl, 63);
      }
      if (lane == 0) s_total = before;
    }
    __syncthreads();
    const int32_t D = s_total;
    // a word belongs to the range of its first rank: up to 31 ranks more than `per`
    const int32_t per = NW == 1 ? RD - 31 : min(RD - 31, max(16, (D + NW - 1) / NW));
    const int32_t nr = (D + per - 1) / per;
    for (int32_t j = wave; j < nr; j += NW) {
      int32_t wA = 0, wB = nw;
      if (nr > 1) {
        wA = wB = 0;
        for (int32_t w0 = 0; w0 < nw; w0 += 64) {
          const int32_t r = w0 + lane < nw ? (int32_t)word[w0 + lane].y : INT_MAX;
          wA += __popcll(__ballot(r < j * per));
          wB += __popcll(__ballot(r < (j + 1) * per));
        }
      }
      if (wA >= wB) continue;
      const int32_t r0 = (int32_t)word[wA].y, r1 = wB < nw ? (int32_t)word[wB].y : D;
      const int bits = log2_up(r1 - r0);
      wave_sync();
      for (int32_t r = lane; r < r1 - r0; r += 64) acc[r] = 0.0;
      wave_sync();
      row_products<S, true>(
          st, lane, xb, xe, 0, 1, tiles || nr > 1, cA + 32 * wA, wB < nw ? cA + 32 * wB : cB,
          xcol, xval, yrp, ycol, yval,
          [&](int32_t, const int32_t (&ed)[S], const int32_t (&last)[S],
              const int32_t (&cd)[S], const double (&vd)[S]) {
            int32_t x[S];
#pragma unroll
            for (int d = 0; d < S; ++d) {
              const int32_t c = ed[d] >= 0 ? cd[d] - cA : 32 * wA;
              const uint2 b = word[c >> 5];
              x[d] = (int32_t)b.y + __popc(b.x & ((1u << (c & 31)) - 1u)) - r0;
            }
            add_products<S>(ed, last, x, bits, vd, acc);
            return true;
          });
      wave_sync();
      for (int32_t r = lane; r < r1 - r0; r += 64) oval[base + at + r0 + r] = acc[r];
      for (int32_t w = wA + lane; w < wB; w += 64) {
        uint32_t b = word[w].x;
        int64_t to = base + at + word[w].y;
        for (; b != 0; b &= b - 1) ocol[to++] = cA + 32 * w + __ffs(b) - 1;
      }
    }
    at += D;
  }
  if (threadIdx.x == 0) ucnt[i] = at;
}

// ---- sums in LDS, in a hash table (wide keys; windows too wide for the ranks) ----------------
// One wavefront per row, an open-addressing table of H slots: the low five bits of a column
// stay (columns next to each other, on different banks), its block of 32 is hashed.  A row
// with more than 3/4 H distinct columns is listed in ovf[].  At the end the row's columns are
// sorted in registers and looked up again.
template <int H>
__device__ __forceinline__ int32_t home_slot(int32_t col) {
  const uint32_t block = ((uint32_t)col >> 5) * 2654435761u;
  return (int32_t)(((block >> 12) << 5 | ((uint32_t)col & 31u)) & (uint32_t)(H - 1));
}
constexpr int32_t kProbe = 37;  // odd: a probe sequence meets every slot
// The row's nd <= 64 P columns in ascending order, each with its sum.
template <int H, int P>
__device__ __forceinline__ void write_sorted(int lane, int32_t nd, const int32_t *key,
                                             const uint16_t *list, const double *acc,
                                             int32_t *ocol, double *oval) {
  uint32_t k[P];
#pragma unroll
  for (int q = 0; q < P; ++q) {
    const int32_t r = 64 * q + lane;
    k[q] = r < nd ? (uint32_t)key[list[r]] : ~0u;
  }
  sort_keys<P>(k, lane);
#pragma unroll
  for (int q = 0; q < P; ++q) {
    const int32_t r = lane * P + q;
    if (r < nd) {
      const int32_t c = (int32_t)k[q];
      int32_t x = home_slot<H>(c);
      while (key[x] != c) x = (x + kProbe) & (H - 1);  // it is in the table
      ocol[r] = c;
      oval[r] = acc[x];
    }
  }
}
template <int H>
__global__ __launch_bounds__(64) void k_esc_table(
    const int32_t *rows, int32_t nrows, const int32_t *xrp, const int32_t *xcol,
    const double *xval, const int32_t *yrp, const int32_t *ycol, const double *yval,
    const int64_t *poff, int32_t *ocol, double *oval, int32_t *ucnt, int32_t *ovf,
    int32_t *novf) {
  constexpr int S = 8;
  __shared__ double acc[H];
  __shared__ int32_t key[H];
  __shared__ uint16_t list[H];
  __shared__ ProductStage st;
  const int lane = threadIdx.x;
  const int32_t slot = xcd_block(blockIdx.x, gridDim.x);
  if (slot >= nrows) return;  // block-uniform
  const int32_t i = rows[slot];
  const int64_t base = poff[i];
  for (int32_t c = lane; c < H; c += 64) {
    key[c] = -1;
    acc[c] = 0.0;
  }
  wave_sync();
  int32_t nd = 0;
  bool over = false;
  row_products<S, true>(
      st, lane, xrp[i], xrp[i + 1], 0, 1, false, 0, 0, xcol, xval, yrp, ycol, yval,
      [&](int32_t, const int32_t (&ed)[S], const int32_t (&last)[S], const int32_t (&cd)[S],
          const double (&vd)[S]) {
        int32_t x[S], kx[S];
#pragma unroll
        for (int d = 0; d < S; ++d) {
          x[d] = home_slot<H>(cd[d]);
          kx[d] = key[x[d]];
        }
        bool full = false;
#pragma unroll
        for (int d = 0; d < S; ++d) {
          bool fresh = false;
          if (ed[d] >= 0 && kx[d] != cd[d]) {
            int32_t t = 0;
            for (; t < H; ++t) {
              const int32_t old = atomicCAS(&key[x[d]], -1, cd[d]);
              fresh = old == -1;
              if (fresh || old == cd[d]) break;
              x[d] = (x[d] + kProbe) & (H - 1);
            }
            full |= t == H;  // every slot holds another column
          }
          const unsigned long long bm = __ballot(fresh);
          if (fresh) list[nd + __popcll(bm & ((1ull << lane) - 1ull))] = (uint16_t)x[d];
          nd += __popcll(bm);
        }
        over = 4 * nd > 3 * H || __ballot(full) != 0;  // wave-uniform
        if (over) return false;
        add_products<S>(ed, last, x, log2_up(H), vd, acc);
        return true;
      });
  if (over) {
    if (lane == 0) ovf[atomicAdd(novf, 1)] = i;
    return;
  }
  wave_sync();
  if (nd <= 256)
    write_sorted<H, 4>(lane, nd, key, list, acc, ocol + base, oval + base);
  else if (H <= 512 || nd <= 512)
    write_sorted<H, 8>(lane, nd, key, list, acc, ocol + base, oval + base);
  else if constexpr (H > 512) {
    if (nd <= 1024)
      write_sorted<H, 16>(lane, nd, key, list, acc, ocol + base, oval + base);
    else
      write_sorted<H, 32>(lane, nd, key, list, acc, ocol + base, oval + base);
  }
  if (lane == 0) ucnt[i] = nd;
}

// C's rows from their slots: a wavefront takes R consecutive rows, whose entries are one
// contiguous run of C; lanes copy consecutive entries, eight each at a time, finding their rows
// by binary search over the row starts held in LDS.  (One entry at a time left the copy at its
// loads' latency, and rows of 20 entries or more searched all row starts in memory: 600K rows of
// 16, 117 -> 90 us; 89K of 62, 197 -> 34.)
template <int R>
__global__ __launch_bounds__(kBlock) void k_compact(int32_t m, const int64_t *__restrict__ poff,
                                                    const int32_t *__restrict__ crp,
                                                    const int32_t *__restrict__ ocol,
                                                    const double *__restrict__ oval,
                                                    int32_t *__restrict__ ccol,
                                                    double *__restrict__ cval) {
  constexpr int NW = kBlock / 64, U = 8;
  __shared__ int32_t s_rp[NW][R + 1];
  __shared__ int64_t s_shift[NW][R];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t r0 = ((int64_t)blockIdx.x * NW + w) * R;  // this wavefront's first row
  if (lane < R) {
    const int64_t row = r0 + lane;
    const int32_t rb = crp[row < m ? row : m];  // rows past the end: empty, at C's end
    s_rp[w][lane] = rb;
    s_shift[w][lane] = (row < m ? poff[row] : 0) - rb;
  }
  if (lane == 0) s_rp[w][R] = crp[r0 + R < m ? r0 + R : m];
  __syncthreads();
  const int32_t d0 = s_rp[w][0], d1 = s_rp[w][R];
  for (int32_t d = d0 + lane; d < d1; d += 64 * U) {
    int32_t c[U];
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int32_t e = min(d + 64 * u, d1 - 1);  // past the run: its last entry again
      int lo = 0;  // last row r with s_rp[r] <= e (empty rows share starts)
#pragma unroll
      for (int step = R / 2; step >= 1; step >>= 1)
        if (s_rp[w][lo + step] <= e) lo += step;
      const int64_t src = s_shift[w][lo] + e;
      c[u] = ocol[src];
      v[u] = oval[src];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (d + 64 * u < d1) {
        ccol[d + 64 * u] = c[u];
        cval[d + 64 * u] = v[u];
      }
  }
}

__global__ void k_put_total(const int64_t *src, int64_t *dst) { *dst = *src; }

// Bins the rows counted by k_count_products_w (one block per row there).
__global__ __launch_bounds__(kBlock) void k_bin_rows(int32_t m, const int64_t *poff,
                                                     int32_t *lists, int32_t *counters) {
  const int64_t i64 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool live = i64 < m;
  const int32_t i = live ? (int32_t)i64 : 0;
  bin_row(live, i, live ? poff[i + 1] - poff[i] : 0, m, lists, counters);
}

// Column tiles that a long row's window may take (environment variable
// SAAMG_SPGEMM_MAX_TILES; 0 sends the long rows to the large hash table).
static int32_t max_tiles() {
  const char *e = std::getenv("SAAMG_SPGEMM_MAX_TILES");
  return e ? std::atoi(e) : 8;
}

// SAAMG_SPGEMM_KEY64=1 takes the hash table where the sort's keys would hold the columns too.
static bool keys64() {
  const char *e = std::getenv("SAAMG_SPGEMM_KEY64");
  return e && std::atoi(e) != 0;
}

void spgemm(const Csr &X, const Csr &Y, Arena &ar, Csr &C, hipStream_t s, int32_t xmax,
            bool max_row, const ReadAlong &along) {
  const int32_t m = X.n;
  C.n = m;
  C.ncols = Y.ncols;
  C.maxrow = -1;
  Arena tmp;
  tmp.stream = s;
  int64_t *cnt = tmp.alloc<int64_t>(m + 1);
  int64_t *poff = tmp.alloc<int64_t>(m + 1);
  int32_t *lists = tmp.alloc<int32_t>(kBins * (int64_t)(m > 0 ? m : 1));
  // kBins bin sizes, the counts of rows left to the large hash table and by it, then (8-byte
  // aligned) the product total in 64 bits
  constexpr int kTotalAt = (kBins + 3) & ~1;
  int32_t *counters = tmp.alloc<int32_t>(kTotalAt + 2);
  fill_i32(counters, 0, kBins + 2, s);
  // rows of up to 64 entries: 8, 16 or 32 lanes each, counted and binned in one launch; longer
  // ones a wavefront each, binned after the scan (a block of few rows would add its atomics to
  // the bins' counters too often).  970K rows of 26 entries: 261 us and 48 for the binning with
  // the products before each entry written out too, now 103; 600K of 16, a thread per row, 117,
  // now 56
  if (xmax < 0) xmax = m > 0 ? (X.maxrow >= 0 ? X.maxrow : max_row_length(m, X.rp, s)) : 0;
  const bool wave_count = m > 0 && xmax > 64;
  auto count_rows = [&](auto gc) {
    constexpr int G = decltype(gc)::value;
    k_count_products<G><<<grid_for(m), kBlock, 0, s>>>(m, X.rp, X.col, Y.rp, cnt, lists,
                                                      counters);
  };
  if (wave_count)
    k_count_products_w<<<grid_for((int64_t)m * kWave), kBlock, 0, s>>>(m, X.rp, X.col, Y.rp, cnt);
  else if (m > 0 && X.nnz > 20 * (int64_t)m)
    count_rows(std::integral_constant<int, 32>{});
  else if (m > 0 && X.nnz > 10 * (int64_t)m)
    count_rows(std::integral_constant<int, 16>{});
  else if (m > 0)
    count_rows(std::integral_constant<int, 8>{});
  SA_LAUNCH_CHECK();
  exclusive_scan_i64(cnt, poff, m, s);
  if (wave_count) {
    k_bin_rows<<<grid_for(m), kBlock, 0, s>>>(m, poff, lists, counters);
    SA_LAUNCH_CHECK();
  }
  // the bin sizes and the product total in one readback
  k_put_total<<<1, 1, 0, s>>>(poff + m, (int64_t *)(counters + kTotalAt));
  SA_LAUNCH_CHECK();
  constexpr int kAlong = 8;
  int32_t hc[kTotalAt + 2 + kAlong];
  WordRuns runs;
  runs.add(counters, kTotalAt + 2);
  if (along.words > 0) runs.add(along.dev, std::min(along.words, kAlong));
  readback_runs(hc, runs, s);
  if (along.words > 0)
    std::memcpy(along.host, hc + kTotalAt + 2, 4 * std::min(along.words, kAlong));
  int64_t total = 0;
  std::memcpy(&total, hc + kTotalAt, sizeof(total));
  int32_t *ocol = tmp.alloc<int32_t>(total > 0 ? total : 1);
  double *oval = tmp.alloc<double>(total > 0 ? total : 1);
  int32_t *ucnt = tmp.alloc<int32_t>(m + 1);
  // the sorts' 32-bit keys hold 28 bits of column at 16 products, 22 at 1024; wider outputs (and
  // SAAMG_SPGEMM_KEY64=1) take the hash table
  auto wide = [&](int bin) { return keys64() || Y.ncols >= (1 << (28 - bin)); };
  int32_t nhash = 0;
  for (int bin = 0; bin < 7; ++bin)
    if (wide(bin)) nhash += hc[bin];
  const int32_t nlong = hc[7] + hc[8] + hc[9] + hc[10];
  int32_t *over1 = nullptr, *nover = counters + kBins;
  if (nhash + nlong > 0) over1 = tmp.alloc<int32_t>(nhash + nlong);
  for (int bin = 0; bin < 7; ++bin) {
    const int32_t nr = hc[bin];
    if (nr == 0) continue;
    const int32_t *rows = lists + bin * (int64_t)m;
    auto group = [&](auto gc) {
      constexpr int G = decltype(gc)::value;
      k_esc_group<G><<<(unsigned)ceil_div(nr, kWave / G), kWave, 0, s>>>(
          rows, nr, X.rp, X.col, X.val, Y.rp, Y.col, Y.val, poff, ocol, oval, ucnt);
    };
    auto sort = [&](auto pc) {
      constexpr int P = decltype(pc)::value;
      k_esc_sort<P><<<(unsigned)nr, 64, 0, s>>>(rows, nr, X.rp, X.col, X.val, Y.rp, Y.col, Y.val,
                                               poff, ocol, oval, ucnt);
    };
    if (wide(bin))
      k_esc_table<512><<<(unsigned)nr, 64, 0, s>>>(rows, nr, X.rp, X.col, X.val, Y.rp, Y.col,
                                                   Y.val, poff, ocol, oval, ucnt, over1, nover);
    else if (bin == 0) group(std::integral_constant<int, 8>{});
    else if (bin == 1) group(std::integral_constant<int, 16>{});
    else if (bin == 2) group(std::integral_constant<int, 32>{});
    else if (bin == 3) sort(std::integral_constant<int, 2>{});
    else if (bin == 4) sort(std::integral_constant<int, 4>{});
    else if (bin == 5) sort(std::integral_constant<int, 8>{});
    else sort(std::integral_constant<int, 16>{});
    SA_LAUNCH_CHECK();
  }
  // The longest rows first (a kernel ends with its last row), the bins of up to 2048 rows
  // together a block of eight wavefronts per row, the others a wavefront per row: 14.6K rows
  // of 8,192 products or more take 910 us with a wavefront each and 2,080 with blocks, 2.6K rows
  // of at most 37K products 185 with blocks and 440 with a wavefront each.  Rows past 32,768
  // products stay with blocks up to 8192 of them: many of their columns are distinct, and a
  // wavefront goes over such a row once per 481 columns while the chip has room (graphs of random
  // neighbours, whole setup: 2.5K rows of 4.7M products 203 ms with a wavefront each, 98 with
  // blocks; 6K of 1M 108 and 86; 5.9K of 75K 22.1 and 20.9; 7.6K of 35K 11.2 both; 21K rows 49
  // and 71).
  int64_t narrow = INT64_MAX;  // the narrowest window that a kernel leaves to the hash table
  int bin = kBins - 1;
  auto ranks = [&](auto nwc, auto rdc, int32_t tile, int64_t limit) {
    constexpr int NW = decltype(nwc)::value, RD = decltype(rdc)::value;
    RowLists rows = {};
    int64_t n = 0;
    for (int q = 0; q < 4; ++q) {
      const int64_t most = bin == kBins - 1 ? std::max<int64_t>(limit, 8192) : limit;
      if (bin >= 7 && n + hc[bin] <= most) {
        rows.list[q] = lists + bin * (int64_t)m;
        n += hc[bin];
        --bin;
      }
      rows.end[q] = (int32_t)n;
    }
    if (n == 0) return;
    const int32_t W = std::min((Y.ncols + 31) & ~31, tile);
    const int64_t maxw = (int64_t)W * max_tiles();
    narrow = std::min(narrow, maxw);
    const size_t lds = NW * RD * sizeof(double) + (size_t)(W / 32) * sizeof(uint2);
    k_esc_rows<NW, RD><<<(unsigned)n, 64 * NW, lds, s>>>(rows, X.rp, X.col, X.val, Y.rp, Y.col,
                                                        Y.val, poff, ocol, oval, ucnt, Y.ncols,
                                                        W, maxw, over1, nover);
    SA_LAUNCH_CHECK();
  };
  ranks(std::integral_constant<int, 8>{}, std::integral_constant<int, 512>{}, 65536, 2048);
  ranks(std::integral_constant<int, 1>{}, std::integral_constant<int, 512>{}, 16384, INT64_MAX);
  // windows wider than the tiles' limit and rows past 3/4 of the small table: the large
  // table, then those past 3/4 of it with a dense accumulator in global memory
  const int32_t nov1 = nhash > 0 || (nlong > 0 && Y.ncols > narrow) ? read1(nover, s) : 0;
  if (nov1 > 0) {
    int32_t *over2 = tmp.alloc<int32_t>(nov1);
    k_esc_table<2048><<<(unsigned)nov1, 64, 0, s>>>(over1, nov1, X.rp, X.col, X.val, Y.rp, Y.col,
                                                    Y.val, poff, ocol, oval, ucnt, over2,
                                                    nover + 1);
    SA_LAUNCH_CHECK();
    const int32_t nov = read1(nover + 1, s);
    if (nov > 0) {
      // dense accumulators: at most ~2 GiB of them at once
      const int64_t per = (int64_t)Y.ncols * 12;
      int64_t nb = std::min<int64_t>(nov, std::max<int64_t>(1, (int64_t(2) << 30) / per));
      nb = std::min<int64_t>(nb, 1024);
      int32_t *xpref = tmp.alloc<int32_t>(X.nnz);
      k_row_prefix<<<(unsigned)nov, kWave, 0, s>>>(over2, X.rp, X.col, Y.rp, xpref);
      SA_LAUNCH_CHECK();
      double *dacc = tmp.alloc<double>(nb * (int64_t)Y.ncols);
      int32_t *dflag = tmp.alloc<int32_t>(nb * (int64_t)Y.ncols);
      k_esc_dense<<<(unsigned)nb, kBlock, 0, s>>>(over2, nov, X.rp, X.col, X.val, xpref, Y.rp,
                                                  Y.col, Y.val, Y.ncols, poff, ocol, oval, ucnt,
                                                  dacc, dflag);
      SA_LAUNCH_CHECK();
    }
  }
  C.rp = ar.alloc<int32_t>(m + 1);
  exclusive_scan_i32(ucnt, C.rp, m, s);
  if (max_row && m > 0) {
    int32_t *mx = tmp.alloc<int32_t>(row_max_words(m) + 1);
    row_max(m, C.rp, mx + 1, mx, s);
    WordRuns last;
    last.add(C.rp + m, 1);
    last.add(mx, 1);
    int32_t h[2];
    readback_runs(h, last, s);
    C.nnz = h[0];
    C.maxrow = h[1];
  } else {
    C.nnz = read1(C.rp + m, s);
  }
  C.col = ar.alloc<int32_t>(C.nnz);
  C.val = ar.alloc<double>(C.nnz);
  if (C.nnz > 0) {
    // (64 rows of more than some 20 entries would leave a matrix of few rows to few wavefronts)
    if (C.nnz <= 20 * (int64_t)m)
      k_compact<64><<<(unsigned)ceil_div(m, kBlock), kBlock, 0, s>>>(m, poff, C.rp, ocol, oval,
                                                                   C.col, C.val);
    else
      k_compact<8><<<(unsigned)ceil_div(m, kBlock / 8), kBlock, 0, s>>>(m, poff, C.rp, ocol, oval,
                                                                      C.col, C.val);
    SA_LAUNCH_CHECK();
  }
}

// ---- numeric plan for a fixed pattern (re-setup) ---------------------------------------------
// Built once from the patterns of X, Y and C, in parallel over X's entries (a thread per
// entry, or a wavefront per entry when Y's rows are long): every product (e, q) finds its
// column in C's sorted row i by binary search.  Pass 1 counts the products of every C entry
// (atomically), pass 2 lists them in arrival order, and a last pass sorts every list by X
// position e, i.e. by inner index: within one list each e occurs once, so the order is total.
__device__ inline int32_t plan_find(const int32_t *ccol, int32_t lo, int32_t hi, int32_t j) {
  while (lo < hi) {
    const int32_t mid = (lo + hi) >> 1;
    if (ccol[mid] < j) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}
__global__ void k_entry_rows(int32_t m, const int32_t *rp, int32_t *row) {
  const int64_t i64 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i64 >= m) return;
  const int32_t i = (int32_t)i64;
  for (int32_t e = rp[i]; e < rp[i + 1]; ++e) row[e] = i;
}
// G lanes per X entry (1 or 64); FILL: place (e, q) at lrp[p] + the next free slot of p.
template <int G, bool FILL>
__global__ void k_plan_entries(int64_t nx, const int32_t *__restrict__ xrow,
                               const int32_t *__restrict__ xcol, const int32_t *__restrict__ yrp,
                               const int32_t *__restrict__ ycol,
                               const int32_t *__restrict__ crp,
                               const int32_t *__restrict__ ccol, int32_t *cnt,
                               const int64_t *__restrict__ lrp, int32_t *le, int32_t *lq,
                               int32_t *err, int32_t bit) {
  const int64_t g = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / G;
  const int32_t lane = G == 1 ? 0 : (int32_t)(threadIdx.x % G);
  if (g >= nx) return;
  const int32_t e = (int32_t)g;
  const int32_t i = xrow[e], k = xcol[e];
  const int32_t cb = crp[i], ce = crp[i + 1];
  for (int32_t q = yrp[k] + lane; q < yrp[k + 1]; q += G) {
    const int32_t j = ycol[q];
    const int32_t p = plan_find(ccol, cb, ce, j);
    if (p >= ce || ccol[p] != j) {
      atomicOr(err, bit);
      continue;
    }
    const int32_t slot = atomicAdd(cnt + p, 1);
    if (FILL) {
      le[lrp[p] + slot] = e;
      lq[lrp[p] + slot] = q;
    }
  }
}
// Thread per C entry: a list of up to kPlanShort entries sorted by X position in place
// (insertion); longer lists are listed for k_plan_sort_long.
constexpr int32_t kPlanShort = 32;
constexpr int32_t kPlanLds = 4096;  // a list is at most as long as X's longest row
__global__ void k_plan_sort(int32_t nnzc, const int64_t *__restrict__ lrp, int32_t *le,
                            int32_t *lq, int32_t *longs, int32_t *nlong) {
  const int64_t p64 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p64 >= nnzc) return;
  const int64_t b = lrp[p64], en = lrp[p64 + 1];
  if (en - b > kPlanShort) {
    longs[atomicAdd(nlong, 1)] = (int32_t)p64;
    return;
  }
  for (int64_t t = b + 1; t < en; ++t) {
    const int32_t ke = le[t], kq = lq[t];
    int64_t u = t - 1;
    while (u >= b && le[u] > ke) {
      le[u + 1] = le[u];
      lq[u + 1] = lq[u];
      --u;
    }
    le[u + 1] = ke;
    lq[u + 1] = kq;
  }
}
// Block per long list (grid-stride over them): keys (e << 32 | q) sorted by a bitonic sort in
// LDS (e is unique within a list, so the order is that of e); a list past kPlanLds entries (X
// rows that long) falls back to thread 0's insertion sort.
__global__ __launch_bounds__(kBlock) void k_plan_sort_long(const int32_t *__restrict__ longs,
                                                           const int32_t *__restrict__ nlong,
                                                           const int64_t *__restrict__ lrp,
                                                           int32_t *le, int32_t *lq) {
  __shared__ uint64_t key[kPlanLds];
  const int32_t nl = *nlong;
  for (int32_t idx = blockIdx.x; idx < nl; idx += gridDim.x) {
    const int32_t p = longs[idx];
    const int64_t b = lrp[p];
    const int32_t len = (int32_t)(lrp[p + 1] - b);
    if (len > kPlanLds) {  // block-uniform
      if (threadIdx.x == 0) {
        for (int32_t t = 1; t < len; ++t) {
          const int32_t ke = le[b + t], kq = lq[b + t];
          int32_t u = t - 1;
          while (u >= 0 && le[b + u] > ke) {
            le[b + u + 1] = le[b + u];
            lq[b + u + 1] = lq[b + u];
            --u;
          }
          le[b + u + 1] = ke;
          lq[b + u + 1] = kq;
        }
      }
      __syncthreads();
      continue;
    }
    int32_t L = 1;
    while (L < len) L <<= 1;
    for (int32_t t = threadIdx.x; t < L; t += blockDim.x)
      key[t] = t < len ? (((uint64_t)(uint32_t)le[b + t] << 32) | (uint32_t)lq[b + t]) : ~0ull;
    __syncthreads();
    for (int32_t kk = 2; kk <= L; kk <<= 1) {
      for (int32_t jj = kk >> 1; jj > 0; jj >>= 1) {
        for (int32_t t = threadIdx.x; t < L; t += blockDim.x) {
          const int32_t u = t ^ jj;
          if (u > t) {
            const uint64_t x = key[t], y = key[u];
            if ((x > y) == ((t & kk) == 0)) {
              key[t] = y;
              key[u] = x;
            }
          }
        }
        __syncthreads();
      }
    }
    for (int32_t t = threadIdx.x; t < len; t += blockDim.x) {
      le[b + t] = (int32_t)(key[t] >> 32);
      lq[b + t] = (int32_t)(uint32_t)key[t];
    }
    __syncthreads();
  }
}
__global__ void k_plan_numeric(int32_t nnzc, const int64_t *__restrict__ lrp,
                               const int32_t *__restrict__ le, const int32_t *__restrict__ lq,
                               const double *__restrict__ xv, const double *__restrict__ yv,
                               double *__restrict__ cv) {
  const int64_t p64 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p64 >= nnzc) return;
  const int32_t p = (int32_t)p64;
  double s = 0.0;
  for (int64_t t = lrp[p]; t < lrp[p + 1]; ++t) s += xv[le[t]] * yv[lq[t]];
  cv[p] = s;
}

__global__ void k_widen_i32(int64_t n, const int32_t *a, int64_t *b) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) b[i] = a[i];
}
static void widen_i32(const int32_t *a, int64_t *b, int64_t n, hipStream_t s) {
  if (n <= 0) return;
  k_widen_i32<<<grid_for(n), kBlock, 0, s>>>(n, a, b);
  SA_LAUNCH_CHECK();
}

void spgemm_plan(const Csr &X, const Csr &Y, const Csr &C, Arena &ar, SpgemmPlan &pl,
                 int32_t *err, int32_t bit, hipStream_t s) {
  pl = SpgemmPlan{};
  Arena tmp;
  tmp.stream = s;
  const int64_t nx = X.nnz;
  int32_t *xrow = tmp.alloc<int32_t>(nx > 0 ? nx : 1);
  int32_t *cnt = tmp.alloc<int32_t>(C.nnz + 1);
  pl.lrp = ar.alloc<int64_t>(C.nnz + 1);
  int64_t *cnt64 = tmp.alloc<int64_t>(C.nnz + 1);
  fill_i32(cnt, 0, C.nnz + 1, s);
  if (X.n > 0) {
    k_entry_rows<<<grid_for(X.n), kBlock, 0, s>>>(X.n, X.rp, xrow);
    SA_LAUNCH_CHECK();
  }
  // long Y rows: a wavefront per X entry
  const bool wide = (Y.maxrow >= 0 ? Y.maxrow : max_row_length(Y.n, Y.rp, s)) > 32;
  auto pass = [&](bool fill) {
    if (nx <= 0) return;
    if (wide) {
      if (fill)
        k_plan_entries<64, true><<<grid_for(nx * 64), kBlock, 0, s>>>(
            nx, xrow, X.col, Y.rp, Y.col, C.rp, C.col, cnt, pl.lrp, pl.le, pl.lq, err, bit);
      else
        k_plan_entries<64, false><<<grid_for(nx * 64), kBlock, 0, s>>>(
            nx, xrow, X.col, Y.rp, Y.col, C.rp, C.col, cnt, nullptr, nullptr, nullptr, err,
            bit);
    } else {
      if (fill)
        k_plan_entries<1, true><<<grid_for(nx), kBlock, 0, s>>>(
            nx, xrow, X.col, Y.rp, Y.col, C.rp, C.col, cnt, pl.lrp, pl.le, pl.lq, err, bit);
      else
        k_plan_entries<1, false><<<grid_for(nx), kBlock, 0, s>>>(
            nx, xrow, X.col, Y.rp, Y.col, C.rp, C.col, cnt, nullptr, nullptr, nullptr, err,
            bit);
    }
    SA_LAUNCH_CHECK();
  };
  pass(false);
  widen_i32(cnt, cnt64, C.nnz, s);
  exclusive_scan_i64(cnt64, pl.lrp, C.nnz, s);
  pl.nprod = read1(pl.lrp + C.nnz, s);
  pl.le = ar.alloc<int32_t>(pl.nprod > 0 ? pl.nprod : 1);
  pl.lq = ar.alloc<int32_t>(pl.nprod > 0 ? pl.nprod : 1);
  fill_i32(cnt, 0, C.nnz + 1, s);
  pass(true);
  if (C.nnz > 0) {
    int32_t *longs = tmp.alloc<int32_t>(C.nnz);
    int32_t *nlong = tmp.alloc<int32_t>(1);
    fill_i32(nlong, 0, 1, s);
    k_plan_sort<<<grid_for(C.nnz), kBlock, 0, s>>>((int32_t)C.nnz, pl.lrp, pl.le, pl.lq, longs,
                                                   nlong);
    k_plan_sort_long<<<1024, kBlock, 0, s>>>(longs, nlong, pl.lrp, pl.le, pl.lq);
    SA_LAUNCH_CHECK();
  }
}

void spgemm_numeric(const Csr &X, const Csr &Y, const SpgemmPlan &pl, Csr &C, hipStream_t s) {
  if (C.nnz <= 0) return;
  k_plan_numeric<<<grid_for(C.nnz), kBlock, 0, s>>>((int32_t)C.nnz, pl.lrp, pl.le, pl.lq, X.val,
                                                    Y.val, C.val);
  SA_LAUNCH_CHECK();
}

// R = P^T: entry k of P (row i, column c) sits in R's row c at column i.
__global__ void k_transpose_perm(int32_t n, const int32_t *__restrict__ prp,
                                 const int32_t *__restrict__ pcol,
                                 const int32_t *__restrict__ rrp,
                                 const int32_t *__restrict__ rcol, int32_t *perm) {
  const int64_t i64 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i64 >= n) return;
  const int32_t i = (int32_t)i64;
  for (int32_t k = prp[i]; k < prp[i + 1]; ++k) {
    const int32_t c = pcol[k];
    const int32_t p = plan_find(rcol, rrp[c], rrp[c + 1], i);
    perm[k] = (p < rrp[c + 1] && rcol[p] == i) ? p : -1;  // -1: never, for R = P^T
  }
}
__global__ void k_transpose_values(int64_t nnz, const int32_t *__restrict__ perm,
                                   const double *__restrict__ pv, double *__restrict__ rv) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < nnz && perm[k] >= 0) rv[perm[k]] = pv[k];
}
void transpose_perm(const Csr &P, const Csr &R, Arena &ar, int32_t **perm, hipStream_t s) {
  *perm = ar.alloc<int32_t>(P.nnz > 0 ? P.nnz : 1);
  if (P.n > 0) {
    k_transpose_perm<<<grid_for(P.n), kBlock, 0, s>>>(P.n, P.rp, P.col, R.rp, R.col, *perm);
    SA_LAUNCH_CHECK();
  }
}
void transpose_values(const Csr &P, const int32_t *perm, Csr &R, hipStream_t s) {
  if (P.nnz <= 0) return;
  k_transpose_values<<<grid_for(P.nnz), kBlock, 0, s>>>(P.nnz, perm, P.val, R.val);
  SA_LAUNCH_CHECK();
}

}  // namespace sa
