// Device-side bodies of the solve-phase kernels (internal).
//
// Every solve kernel exists twice: a standalone launch over one vector or matrix
// (solve_kernels.hip) and a grouped launch over a table of segments, one per hierarchy
// (solve_batch.hip).  Both call the functions below with the segment's own arguments, so a
// hierarchy's arithmetic is the same whichever way its work was launched.
#pragma once
#include <type_traits>

#include "kernels.hpp"

namespace sa {

// Epilogues with a block_max member also reduce a per-row value over the row block:
// row_max(has_row, s, pre) is called by every thread, block_max(b, m) once per block.
template <class E, class = void>
struct HasBlockMax : std::false_type {};
template <class E>
struct HasBlockMax<E, std::void_t<decltype(&E::block_max)>> : std::true_type {};

// Maximum over the wavefront's lanes (row shifts within 16 lanes, then the last lane of each
// row into the next rows), as a scalar.
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  int x = (int)v;
  auto step = [&](int o) { x = (int)max((uint32_t)x, (uint32_t)o); };
  step(__builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false));  // row_shr:1
  step(__builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false));  // row_shr:2
  step(__builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false));  // row_shr:4
  step(__builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false));  // row_shr:8
  step(__builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false));  // row_bcast:15
  step(__builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false));  // row_bcast:31
  return (uint32_t)__builtin_amdgcn_readlane(x, 63);
}

// An epilogue with exponent(b, t) has x scaled by 2^-exponent as it is gathered; called by every
// thread t of block b.
template <class E, class = void>
struct HasScale : std::false_type {};
template <class E>
struct HasScale<E, std::void_t<decltype(&E::exponent)>> : std::true_type {};

template <class T>
struct Chunk {
  static constexpr int value = sizeof(T) == 8 ? 2048 : 4096;
};

constexpr int32_t kPlanWindow = 2048;  // cost units per SpMV block
constexpr int32_t kPlanRowCost = 8;     // cost of a row besides its entries

// Row sums.  A row of at most kLongRow = 64 entries is summed in ascending column order from
// 0.  A longer row is summed the same way by its own thread when Split is false (the plain
// definition, used where the result must equal the sequential sum bit for bit), and
// otherwise, with in-row positions k = 0..L-1 in ascending column order, as 64 interleaved
// partial sums p_l over the positions l, l+64, l+128, ... (each in order from 0), followed by
// p_0 + ... + p_63 in order from 0.  For L <= 64 the two forms agree exactly; the split lets
// lane l of a wavefront form p_l instead of one thread adding all L products in a dependent
// chain.
constexpr int32_t kLongRow = 64;

// The rows of a row block start within one window of kPlanWindow cost units (row r costs
// rp[r] + kPlanRowCost r, at least its entry count), and a chunk holds kPlanWindow entries:
// every row of a block but its last lies in the block's first chunk, so at most one row (the
// last) spans chunks.
static_assert(Chunk<double>::value >= kPlanWindow && Chunk<float>::value >= kPlanWindow,
              "rows other than a block's last fit its first chunk");

// LDS of one SpMV row block: the chunk's products (a long row that lies in the chunk gets
// its 64 partial sums written over its own first 64 products), the partials of a long row
// that spans chunks, and per wavefront the mask of its threads whose rows are long.
template <class T>
struct SpmvShared {
  T prod[Chunk<T>::value];
  T lastp[64];
  uint64_t longmask[kBlock / 64];
};

// One SpMV row block b (rows plan[2b] .. plan[2b+2]-1, entries from plan[2b+1]): the block
// streams the rows' entries through LDS in coalesced chunks, forming each product
// val*x[col] once.  Every thread adds the products of its own short row in ascending column
// order from 0.  The block's j-th long row is taken by wavefront j mod 4: lane l forms p_l
// (carried in a register across chunks for the one row that spans chunks) and stores it in
// LDS; after the chunk's barrier the row's own thread adds its 64 partials in order.  Each
// row's sum goes to the epilogue from the row's own thread.
template <class T, class Epi, bool Split = true>
__device__ __forceinline__ void spmv_block(int32_t b, const int32_t *__restrict__ plan,
                                           const int32_t *__restrict__ rp,
                                           const int32_t *__restrict__ col,
                                           const T *__restrict__ val,
                                           const T *__restrict__ x, const Epi &epi,
                                           SpmvShared<T> &sh) {
  constexpr int CH = Chunk<T>::value;
  constexpr int NW = kBlock / 64;
  const int t = threadIdx.x;
  const int lane = t & 63, wv = t >> 6;
  // row and entry ranges: two independent 8-byte loads (one round trip)
  const int2 p0 = ((const int2 *)plan)[b], p1 = ((const int2 *)plan)[b + 1];
  int ex = 0;
  if constexpr (HasScale<Epi>::value) ex = -epi.exponent(b, t);
  const int32_t r0 = p0.x, e0 = p0.y, r1 = p1.x, e1 = p1.y;
  if (r0 >= r1) {  // block-uniform: no rows (a block max, if any, is 0)
    if constexpr (HasBlockMax<Epi>::value)
      if (t == 0) epi.block_max(b, 0ull);
    return;
  }
  const int32_t row = r0 + t;
  int32_t mb = 0, me = 0;
  typename Epi::Pre pre{};
  if (row < r1) {
    mb = rp[row];
    me = rp[row + 1];
    pre = epi.load(row);  // the epilogue's vector reads overlap the entry loads
  }
  T s = T(0);
  T cp = T(0);       // p_lane of the long row that continues into the next chunk
  bool lng = false;  // this thread's row is long
  bool any = false;  // block-uniform: the block has long rows
  for (int32_t c0 = e0; c0 < e1; c0 += CH) {
    const int32_t c1 = min(c0 + CH, e1);
#pragma unroll 8
    for (int32_t e = c0 + t; e < c1; e += kBlock) {
      T xv = x[col[e]];
      if constexpr (HasScale<Epi>::value) xv = ldexp(xv, ex);
      sh.prod[e - c0] = val[e] * xv;
    }
    if (c0 == e0) {
      // classified after the first chunk's loads are issued, so the row-pointer reads
      // overlap them (the empty asm keeps the compiler from hoisting the test, and with it
      // the wait for mb and me, above the loop)
      int32_t b2 = mb, e2 = me;
      asm volatile("" : "+v"(b2), "+v"(e2));
      lng = Split && e2 - b2 > kLongRow;
      const uint64_t lmask = __ballot(lng);
      if (lane == 0) sh.longmask[wv] = lmask;
      any = __syncthreads_or(lng) != 0;
    } else {
      __syncthreads();
    }
    if (!lng) {
      // in-order sum of the row's products in this chunk; loads are issued 8 at a time
      // ahead of the (sequential) adds
      int32_t e = max(mb, c0);
      const int32_t en = min(me, c1);
      for (; e + 8 <= en; e += 8) {
        T v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = sh.prod[e - c0 + q];
#pragma unroll
        for (int q = 0; q < 8; ++q) s += v[q];
      }
      for (; e < en; ++e) s += sh.prod[e - c0];
    }
    // long rows: this wavefront's share, in row order (block-uniform masks)
    int32_t j = 0;
#pragma unroll 1
    for (int q = 0; q < (any ? NW : 0); ++q) {
      uint64_t m = sh.longmask[q];
      while (m) {
        const int bit = __builtin_ctzll(m);
        m &= m - 1;
        if ((j++ & (NW - 1)) != wv) continue;  // wave-uniform
        const int32_t rb = rp[r0 + q * 64 + bit], re = rp[r0 + q * 64 + bit + 1];
        const int32_t lo = max(rb, c0), hi = min(re, c1);
        if (lo >= hi) continue;  // no entries in this chunk
        // this lane's positions k = lane (mod 64) in [lo, hi), 4 loads ahead of the adds
        const int32_t k0 = lo - rb;
        int32_t e = lo + ((lane - k0) & 63);
        T acc = rb < c0 ? cp : T(0);
        for (; e + 192 < hi; e += 256) {
          const T a0 = sh.prod[e - c0], a1 = sh.prod[e + 64 - c0];
          const T a2 = sh.prod[e + 128 - c0], a3 = sh.prod[e + 192 - c0];
          acc += a0;
          acc += a1;
          acc += a2;
          acc += a3;
        }
        for (; e < hi; e += 64) acc += sh.prod[e - c0];
        if (re > c1) cp = acc;                         // continues into the next chunk
        else if (rb >= c0) sh.prod[rb - c0 + lane] = acc;  // over this lane's first product
        else sh.lastp[lane] = acc;                      // a spanning row ends here
      }
    }
    __syncthreads();
    if (any) {  // block-uniform: long rows ending in this chunk add their partials in order
      if (lng && me > c0 && me <= c1) {
        const T *pj = mb >= c0 ? sh.prod + (mb - c0) : sh.lastp;
#pragma unroll 1
        for (int l = 0; l < 64; l += 8) {
          T v[8];
#pragma unroll
          for (int q = 0; q < 8; ++q) v[q] = pj[l + q];
#pragma unroll
          for (int q = 0; q < 8; ++q) s += v[q];
        }
      }
      if (c1 < e1) __syncthreads();  // before the next chunk's products
    }
  }
  if (row < r1) epi.store(row, s, pre);
  if constexpr (HasBlockMax<Epi>::value) {
    // the block's largest epilogue value: wavefront maxima, then thread 0 over the four (the
    // long-row masks' words are free by now)
    unsigned long long m = epi.row_max(row < r1, s, pre);
    for (int off = 32; off >= 1; off >>= 1) {
      const unsigned long long o = __shfl_xor(m, off, 64);
      m = o > m ? o : m;
    }
    if (lane == 0) sh.longmask[wv] = m;
    __syncthreads();
    if (t == 0) {
      unsigned long long mb2 = sh.longmask[0];
#pragma unroll
      for (int q = 1; q < NW; ++q) mb2 = sh.longmask[q] > mb2 ? sh.longmask[q] : mb2;
      epi.block_max(b, mb2);
    }
  }
}

// Rows by lanes: G lanes of a wavefront share a row; lane j adds the products of the row's
// entries j, j + G, ... in order from 0, and the lanes' sums are added pairwise (j with j ^ G/2,
// then j ^ G/4, ...).  A lane's loads are issued U at a time.  No LDS and no barriers: where
// rows are of similar length, or the matrix is small, a row costs its chain of dependent
// loads (row range, entries, x) instead of a block's.  100^3 27-point level 0 (26 entries per
// row, 309 MB): row blocks 93-97 us; 4 lanes 77-82 us; 2 and 8 lanes 102 and 97-114 us.
// 180,000-row elasticity level 0 (76 per row, 165 MB): 51-58 against 29-33 us with 8 lanes.
// 1,631 rows of 721: 7.4-9.4 against 4.6-6.4 us with 64.
template <class T, class Epi, int G>
__device__ __forceinline__ void spmv_rows(int64_t blk, int32_t n, const int32_t *__restrict__ rp,
                                          const int32_t *__restrict__ col,
                                          const T *__restrict__ val, const T *__restrict__ x,
                                          const Epi &epi) {
  constexpr int U = G == 4 ? 8 : 4;
  const int64_t row64 = blk * (kBlock / G) + threadIdx.x / G;
  if (row64 >= n) return;
  const int32_t row = (int32_t)row64;
  const int j = threadIdx.x % G;
  const int32_t b = rp[row], e = rp[row + 1];
  typename Epi::Pre pre{};
  if (j == 0) pre = epi.load(row);
  T s = T(0);
  int32_t k = b + j;
  for (; k + (U - 1) * G < e; k += U * G) {
    int32_t c[U];
    T v[U], xv[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      c[q] = col[k + q * G];
      v[q] = val[k + q * G];
    }
#pragma unroll
    for (int q = 0; q < U; ++q) xv[q] = x[c[q]];
#pragma unroll
    for (int q = 0; q < U; ++q) s += v[q] * xv[q];
  }
  if (k < e) {  // up to U - 1 more, loaded together (the row's last entry past its end)
    int32_t c[U - 1];
    T v[U - 1], xv[U - 1];
#pragma unroll
    for (int q = 0; q < U - 1; ++q) {
      const int32_t kk = min(k + q * G, e - 1);
      c[q] = col[kk];
      v[q] = val[kk];
    }
#pragma unroll
    for (int q = 0; q < U - 1; ++q) xv[q] = x[c[q]];
#pragma unroll
    for (int q = 0; q < U - 1; ++q)
      if (k + q * G < e) s += v[q] * xv[q];
  }
#pragma unroll
  for (int off = G / 2; off >= 1; off >>= 1) s += __shfl_xor(s, off, G);
  if (j == 0) epi.store(row, s, pre);
}

// ---- fused SpMV epilogues: row i receives s = (A x)_i ------------------------------------
// load(i) reads the row's other inputs (issued before the row's entries are gathered, so
// their latency overlaps); store(i, s, pre) computes and writes.  Inputs are never vectors
// the same launch writes at another row.
template <class T>
struct EpStore {
  T *y;
  struct Pre {};
  __device__ Pre load(int32_t) const { return {}; }
  __device__ void store(int32_t i, T s, const Pre &) const { y[i] = s; }
};
template <class T>
struct EpScale {
  const T *d;
  T *y;
  struct Pre {
    T d;
  };
  __device__ Pre load(int32_t i) const { return {d[i]}; }
  __device__ void store(int32_t i, T s, const Pre &p) const { y[i] = p.d * s; }
};
// y = d (A x') as EpScale, and the largest |y_i| (NaN left out) as the bit pattern of a
// non-negative double (monotone for non-negative values): each row block adds its maximum
// with one atomic maximum to slot (block mod kMaxSlots).  x' = x / 2^ilogb(m) with m the largest
// of prev, the slots that the launch before filled (none: x' = x): every wavefront reduces
// them, which is cheaper than a pass over the vector between two products and a launch less
// (101x97x89 re-setup + solve 9.54 -> 9.37 ms).  A zero or non-finite m marks the iteration dead.
// The first block clears next, which the next launch fills.
template <class T>
struct EpScaleMax {
  const T *d;
  T *y;
  unsigned long long *slots;
  const unsigned long long *prev;
  unsigned long long *next;
  int32_t *dead;
  __device__ int exponent(int32_t b, int t) const {
    static_assert(kMaxSlots == kBlock && kMaxSlots == 4 * 64, "four slots per lane");
    if (b == 0) next[t] = 0ull;
    if (!prev) return 0;
    // the high words hold the exponent, unless the largest is zero or subnormal
    const uint32_t *hi = (const uint32_t *)prev + 1;
    const int lane = t & 63;
    uint32_t h = max(max(hi[2 * lane], hi[2 * (64 + lane)]),
                     max(hi[2 * (128 + lane)], hi[2 * (192 + lane)]));
    h = wave_max(h);
    if (h >= 0x7ff00000u) {
      if (b == 0 && t == 0) *dead = 1;
      return 0;
    }
    if (h >= 0x00100000u) return (int)(h >> 20) - 1023;
    unsigned long long m = 0ull;
    for (int q = 0; q < kMaxSlots; ++q) m = prev[q] > m ? prev[q] : m;
    if (m == 0ull) {
      if (b == 0 && t == 0) *dead = 1;
      return 0;
    }
    return ilogb(__longlong_as_double((long long)m));
  }
  struct Pre {
    T d;
  };
  __device__ Pre load(int32_t i) const { return {d[i]}; }
  __device__ void store(int32_t i, T s, const Pre &p) const { y[i] = p.d * s; }
  __device__ unsigned long long row_max(bool has, T s, const Pre &p) const {
    if (!has) return 0ull;
    const double a = fabs((double)(p.d * s));
    return (a == a) ? (unsigned long long)__double_as_longlong(a) : 0ull;
  }
  __device__ void block_max(int32_t b, unsigned long long m) const {
    if (m != 0ull) atomicMax(slots + (b % kMaxSlots), m);
  }
};
// y = A x, the coarse residual of the restriction, and the first smoother step on it
// (u = 0): Chebyshev d = (invD .* y) / theta, with write_u also u = 0 + d.
template <class T>
struct EpRestrictCheb {
  T *y;
  const T *invD;
  T theta;
  T *d, *u;
  bool write_u;
  struct Pre {
    T invD;
  };
  __device__ Pre load(int32_t i) const { return {invD[i]}; }
  __device__ void store(int32_t i, T s, const Pre &p) const {
    y[i] = s;
    const T di = (p.invD * s) / theta;
    d[i] = di;
    if (write_u) u[i] = T(0) + di;
  }
};
// The same with Jacobi: u = 0 + w (invD .* y).
template <class T>
struct EpRestrictJacobi {
  T *y;
  const T *invD;
  T w;
  T *u;
  struct Pre {
    T invD;
  };
  __device__ Pre load(int32_t i) const { return {invD[i]}; }
  __device__ void store(int32_t i, T s, const Pre &p) const {
    y[i] = s;
    u[i] = T(0) + w * (p.invD * s);
  }
};
template <class T>
struct EpResid {
  const T *f;
  T *r;
  struct Pre {
    T f;
  };
  __device__ Pre load(int32_t i) const { return {f[i]}; }
  __device__ void store(int32_t i, T s, const Pre &p) const { r[i] = p.f - s; }
};
template <class T>
struct EpAdd {
  T *u;
  struct Pre {
    T u;
  };
  __device__ Pre load(int32_t i) const { return {u[i]}; }
  __device__ void store(int32_t i, T s, const Pre &p) const { u[i] = p.u + s; }
};
template <class T>
struct EpChebStart {
  const T *f, *invD;
  T theta;
  T *r, *d;
  struct Pre {
    T f, invD;
  };
  __device__ Pre load(int32_t i) const { return {f[i], invD[i]}; }
  __device__ void store(int32_t i, T s, const Pre &p) const {
    T ri = p.f - s;
    r[i] = ri;
    d[i] = (p.invD * ri) / theta;
  }
};
template <class T>
struct EpChebStep {
  const T *d, *rin, *invD;
  T *rout, *u, *dout;
  T c1, c2;
  bool uzero, last;
  double *z;  // the last step's u in FP64 too (null: not wanted)
  struct Pre {
    T d, rin, invD, u;
  };
  __device__ Pre load(int32_t i) const {
    return {d[i], rin[i], invD[i], uzero ? T(0) : u[i]};
  }
  __device__ void store(int32_t i, T s, const Pre &p) const {
    T di = p.d;
    T ui = p.u + di;
    T ri = p.rin - s;
    rout[i] = ri;
    T dn = c1 * di + c2 * (p.invD * ri);
    if (last) {
      const T un = ui + dn;
      u[i] = un;
      if (z) z[i] = (double)un;
    } else {
      u[i] = ui;
      dout[i] = dn;
    }
  }
};
template <class T>
struct EpJacobi {
  const T *u, *f, *invD;
  T w;
  T *u2;
  struct Pre {
    T u, f, invD;
  };
  __device__ Pre load(int32_t i) const { return {u[i], f[i], invD[i]}; }
  __device__ void store(int32_t i, T s, const Pre &p) const {
    T r = p.f - s;
    u2[i] = p.u + w * (p.invD * r);
  }
};

// ---- element-wise bodies -----------------------------------------------------------------
template <class T>
__device__ __forceinline__ void cheb_first_at(int32_t i, const T *f, const T *invD, T theta,
                                              T *d, T *u, bool write_u) {
  T di = (invD[i] * f[i]) / theta;
  d[i] = di;
  if (write_u) u[i] = T(0) + di;
}
template <class T>
__device__ __forceinline__ void vec_add_at(int32_t i, T *u, const T *d) {
  u[i] = u[i] + d[i];
}
template <class T>
__device__ __forceinline__ void jacobi_first_at(int32_t i, const T *f, const T *invD, T w,
                                                T *u) {
  u[i] = T(0) + w * (invD[i] * f[i]);
}

// ---- canonical inner product: one block of 4096 terms --------------------------------------
// Lane t of 256 sums terms t + 256 m (m = 0..15) sequentially from 0 (products x[i]*y[i], or
// x[i] alone when y is null), then s[t] += s[t + w] for w = 128 ... 1.  The blocks of kDotBlock
// threads form a block's 4096 terms in LDS first (four per thread; absent terms are 0.0, which
// leaves a sum from 0.0 unchanged), so the 216 blocks of 885K unknowns fill the chip: with
// 256 threads holding 16 terms each an update of x and r took 18.1 us there and one of p 11.5,
// now 10.9 and 5.6.
constexpr int kDotBlock = 1024;
constexpr int kDotTerms = 4096;
struct DotShared {
  double term[kDotTerms];
  double sum[kBlock];
};
// The sum of the block's terms, for every thread; ends with a barrier.
__device__ __forceinline__ double dot_sum_terms(DotShared &sh) {
  const int t = threadIdx.x;
  __syncthreads();
  if (t < kBlock) {
    double acc = 0.0;
#pragma unroll
    for (int m = 0; m < kDotTerms / kBlock; ++m) acc += sh.term[t + kBlock * m];
    sh.sum[t] = acc;
  }
  __syncthreads();
  for (int w = kBlock / 2; w >= 64; w >>= 1) {
    if (t < w) sh.sum[t] = sh.sum[t] + sh.sum[t + w];
    __syncthreads();
  }
  if (t < 64) {  // one wavefront: lanes below w add the sums w above them
    double v = sh.sum[t];
#pragma unroll
    for (int w = 32; w >= 1; w >>= 1) {
      const double o = __shfl_down(v, w, 64);
      v = v + o;
    }
    if (t == 0) sh.sum[0] = v;
  }
  __syncthreads();
  const double r = sh.sum[0];
  __syncthreads();
  return r;
}
__device__ __forceinline__ void dot_block(int64_t blk, const double *__restrict__ x,
                                          const double *__restrict__ y, int64_t n,
                                          double *__restrict__ out, DotShared &sh) {
  const int t = threadIdx.x;
  const int64_t base = blk * kDotTerms + t;
#pragma unroll
  for (int m = 0; m < kDotTerms / kDotBlock; ++m) {
    const int64_t i = base + kDotBlock * m;
    double v = 0.0;
    if (i < n) v = y ? x[i] * y[i] : x[i];
    sh.term[t + kDotBlock * m] = v;
  }
  const double s = dot_sum_terms(sh);
  if (t == 0) *out = s;
}

// The two inner products r.z and r.(z - zold) of one block (zold null: the first only).
__device__ __forceinline__ void dot_rz_block(int64_t blk, const double *__restrict__ r,
                                             const double *__restrict__ z,
                                             const double *__restrict__ zold, int64_t n,
                                             double *__restrict__ out, double *__restrict__ outw,
                                             DotShared &sh) {
  constexpr int M = kDotTerms / kDotBlock;
  const int t = threadIdx.x;
  const int64_t base = blk * kDotTerms + t;
  double w[M];
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const int64_t i = base + kDotBlock * m;
    double v = 0.0;
    w[m] = 0.0;
    if (i < n) {
      const double ri = r[i], zi = z[i];
      v = ri * zi;
      if (zold) w[m] = ri * (zi - zold[i]);
    }
    sh.term[t + kDotBlock * m] = v;
  }
  const double s = dot_sum_terms(sh);
  if (t == 0) *out = s;
  if (!zold) return;  // uniform
#pragma unroll
  for (int m = 0; m < M; ++m) sh.term[t + kDotBlock * m] = w[m];
  const double sw = dot_sum_terms(sh);
  if (t == 0) *outw = sw;
}

// The last stage of the canonical inner product (m <= 4096 partials), taken by every block
// that needs the value instead of by a launch of its own; all threads get the sum.
constexpr int32_t kDotFinal = 4096;
__device__ __forceinline__ double dot_final(const double *__restrict__ part, int32_t m,
                                            DotShared &sh) {
  const int t = threadIdx.x;
#pragma unroll
  for (int q = 0; q < kDotTerms / kDotBlock; ++q) {
    const int32_t i = t + kDotBlock * q;
    sh.term[i] = i < m ? part[i] : 0.0;
  }
  return dot_sum_terms(sh);
}

// ---- dense GEMV row (coarsest level): one wavefront per row --------------------------------
template <class T>
__device__ __forceinline__ void gemv_row(int64_t row, int32_t n, const double *__restrict__ M,
                                         const T *__restrict__ x, T *__restrict__ y) {
  const int lane = threadIdx.x & 63;
  const double *m = M + row * n;
  double acc = 0.0;
  for (int32_t j = lane; j < n; j += 64) acc += m[j] * (double)x[j];
  for (int off = 32; off >= 1; off >>= 1) acc += __shfl_down(acc, off, 64);
  if (lane == 0) y[row] = (T)acc;
}

// ---- PCG steps ---------------------------------------------------------------------------------
// What a launch of CG work costs beyond its vectors is about 4.5 us, so the scalar steps and
// the last stages of the inner products are not launches of their own: the blocks that use
// alpha or beta each reduce the partials again (4 KB at n = 2M).  The scalars alternate
// between two sets, because every block reads rho while block 0 writes the next one.

// First smoother step of the next preconditioner application on the new residual.
struct FirstNone {
  __device__ void operator()(int64_t, double) const {}
};
struct FirstCheb64 {
  const double *invD;
  double theta;
  double *d, *u;
  bool write_u;
  __device__ void operator()(int64_t i, double r) const {
    const double di = (invD[i] * r) / theta;
    d[i] = di;
    if (write_u) u[i] = 0.0 + di;
  }
};
struct FirstCheb32 {
  float *f;
  const float *invD;
  float theta;
  float *d, *u;
  bool write_u;
  __device__ void operator()(int64_t i, double r) const {
    const float ri = (float)r;
    f[i] = ri;
    const float di = (invD[i] * ri) / theta;
    d[i] = di;
    if (write_u) u[i] = 0.0f + di;
  }
};

// alpha = rho / p.q (partials part[0..m)), x += alpha p, r -= alpha q, and the block's share
// of the new r.r: block blk takes the 4096 elements of its block of the inner product.
template <class First>
__device__ __forceinline__ void pcg_xr_block(int64_t blk, int64_t n, double *__restrict__ x,
                                             double *__restrict__ r,
                                             const double *__restrict__ p,
                                             const double *__restrict__ q,
                                             const double *__restrict__ part, int32_t m,
                                             PcgScalars *S, double *__restrict__ out,
                                             const First &first, DotShared &sh) {
  constexpr int M = kDotTerms / kDotBlock;
  const int t = threadIdx.x;
  const int64_t base = blk * kDotTerms + t;
  double pi[M], qi[M], xi[M], ri[M];  // loaded ahead of the reduction
#pragma unroll
  for (int k = 0; k < M; ++k) {
    const int64_t i = base + kDotBlock * k;
    if (i < n) {
      pi[k] = p[i];
      qi[k] = q[i];
      xi[k] = x[i];
      ri[k] = r[i];
    }
  }
  const double pq = dot_final(part, m, sh);
  const double alpha = S->rho / pq;
  if (blk == 0 && t == 0) {
    if (!(pq > 0.0)) S->err = 1;
    S->pq = pq;
    S->alpha = alpha;
  }
#pragma unroll
  for (int k = 0; k < M; ++k) {
    const int64_t i = base + kDotBlock * k;
    double v = 0.0;
    if (i < n) {
      x[i] = xi[k] + alpha * pi[k];
      const double rn = ri[k] - alpha * qi[k];
      r[i] = rn;
      v = rn * rn;
      first(i, rn);
    }
    sh.term[t + kDotBlock * k] = v;
  }
  const double s = dot_sum_terms(sh);
  if (t == 0) out[blk] = s;
}

// rho1 = r.z and, with pr, rw = r.(z - zold) from their partials; beta; p = z + beta p (init:
// p = z).  Reads the scalars cur, writes next (init: the same set).
__device__ __forceinline__ void pcg_p_block(int64_t blk, int64_t n, double *__restrict__ p,
                                            const double *__restrict__ z,
                                            const double *__restrict__ part,
                                            const double *__restrict__ partw, int32_t m,
                                            const PcgScalars *cur, PcgScalars *next, bool pr,
                                            bool init, DotShared &sh) {
  constexpr int M = kDotTerms / kDotBlock;
  const int t = threadIdx.x;
  const int64_t base = blk * kDotTerms + t;
  double zi[M], pi[M];
#pragma unroll
  for (int k = 0; k < M; ++k) {
    const int64_t i = base + kDotBlock * k;
    if (i < n) {
      zi[k] = z[i];
      pi[k] = init ? 0.0 : p[i];
    }
  }
  const double rho1 = dot_final(part, m, sh);
  const double rw = pr && !init ? dot_final(partw, m, sh) : 0.0;
  const double beta = init ? 0.0 : (pr ? rw : rho1) / cur->rho;
#pragma unroll
  for (int k = 0; k < M; ++k) {
    const int64_t i = base + kDotBlock * k;
    if (i < n) p[i] = init ? zi[k] : zi[k] + beta * pi[k];
  }
  if (blk == 0 && t == 0) {
    next->rho1 = rho1;
    next->rw = rw;
    next->beta = beta;
    next->rho = rho1;
    next->err = !(rho1 > 0.0) ? 2 : cur->err;
  }
}

}  // namespace sa
