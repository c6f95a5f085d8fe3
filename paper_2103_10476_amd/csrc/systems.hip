// Systems SA with a multi-vector nullspace (internal): node graph, block strength, dof labels,
// the QR tentative prolongator and its smoothing.
//
// The paper treats scalar PDEs and names systems as future work; this is the standard
// smoothed aggregation for systems (Vanek, Mandel, Brezina) with these readings:
//  * dofs are numbered node-major (dof = bs * node + component);
//  * node I is linked to node J when a row of I has an entry in a column of J; the block
//    strength is F_IJ = sum of a_ij^2 over the bs x bs block (rows ascending, then columns
//    ascending) and (I,J) is strong iff F_IJ^2 >= theta^4 F_II F_JJ, i.e. ||A_IJ||_F >=
//    theta sqrt(||A_II||_F ||A_JJ||_F) (the scalar test for bs = 1);
//  * a dof entry between two nodes takes the node pair's label; entries inside a node are kept;
//  * aggregate J's dofs (members ascending, components ascending) take the rows of the
//    nullspace B, factored B_J = Q_J R_J by Householder reflections (R's diagonal made
//    non-negative); P_t holds Q_J in columns kJ..kJ+k-1 and the coarse nullspace holds R_J;
//  * P = P_t - (omega invD_i) (Abar P_t)_i per row, on the pattern of Abar P_t.
// Every sum runs in the order stated, so the results equal the sequential definitions bit for
// bit.
#include <climits>

#include "kernels.hpp"

namespace sa {

#define SA_ROW_BEGIN(n)                                              \
  const int64_t i64_ = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; \
  if (i64_ >= (n)) return;                                           \
  const int32_t I = (int32_t)i64_;

constexpr int kMaxBs = 16;

// ---- node graph ------------------------------------------------------------------------------
// Each of node I's bs rows lists its columns ascending, so col / bs is non-decreasing along a
// row.  Where the rows of a node have the same block columns entry by entry (whole blocks), its
// neighbours are the distinct ones of its first row; the wavefront that takes the node compares
// the rows and counts or writes them 64 entries at a time.  Otherwise one lane merges the bs
// lists with duplicates removed.  Either way the neighbours come in ascending order.
// (A thread per node walking its rows: 160 us per pass on 60,000 nodes of 3 rows of 76, 350 us
// on 2,592 nodes of 6 rows of 136; now 45 and 14 us.)
template <bool FILL>
__device__ __forceinline__ void node_row(int32_t I, int32_t bs, const int32_t *rp,
                                         const int32_t *col, int32_t *cnt, const int32_t *grp,
                                         int32_t *gcol) {
  const int lane = threadIdx.x & 63;
  const int32_t *nrp = rp + (int64_t)I * bs;
  const int32_t b0 = nrp[0], len = nrp[1] - b0;
  bool same = true;
  for (int r = 1; r < bs; ++r) same = same && nrp[r + 1] - nrp[r] == len;
  for (int32_t k = lane; same && k < len; k += 64) {
    const int32_t J = col[b0 + k] / bs;
    for (int r = 1; r < bs; ++r) same = same && col[nrp[r] + k] / bs == J;
  }
  const int32_t w = FILL ? grp[I] : 0;
  if (__all(same)) {
    int32_t c = 0;
    for (int32_t k0 = 0; k0 < len; k0 += 64) {
      const int32_t k = k0 + lane;
      bool first = false;
      int32_t J = 0;
      if (k < len) {
        J = col[b0 + k] / bs;
        first = k == 0 || col[b0 + k - 1] / bs != J;
      }
      const uint64_t mask = __ballot(first);
      if (FILL && first)
        gcol[w + c + __builtin_amdgcn_mbcnt_hi(
                         (uint32_t)(mask >> 32),
                         __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u))] = J;
      c += __popcll(mask);
    }
    if (!FILL && lane == 0) cnt[I] = c;
    return;
  }
  if (lane != 0) return;
  int32_t cur[kMaxBs], end[kMaxBs];
  for (int r = 0; r < bs; ++r) {
    cur[r] = nrp[r];
    end[r] = nrp[r + 1];
  }
  int32_t c = 0;
  for (;;) {
    int32_t J = INT_MAX;
    for (int r = 0; r < bs; ++r)
      if (cur[r] < end[r]) J = min(J, col[cur[r]] / bs);
    if (J == INT_MAX) break;
    for (int r = 0; r < bs; ++r)
      while (cur[r] < end[r] && col[cur[r]] / bs == J) ++cur[r];
    if (FILL) gcol[w + c] = J;
    ++c;
  }
  if (!FILL) cnt[I] = c;
}
template <bool FILL>
__global__ __launch_bounds__(kBlock) void k_node_graph(int32_t m, int32_t bs, const int32_t *rp,
                                                       const int32_t *col, int32_t *cnt,
                                                       const int32_t *grp, int32_t *gcol) {
  for (int64_t i = first_row<64>(); i < m; i += row_stride<64>())  // wave-uniform
    node_row<FILL>((int32_t)i, bs, rp, col, cnt, grp, gcol);
}
void node_graph(const Csr &A, int32_t bs, Arena &ar, Csr &G, hipStream_t s) {
  if (bs < 1 || bs > kMaxBs) throw Error(SA_ERR_INVALID_ARG, "block size not in 1..16");
  const int32_t m = A.n / bs;
  int32_t *cnt = (int32_t *)dev_alloc(sizeof(int32_t) * (m + 1), s);
  G.n = G.ncols = m;
  G.rp = ar.alloc<int32_t>(m + 1);
  if (m > 0) {
    k_node_graph<false><<<grid_rows(m, 64), kBlock, 0, s>>>(m, bs, A.rp, A.col, cnt, nullptr,
                                                           nullptr);
    SA_LAUNCH_CHECK();
  }
  exclusive_scan_i32(cnt, G.rp, m, s);
  dev_free(cnt, s);
  G.nnz = read1(G.rp + m, s);
  G.col = ar.alloc<int32_t>(G.nnz > 0 ? G.nnz : 1);
  G.val = nullptr;
  if (m > 0) {
    k_node_graph<true><<<grid_rows(m, 64), kBlock, 0, s>>>(m, bs, A.rp, A.col, nullptr, G.rp,
                                                          G.col);
    SA_LAUNCH_CHECK();
  }
}

// ---- block strength ----------------------------------------------------------------------------
// 32 lanes per node, a lane per neighbour J: the block's entries in row r start where the row
// before had them if that is where J begins there too (whole blocks), else at a binary search,
// and are added one by one in the stated order.  (A thread per node adding entry by entry
// into F: 450 us on 60,000 nodes, 790 us on 2,592; now 59 and 28 us.)
__global__ __launch_bounds__(kBlock) void k_block_F(int32_t m, int32_t bs,
                                                    const int32_t *__restrict__ rp,
                                                    const int32_t *__restrict__ col,
                                                    const double *__restrict__ val,
                                                    const int32_t *__restrict__ grp,
                                                    const int32_t *__restrict__ gcol,
                                                    double *__restrict__ F,
                                                    double *__restrict__ Fd) {
  for (int64_t i64 = first_row<32>(); i64 < m; i64 += row_stride<32>()) {  // uniform over the lanes
    const int32_t I = (int32_t)i64;
    const int32_t g0 = grp[I], g1 = grp[I + 1];
    const int32_t *nrp = rp + (int64_t)I * bs;
    bool own = false;
    for (int32_t q = g0 + (int32_t)(threadIdx.x & 31); q < g1; q += 32) {
      const int32_t J = gcol[q];
      double f = 0.0;
      int32_t off = 0;
      for (int r = 0; r < bs; ++r) {
        const int32_t b = nrp[r], e = nrp[r + 1];
        int32_t k = b + off;
        const bool here = r > 0 && k < e && col[k] / bs == J && (off == 0 || col[k - 1] / bs < J);
        if (!here) {  // first entry of the row with col / bs >= J
          int32_t lo = b, hi = e;
          while (lo < hi) {
            const int32_t mid = (lo + hi) >> 1;
            if (col[mid] / bs < J) lo = mid + 1;
            else hi = mid;
          }
          k = lo;
          off = k - b;
        }
        for (; k < e && col[k] / bs == J; ++k) f = f + val[k] * val[k];
      }
      F[q] = f;
      if (J == I) {
        Fd[I] = f;
        own = true;
      }
    }
    const uint64_t any = __ballot(own) >> (threadIdx.x & 32);  // this node's half
    if ((any & 0xffffffffull) == 0 && (threadIdx.x & 31) == 0) Fd[I] = 0.0;
  }
}
__global__ void k_block_label(int32_t m, const int32_t *grp, const int32_t *gcol,
                              const double *F, const double *Fd, double th4, uint8_t *nmask,
                              int32_t *scount) {
  SA_ROW_BEGIN(m)
  int32_t cnt = 0;
  for (int32_t q = grp[I]; q < grp[I + 1]; ++q) {
    const int32_t J = gcol[q];
    if (J == I) {
      nmask[q] = 3;
      continue;
    }
    const double p = Fd[I] * Fd[J];
    const bool strong = (p > 0.0) && (F[q] * F[q] >= th4 * p);
    nmask[q] = strong ? 1 : 0;
    cnt += strong;
  }
  scount[I] = cnt;
}

void block_strength(const Csr &A, int32_t bs, const Csr &G, double theta, uint8_t *nmask,
                    int32_t *scount, hipStream_t s) {
  const int32_t m = G.n;
  if (m <= 0) return;
  Arena tmp;
  tmp.stream = s;
  double *F = tmp.alloc<double>(G.nnz > 0 ? G.nnz : 1);
  double *Fd = tmp.alloc<double>(m);
  k_block_F<<<grid_rows(m, 32), kBlock, 0, s>>>(m, bs, A.rp, A.col, A.val, G.rp, G.col, F, Fd);
  const double th4 = (theta * theta) * (theta * theta);
  k_block_label<<<grid_for(m), kBlock, 0, s>>>(m, G.rp, G.col, F, Fd, th4, nmask, scount);
  SA_LAUNCH_CHECK();
}

// ---- dof labels from node labels -----------------------------------------------------------------
// A wavefront per row, a lane per entry.  (A thread per row: 396 us on 180,000 rows of 76,
// 240 us on 15,552 of 136; now 118 and 17 us.)
__global__ __launch_bounds__(kBlock) void k_dof_mask(int32_t n, int32_t bs,
                                                     const int32_t *__restrict__ rp,
                                                     const int32_t *__restrict__ col,
                                                     const int32_t *__restrict__ grp,
                                                     const int32_t *__restrict__ gcol,
                                                     const uint8_t *__restrict__ nmask,
                                                     uint8_t *__restrict__ mask) {
  for (int64_t i64 = first_row<64>(); i64 < n; i64 += row_stride<64>()) {
    const int32_t i = (int32_t)i64, I = i / bs;
    const int32_t g0 = grp[I], g1 = grp[I + 1];
    const int32_t end = rp[i + 1];
    for (int32_t e = rp[i] + (int32_t)(threadIdx.x & 63); e < end; e += 64) {
      const int32_t j = col[e], J = j / bs;
      uint8_t lab;
      if (i == j) {
        lab = 3;
      } else if (I == J) {
        lab = 1;
      } else {
        int32_t lo = g0, hi = g1 - 1;
        lab = 0;
        while (lo <= hi) {
          const int32_t mid = (lo + hi) >> 1;
          const int32_t c = gcol[mid];
          if (c == J) {
            lab = nmask[mid];
            break;
          }
          if (c < J) lo = mid + 1;
          else hi = mid - 1;
        }
      }
      mask[e] = lab;
    }
  }
}
void dof_mask(const Csr &A, int32_t bs, const Csr &G, const uint8_t *nmask, uint8_t *mask,
              hipStream_t s) {
  if (A.n <= 0) return;
  k_dof_mask<<<grid_rows(A.n, 64), kBlock, 0, s>>>(A.n, bs, A.rp, A.col, G.rp, G.col, nmask,
                                                  mask);
  SA_LAUNCH_CHECK();
}

// ---- QR tentative prolongator ----------------------------------------------------------------------
__global__ void k_pt_count(int32_t n, int32_t bs, int32_t k, const int32_t *agg, int32_t *cnt) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) cnt[i] = agg[i / bs] >= 0 ? k : 0;
}

// One thread per aggregate; M, V and Q live in the aggregate's slice of the scratch arrays
// (rows x k each, row-major).  err |= ebit when the aggregate has fewer dofs than k.
__global__ void k_agg_qr(int32_t nc, int32_t bs, int32_t k, const int32_t *mrp,
                         const int32_t *mem, const double *B, const int32_t *ptrp,
                         int32_t *ptcol, double *ptval, double *Bc, double *Ms, double *Vs,
                         double *Qs, int32_t *err, int32_t ebit) {
  SA_ROW_BEGIN(nc)
  const int32_t J = I;
  const int32_t m0 = mrp[J], cntn = mrp[J + 1] - m0;
  const int32_t rows = cntn * bs;
  if (rows < k) {
    atomicOr(err, ebit);
    return;
  }
  const int64_t base = (int64_t)m0 * bs * k;
  double *M = Ms + base, *V = Vs + base, *Q = Qs + base;
  auto dof = [&](int32_t q) -> int64_t { return (int64_t)mem[m0 + q / bs] * bs + q % bs; };
  for (int32_t q = 0; q < rows; ++q)
    for (int c = 0; c < k; ++c) {
      M[(int64_t)q * k + c] = B[dof(q) * k + c];
      V[(int64_t)q * k + c] = 0.0;
    }
  double vv[kMaxBs];
  for (int j = 0; j < k; ++j) {
    vv[j] = 0.0;
    double sigma = 0.0;
    for (int32_t i = j; i < rows; ++i) sigma = sigma + M[(int64_t)i * k + j] * M[(int64_t)i * k + j];
    const double nrm = sqrt(sigma);
    if (nrm == 0.0) continue;
    const double ajj = M[(int64_t)j * k + j];
    const double alpha = ajj > 0.0 ? -nrm : nrm;
    for (int32_t i = j; i < rows; ++i) V[(int64_t)i * k + j] = M[(int64_t)i * k + j];
    V[(int64_t)j * k + j] = ajj - alpha;
    double d = 0.0;
    for (int32_t i = j; i < rows; ++i) d = d + V[(int64_t)i * k + j] * V[(int64_t)i * k + j];
    vv[j] = d;
    if (d == 0.0) continue;
    for (int c = j; c < k; ++c) {
      double t = 0.0;
      for (int32_t i = j; i < rows; ++i) t = t + V[(int64_t)i * k + j] * M[(int64_t)i * k + c];
      const double f = (t + t) / d;
      for (int32_t i = j; i < rows; ++i)
        M[(int64_t)i * k + c] = M[(int64_t)i * k + c] - f * V[(int64_t)i * k + j];
    }
  }
  for (int32_t q = 0; q < rows; ++q)
    for (int c = 0; c < k; ++c) Q[(int64_t)q * k + c] = (q == c) ? 1.0 : 0.0;
  for (int j = k - 1; j >= 0; --j) {
    if (vv[j] == 0.0) continue;
    for (int c = 0; c < k; ++c) {
      double t = 0.0;
      for (int32_t i = j; i < rows; ++i) t = t + V[(int64_t)i * k + j] * Q[(int64_t)i * k + c];
      const double f = (t + t) / vv[j];
      for (int32_t i = j; i < rows; ++i)
        Q[(int64_t)i * k + c] = Q[(int64_t)i * k + c] - f * V[(int64_t)i * k + j];
    }
  }
  for (int r = 0; r < k; ++r) {
    const bool flip = M[(int64_t)r * k + r] < 0.0;
    for (int c = 0; c < k; ++c) {
      double rv = (c >= r) ? M[(int64_t)r * k + c] : 0.0;
      if (flip) rv = -rv;
      Bc[((int64_t)J * k + r) * k + c] = rv;
    }
    if (flip)
      for (int32_t q = 0; q < rows; ++q) Q[(int64_t)q * k + r] = -Q[(int64_t)q * k + r];
  }
  for (int32_t q = 0; q < rows; ++q) {
    const int64_t i = dof(q);
    for (int c = 0; c < k; ++c) {
      ptcol[ptrp[i] + c] = J * k + c;
      ptval[ptrp[i] + c] = Q[(int64_t)q * k + c];
    }
  }
}

// The sum over i = from..to-1 of a[i k] * b[i k], added one by one from `from` upward.  The next
// eight products are formed while the current eight are added.
__device__ __forceinline__ double chain_dot(const double *a, const double *b, int32_t k,
                                            int32_t from, int32_t to) {
  double cur[8], nxt[8], t = 0.0;
  auto load = [&](int32_t i0, double *p) {
    const double *x = a + i0 * k, *y = b + i0 * k;
#pragma unroll
    for (int q = 0; q < 8; ++q) p[q] = x[q * k] * y[q * k];
  };
  int32_t i = from;
  if (i + 8 <= to) load(i, cur);
  for (; i + 8 <= to; i += 8) {
    const bool more = i + 16 <= to;
    if (more) load(i + 8, nxt);
#pragma unroll
    for (int q = 0; q < 8; ++q) t = t + cur[q];
    if (more) {
#pragma unroll
      for (int q = 0; q < 8; ++q) cur[q] = nxt[q];
    }
  }
#pragma unroll
  for (int q = 0; q < 7; ++q)  // the last rows: clamped reads, then the additions
    nxt[q] = i < to ? a[min(i + q, to - 1) * k] * b[min(i + q, to - 1) * k] : 0.0;
#pragma unroll
  for (int q = 0; q < 7; ++q)
    if (i + q < to) t = t + nxt[q];
  return t;
}

// The same QR with one wavefront per aggregate and M, V, Q in LDS (rows x k each, rows <=
// maxrows): every sum keeps k_agg_qr's order (one lane runs it from i = j upward), so the
// results are bitwise the same.  Bound by those sums' chains of dependent additions: a column
// takes two of them (its norm; then V.V and V with every column left, one lane each, at once),
// Q's columns one.  The updates between them take a row per lane.  (2,592 aggregates of about 70
// rows, k = 6: 241 us with lane 0 forming the vectors and a lane per column the updates, now 120;
// 99 aggregates of about 157 rows: 424, now 176.)
__global__ __launch_bounds__(64) void k_agg_qr_lds(int32_t nc, int32_t bs, int32_t k,
                                                   int32_t maxrows, const int32_t *mrp,
                                                   const int32_t *mem, const double *B,
                                                   const int32_t *ptrp, int32_t *ptcol,
                                                   double *ptval, double *Bc, int32_t *err,
                                                   int32_t ebit) {
  extern __shared__ double qr_lds[];
  __shared__ double s_vv[kMaxBs], s_f[kMaxBs];
  const int32_t J = blockIdx.x;
  const int lane = threadIdx.x;
  const int32_t m0 = mrp[J], cntn = mrp[J + 1] - m0;
  const int32_t rows = cntn * bs;
  if (rows < k) {  // block-uniform
    if (lane == 0) atomicOr(err, ebit);
    return;
  }
  double *M = qr_lds, *V = qr_lds + (int64_t)maxrows * k, *Q = V + (int64_t)maxrows * k;
  auto dof = [&](int32_t q) -> int64_t { return (int64_t)mem[m0 + q / bs] * bs + q % bs; };
  for (int32_t e = lane; e < rows * k; e += 64) {
    const int32_t q = e / k, c = e % k;
    M[e] = B[dof(q) * k + c];
    Q[e] = q == c ? 1.0 : 0.0;
  }
  __syncthreads();
  for (int j = 0; j < k; ++j) {
    const double nrm = sqrt(chain_dot(M + j, M + j, k, j, rows));  // the same in every lane
    if (nrm == 0.0) {
      if (lane == 0) s_vv[j] = 0.0;
      __syncthreads();
      continue;
    }
    const double ajj = M[(int64_t)j * k + j];
    const double alpha = ajj > 0.0 ? -nrm : nrm;
    for (int32_t i = j + lane; i < rows; i += 64)
      V[(int64_t)i * k + j] = i == j ? ajj - alpha : M[(int64_t)i * k + j];
    __syncthreads();
    const int c = j + lane;  // lane k - j: V.V
    const double t = c <= k ? chain_dot(V + j, c < k ? M + c : V + j, k, j, rows) : 0.0;
    const double d = __shfl(t, k - j);
    if (c < k) s_f[c] = (t + t) / d;
    if (lane == 0) s_vv[j] = d;
    __syncthreads();
    if (d != 0.0)
      for (int32_t i = j + lane; i < rows; i += 64) {
        const double v = V[(int64_t)i * k + j];
#pragma unroll 4
        for (int cc = j; cc < k; ++cc)
          M[(int64_t)i * k + cc] = M[(int64_t)i * k + cc] - s_f[cc] * v;
      }
    __syncthreads();
  }
  for (int j = k - 1; j >= 0; --j) {
    const double vj = s_vv[j];
    if (vj == 0.0) continue;  // block-uniform
    if (lane < k) {
      const double t = chain_dot(V + j, Q + lane, k, j, rows);
      s_f[lane] = (t + t) / vj;
    }
    __syncthreads();
    for (int32_t i = j + lane; i < rows; i += 64) {
      const double v = V[(int64_t)i * k + j];
#pragma unroll 4
      for (int c = 0; c < k; ++c)
        Q[(int64_t)i * k + c] = Q[(int64_t)i * k + c] - s_f[c] * v;
    }
    __syncthreads();
  }
  for (int32_t e = lane; e < k * k; e += 64) {  // R; its rows' signs go to Q's columns
    const int r = e / k, c = e % k;
    double rv = (c >= r) ? M[e] : 0.0;
    if (M[(int64_t)r * k + r] < 0.0) rv = -rv;
    Bc[(int64_t)J * k * k + e] = rv;
  }
  for (int32_t e = lane; e < rows * k; e += 64) {
    const int32_t q = e / k, c = e % k;
    const int64_t i = dof(q);
    ptcol[ptrp[i] + c] = J * k + c;
    ptval[ptrp[i] + c] = M[(int64_t)c * k + c] < 0.0 ? -Q[e] : Q[e];
  }
}

void tentative_qr(int32_t n, int32_t bs, int32_t k, const int32_t *agg, int32_t nc,
                  const double *B, Arena &ar, Csr &Pt, double *Bc, int32_t *err, int32_t ebit,
                  hipStream_t s) {
  if (k < 1 || k > kMaxBs) throw Error(SA_ERR_INVALID_ARG, "nullspace dimension not in 1..16");
  const int32_t m = n / bs;
  Arena tmp;
  tmp.stream = s;
  int32_t *cnt = tmp.alloc<int32_t>(n + 1);
  k_pt_count<<<grid_for(n), kBlock, 0, s>>>(n, bs, k, agg, cnt);
  SA_LAUNCH_CHECK();
  Pt.n = n;
  Pt.ncols = nc * k;
  Pt.rp = ar.alloc<int32_t>(n + 1);
  exclusive_scan_i32(cnt, Pt.rp, n, s);
  Pt.nnz = read1(Pt.rp + n, s);
  Pt.col = ar.alloc<int32_t>(Pt.nnz > 0 ? Pt.nnz : 1);
  Pt.val = ar.alloc<double>(Pt.nnz > 0 ? Pt.nnz : 1);
  if (nc <= 0) return;
  int32_t *mrp, *mem;
  member_lists(m, agg, nc, true, tmp, &mrp, &mem, s);
  // one wavefront per aggregate with M, V, Q in LDS when the largest aggregate fits 64 KB
  const int64_t maxrows = (int64_t)max_row_length(nc, mrp, s) * bs;
  const int64_t lds = 3 * maxrows * k * (int64_t)sizeof(double);
  if (lds <= (48 << 10)) {
    k_agg_qr_lds<<<(unsigned)nc, 64, (size_t)lds, s>>>(nc, bs, k, (int32_t)maxrows, mrp, mem, B,
                                                        Pt.rp, Pt.col, Pt.val, Bc, err, ebit);
    SA_LAUNCH_CHECK();
    return;
  }
  const int64_t sz = (int64_t)n * k;
  double *Ms = tmp.alloc<double>(sz), *Vs = tmp.alloc<double>(sz), *Qs = tmp.alloc<double>(sz);
  k_agg_qr<<<grid_for(nc), kBlock, 0, s>>>(nc, bs, k, mrp, mem, B, Pt.rp, Pt.col, Pt.val, Bc, Ms,
                                           Vs, Qs, err, ebit);
  SA_LAUNCH_CHECK();
}

// ---- smoothing: P = P_t - (omega invD_i) (Abar P_t)_i --------------------------------------------
// Eight lanes per row of P; a row of P_t holds its aggregate's columns, which are consecutive (or
// nothing), so an entry's place there is a subtraction.  (180K rows of about 26 entries: 184 us
// with a thread per row that searched P_t's row, now 29.)
__global__ __launch_bounds__(kBlock) void k_smooth_pt(
    int32_t n, const int32_t *__restrict__ aprp, const int32_t *__restrict__ apcol, double *apval,
    const int32_t *__restrict__ ptrp, const int32_t *__restrict__ ptcol,
    const double *__restrict__ ptval, const double *__restrict__ invD,
    const double *__restrict__ omega) {
  for (int64_t i = first_row<8>(); i < n; i += row_stride<8>()) {
    const double t = (*omega) * invD[i];
    const int32_t p0 = ptrp[i], np = ptrp[i + 1] - p0;
    const int32_t c0 = np > 0 ? ptcol[p0] : 0;
    const int32_t e1 = aprp[i + 1];
    for (int32_t e = aprp[i] + (threadIdx.x & 7); e < e1; e += 8) {
      const int32_t q = apcol[e] - c0;
      const double pt = q >= 0 && q < np ? ptval[p0 + q] : 0.0;
      apval[e] = pt - t * apval[e];
    }
  }
}
void smooth_tentative(const Csr &abar, const Csr &Pt, const double *invD, const double *omega,
                      Arena &ar, Csr &P, hipStream_t s) {
  spgemm(abar, Pt, ar, P, s);
  if (P.n > 0) {
    k_smooth_pt<<<grid_rows(P.n, 8), kBlock, 0, s>>>(P.n, P.rp, P.col, P.val, Pt.rp, Pt.col,
                                                    Pt.val, invD, omega);
    SA_LAUNCH_CHECK();
  }
}

}  // namespace sa
