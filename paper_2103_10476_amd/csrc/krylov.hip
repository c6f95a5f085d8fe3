// GMRES building blocks (restarted flexible GMRES, Sec. 3.4): multi-vector canonical inner
// products, Gram-Schmidt updates, the Hessenberg column, Givens rotations and the
// least-squares back substitution.  Scalar steps run in one thread on the device, in the
// order of the textbook algorithm, so the iterates match a sequential implementation bit for
// bit.
#include <algorithm>

#include "solve_device.hpp"

namespace sa {

// ---- GMRES building blocks ----------------------------------------------------------------
// Multi-vector canonical dot: the same blocks and trees as dot_f64, one per vector (grid.y).
__global__ __launch_bounds__(kDotBlock) void k_mdot_stage(const double *__restrict__ x,
                                                       int64_t ldx,
                                                       const double *__restrict__ y, int64_t m,
                                                       double *__restrict__ part,
                                                       int64_t ldp) {
  __shared__ DotShared sh;
  const int64_t v = blockIdx.y;
  dot_block(blockIdx.x, x + v * ldx, y, m, part + v * ldp + blockIdx.x, sh);
}
// Partials per vector that k_gmres_project reduces itself: every block of the basis' length
// reads those of every vector, nb blocks nb partials each, so their traffic grows with the square
// of the length (as much as the vectors' own at 4,096).  Beyond this a stage of one block per
// vector comes between, 4.5 us a pass (GMRES of 20 steps, without and with it: 1.2M and 2.1M
// unknowns 14.0 and 17.7 ms either way, 3.0M 26.5 and 26.3, 8.0M 72.5 and 70.7, 16.6M 165.6 and
// 157.0).
constexpr int64_t kProjectParts = 512;
static_assert(kProjectParts <= kDotFinal, "the projection takes one last stage");
// Stages of partials until at most kProjectParts are left per vector.
static DotParts multi_dot_parts(const double *V, int64_t ldv, int32_t nv, const double *w,
                                int64_t n, double *ws, hipStream_t s) {
  int64_t nb = std::max<int64_t>(ceil_div(n, kDotTerms), 1);
  k_mdot_stage<<<dim3((unsigned)nb, (unsigned)nv), kDotBlock, 0, s>>>(V, ldv, w, n, ws, nb);
  SA_LAUNCH_CHECK();
  while (nb > kProjectParts) {
    const int64_t nb2 = ceil_div(nb, kDotTerms);
    double *out = ws + nb * nv;
    k_mdot_stage<<<dim3((unsigned)nb2, (unsigned)nv), kDotBlock, 0, s>>>(ws, nb, nullptr, nb, out,
                                                                       nb2);
    SA_LAUNCH_CHECK();
    ws = out;
    nb = nb2;
  }
  return DotParts{ws, (int32_t)nb};
}
// The last stage of the canonical inner product by one wavefront (m <= 4096 partials; the same
// sums in the same order): lane l has the places l, l + 64, l + 128 and l + 192 of the 256.
// The result is lane 0's.
__device__ __forceinline__ double dot_final_wave(const double *__restrict__ part, int32_t m,
                                                 int lane) {
  double a[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    a[k] = 0.0;
    for (int32_t i = lane + 64 * k; i < m; i += 256) a[k] += part[i];
  }
  a[0] = a[0] + a[2];
  a[1] = a[1] + a[3];
  double v = a[0] + a[1];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = v + __shfl_down(v, off, 64);
  return v;
}
// One Gram-Schmidt pass: c_i = V_i . w from its partials (every block takes the last stage, a
// wavefront per vector), w -= c_0 V_0 + c_1 V_1 + ... in ascending order, column j of H by
// block 0, and with wpart the partials of the new w.w: a block has the elements of its block of
// the inner product.  V's traffic bounds it from some ten vectors on; before, the launches and
// their chain: 90^3 convection, 12 steps, the last stages (4.7 us), updates (9.8), column sums
// (3.8) and the norm's first stage (4.2) with a gap between each, now 13.1 in one.
__global__ __launch_bounds__(kDotBlock) void k_gmres_project(
    const double *__restrict__ V, int64_t ldv, int32_t nv, const double *__restrict__ part,
    int32_t np, double *H, int32_t m, int32_t pass, double *__restrict__ w, int64_t n,
    double *__restrict__ wpart) {
  constexpr int M = kDotTerms / kDotBlock;
  __shared__ double s_c[kMaxRestart];
  __shared__ DotShared sh;
  const int t = threadIdx.x;
  const int64_t base = (int64_t)blockIdx.x * kDotTerms + t;
  double x[M];  // loaded ahead of the reductions
#pragma unroll
  for (int q = 0; q < M; ++q) x[q] = base + kDotBlock * q < n ? w[base + kDotBlock * q] : 0.0;
  for (int32_t i = t >> 6; i < nv; i += kDotBlock / 64) {
    const double c = dot_final_wave(part + (int64_t)i * np, np, t & 63);
    if ((t & 63) == 0) s_c[i] = c;
  }
  __syncthreads();
  if (blockIdx.x == 0 && t < nv) {
    double *h = H + (int64_t)t * m + (nv - 1);
    *h = pass == 0 ? s_c[t] : *h + s_c[t];
  }
#pragma unroll 2
  for (int32_t i = 0; i < nv; ++i) {
    const double c = s_c[i];
    const double *v = V + i * ldv;
#pragma unroll
    for (int q = 0; q < M; ++q)
      if (base + kDotBlock * q < n) x[q] = x[q] - c * v[base + kDotBlock * q];
  }
#pragma unroll
  for (int q = 0; q < M; ++q) {
    if (base + kDotBlock * q < n) w[base + kDotBlock * q] = x[q];
    sh.term[t + kDotBlock * q] = base + kDotBlock * q < n ? x[q] * x[q] : 0.0;
  }
  if (!wpart) return;  // uniform
  const double s = dot_sum_terms(sh);
  if (t == 0) wpart[blockIdx.x] = s;
}
DotParts gmres_project(const double *V, int64_t ldv, int32_t nv, double *ws, double *H, int32_t m,
                       int32_t pass, double *w, int64_t n, double *wpart, hipStream_t s) {
  const DotParts c = multi_dot_parts(V, ldv, nv, w, n, ws, s);
  const int64_t nb = std::max<int64_t>(ceil_div(n, kDotTerms), 1);
  k_gmres_project<<<(unsigned)nb, kDotBlock, 0, s>>>(V, ldv, nv, c.p, c.m, H, m, pass, w, n,
                                                    wpart);
  SA_LAUNCH_CHECK();
  return wpart ? reduce_parts(wpart, nb, wpart + nb, s, 2048) : DotParts{};
}
__global__ void k_multi_axpy(const double *__restrict__ V, int64_t ldv, int32_t nv,
                             const double *__restrict__ c, double *__restrict__ w, int64_t n) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  double t = w[k];
  for (int32_t i = 0; i < nv; ++i) t = t + c[i] * V[i * ldv + k];
  w[k] = t;
}
void multi_axpy_f64(const double *V, int64_t ldv, int32_t nv, const double *c, double *w,
                    int64_t n, hipStream_t s) {
  if (n <= 0 || nv <= 0) return;
  k_multi_axpy<<<grid_for(n), kBlock, 0, s>>>(V, ldv, nv, c, w, n);
  SA_LAUNCH_CHECK();
}
__global__ void k_div_scalar(const double *w, double *v, int64_t n, const double *den) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const double d = *den;
  if (k < n && d > 0.0) v[k] = w[k] / d;
}
// Rotations of column j (c[0..j] in LDS, hn below it) and the new one, by one thread; cs and sn
// are LDS copies too, so the chain of rotations waits for no memory.
__device__ void gmres_givens(const double *c, double hn, const double *lcs, const double *lsn,
                             double *H, int32_t m, int32_t j, double *cs, double *sn, double *g,
                             GmresScalars *S) {
  double a = c[0];  // h(i, j) as the rotations before i left it
  for (int32_t i = 0; i < j; ++i) {
    const double next = c[i + 1];
    H[(int64_t)i * m + j] = lcs[i] * a + lsn[i] * next;
    a = -lsn[i] * a + lcs[i] * next;
  }
  const double gj = g[j];
  double cj = 1.0, sj = 0.0;
  if (hn != 0.0) {
    const double rho = sqrt(a * a + hn * hn);
    cj = a / rho;
    sj = hn / rho;
  }
  cs[j] = cj;
  sn[j] = sj;
  H[(int64_t)j * m + j] = cj * a + sj * hn;
  H[(int64_t)(j + 1) * m + j] = 0.0;
  g[j + 1] = -sj * gj;
  g[j] = cj * gj;
  S->res = fabs(-sj * gj);
}
// The new basis vector v = w / hn (hn from the partials of w.w; in place), the next
// preconditioner application's first step on it, and by block 0 column j's rotations and the
// scalars, posted to the host words if there are any (11 us, against 24 and five gaps for the
// norm's last stage, its root, the division, the rotations, the readback and the first step).
template <class First>
__global__ __launch_bounds__(kDotBlock) void k_gmres_next(
    const double *__restrict__ part, int32_t np, double *__restrict__ w, int64_t n, double *H,
    int32_t m, int32_t j, double *cs, double *sn, double *g, GmresScalars *S, First first,
    HostWords host) {
  constexpr int M = kDotTerms / kDotBlock;
  __shared__ double s_hn2;
  __shared__ double s_h[kMaxRestart], s_cs[kMaxRestart], s_sn[kMaxRestart];
  const int t = threadIdx.x;
  if (blockIdx.x == 0 && t <= j) {
    s_h[t] = H[(int64_t)t * m + j];
    s_cs[t] = t < j ? cs[t] : 0.0;
    s_sn[t] = t < j ? sn[t] : 0.0;
  }
  const int64_t base = (int64_t)blockIdx.x * kDotTerms + t;
  double x[M];
#pragma unroll
  for (int q = 0; q < M; ++q) x[q] = base + kDotBlock * q < n ? w[base + kDotBlock * q] : 0.0;
  if (t < 64) {
    const double hn2 = dot_final_wave(part, np, t);
    if (t == 0) s_hn2 = hn2;
  }
  __syncthreads();
  const double hn = sqrt(s_hn2);
#pragma unroll
  for (int q = 0; q < M; ++q) {
    const int64_t i = base + kDotBlock * q;
    if (i < n && hn > 0.0) {
      const double v = x[q] / hn;
      w[i] = v;
      first(i, v);
    }
  }
  if (blockIdx.x != 0) return;
  if (t == 0) {
    S->hn2 = s_hn2;
    S->hn = hn;
    gmres_givens(s_h, hn, s_cs, s_sn, H, m, j, cs, sn, g, S);
  }
  __syncthreads();
  if (host.dev) post_words(host, (const uint32_t *)S, (int32_t)(sizeof(GmresScalars) / 4));
}
template <class First>
void gmres_next(const DotParts &ww, double *w, int64_t n, double *H, int32_t m, int32_t j,
                double *cs, double *sn, double *g, GmresScalars *S, const First &first,
                const HostWords &host, hipStream_t s) {
  const int64_t nb = std::max<int64_t>(ceil_div(n, kDotTerms), 1);
  k_gmres_next<<<(unsigned)nb, kDotBlock, 0, s>>>(ww.p, ww.m, w, n, H, m, j, cs, sn, g, S, first,
                                                 host);
  SA_LAUNCH_CHECK();
}
#define SA_INST_NEXT(F)                                                                        \
  template void gmres_next<F>(const DotParts &, double *, int64_t, double *, int32_t, int32_t, \
                              double *, double *, double *, GmresScalars *, const F &,        \
                              const HostWords &, hipStream_t);
SA_INST_NEXT(FirstNone)
SA_INST_NEXT(FirstCheb64)
SA_INST_NEXT(FirstCheb32)
#undef SA_INST_NEXT
__global__ void k_gmres_backsolve(const double *H, int32_t m, int32_t k, const double *g,
                                  double *y, GmresScalars *S) {
  for (int32_t i = k - 1; i >= 0; --i) {
    double t = g[i];
    for (int32_t q = i + 1; q < k; ++q) t = t - H[(int64_t)i * m + q] * y[q];
    const double d = H[(int64_t)i * m + i];
    if (d == 0.0) S->err = 1;
    y[i] = t / d;
  }
}
void gmres_backsolve(const double *H, int32_t m, int32_t k, const double *g, double *y,
                     GmresScalars *S, hipStream_t s) {
  k_gmres_backsolve<<<1, 1, 0, s>>>(H, m, k, g, y, S);
  SA_LAUNCH_CHECK();
}
// (every entry of H and g that a cycle reads is written by that cycle first)
__global__ void k_gmres_beta(GmresScalars *S, double *g) {
  const double beta = sqrt(S->nrm2);
  S->beta = beta;
  g[0] = beta;
}
void gmres_start(GmresScalars *S, const double *r, double *v, int64_t n, double *g,
                 hipStream_t s) {
  k_gmres_beta<<<1, 1, 0, s>>>(S, g);
  k_div_scalar<<<grid_for(n), kBlock, 0, s>>>(r, v, n, &S->beta);
  SA_LAUNCH_CHECK();
}

}  // namespace sa
