// Coarsest level (Sec. 3.1: a direct solve once the hierarchy reaches <= 1000 unknowns, or
// a level left without strong connections): blocked dense Cholesky A_L = L L^T with the
// trailing updates on the FP64 matrix cores, L^{-1} by blocks (the off-diagonal blocks on
// the matrix cores), and A_L^{-1} = L^{-T} L^{-1} on the matrix cores (v_mfma_f64_16x16x4f64).
// Nonsymmetric operators (GMRES, Sec. 3.4) take a blocked LU without pivoting instead,
// A_L = L U, and A_L^{-1} = U^{-1} L^{-1} = W^T L^{-1} with W = (U^T)^{-1}.
// The V-cycle then applies A_L^{-1} as a dense GEMV.  The factor's rounding order differs
// from a sequential factorization, so this is the one setup result that matches a CPU
// reference to rounding (~1e-16 relative) rather than bit for bit.
#include "kernels.hpp"

namespace sa {

typedef double v4d __attribute__((ext_vector_type(4)));

// A wavefront per row (a thread per row took 76 us on 569 rows of 80 entries).
__global__ __launch_bounds__(kBlock) void k_dense_scatter(int32_t n, int32_t ld,
                                                          const int32_t *rp, const int32_t *col,
                                                          const double *val, double *D) {
  const int64_t i = ((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 6;
  if (i >= n) return;
  for (int32_t k = rp[i] + (int32_t)(threadIdx.x & 63); k < rp[i + 1]; k += 64)
    D[i * ld + col[k]] = val[k];
}

// ---- blocked right-looking Cholesky, 64 x 64 blocks ---------------------------------------
// D is ld x ld row-major (ld a multiple of 64) and holds the matrix in its lower triangle;
// rows and columns n..ld-1 are an identity pad, so every block is full.  Step kb factors the
// diagonal block, solves the panel below it, and updates the trailing lower triangle on the
// FP64 matrix cores.  The factor's rounding order differs from the sequential textbook
// Cholesky; the result is checked against a dense inverse to ~1e-16 relative.
constexpr int kNB = 64;

__global__ void k_pad_identity(int32_t n, int32_t ld, double *D) {
  const int32_t i = n + blockIdx.x * blockDim.x + threadIdx.x;
  if (i < ld) D[(int64_t)i * ld + i] = 1.0;
}

// 16 x 16 block product by one wavefront: acc += A B with A[r][k] = a[r * lda + k] and
// B[k][c] = b[k * ldk + c * ldc], k = 0..K-1 (lane l supplies A[l%16][l/16] and B[l/16][l%16] of
// each 4-deep step and receives rows 4v + l/16, column l%16 of the product in register v).
template <int K>
__device__ __forceinline__ v4d mfma_16(const double *a, int lda, const double *b, int ldk, int ldc,
                                       v4d acc) {
  const int lr = threadIdx.x & 15, lk = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int k = 0; k < K; k += 4)
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[lr * lda + k + lk], b[(k + lk) * ldk + lr * ldc],
                                              acc, 0, 0, 0);
  return acc;
}
// c[r * ldc + col] = sign acc (+ c when add).
__device__ __forceinline__ void put_16(double *c, int ldc, v4d acc, double sign, bool add) {
  const int lr = threadIdx.x & 15, lk = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    double *q = c + (4 * v + lk) * ldc + lr;
    *q = add ? *q + sign * acc[v] : sign * acc[v];
  }
}

// The lower-left H x H block at (o + H, o) of a triangular inverse from its two diagonal blocks,
// tile (ti, tj) by this wavefront (live: it has one): Z = -X22 Y with Y = L21 X11, then
// Z -= X22 (Y + L22 Z).  Without the correction the inverse's residual L X - I is 50 to 10,000
// times that of a forward substitution by columns, and so is the error of L^{-1} from there on;
// with it they are the same.  t: H x H scratch.
template <int H>
__device__ __forceinline__ void trtri_corner(const double (*l)[kNB + 1], double (*x)[kNB + 1],
                                             double *t, int o, int ti, int tj, bool live) {
  constexpr int LD = kNB + 1;
  const v4d zero = {0.0, 0.0, 0.0, 0.0};
  double *z = &x[o + H + ti][o + tj], *tt = t + ti * 33 + tj;
  const double *x22 = &x[o + H + ti][o + H];
  v4d y = zero;
  if (live) {
    y = mfma_16<H>(&l[o + H + ti][o], LD, &x[o][o + tj], LD, 1, zero);
    put_16(tt, 33, y, 1.0, false);
  }
  __syncthreads();
  if (live) put_16(z, LD, mfma_16<H>(x22, LD, t + tj, 33, 1, zero), -1.0, false);
  __syncthreads();
  if (live) {
    y = mfma_16<H>(&l[o + H + ti][o + H], LD, &x[o + H][o + tj], LD, 1, y);
    put_16(tt, 33, y, 1.0, false);
  }
  __syncthreads();
  if (live) put_16(z, LD, mfma_16<H>(x22, LD, t + tj, 33, 1, zero), -1.0, true);
  __syncthreads();
}

// Inverse of the lower-triangular 64 x 64 block l into x (both with leading dimension
// kNB + 1 in LDS, zero above their diagonals, rd[i] = 1 / l[i][i]): the four 16 x 16 diagonal
// blocks by forward substitution, a wavefront each (lane c: column c), then the corners of the
// two 32 x 32 halves and of the whole block on the matrix cores.
__device__ __forceinline__ void trtri_64(const double (*l)[kNB + 1], double (*x)[kNB + 1],
                                         const double *rd, double (*t)[33]) {
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  for (int q = tid; q < kNB * kNB; q += 256) x[q / kNB][q % kNB] = 0.0;
  __syncthreads();
  if (lane < 16) {
    const int o = 16 * w;
    double y[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      double v = i == lane ? 1.0 : 0.0;
#pragma unroll
      for (int k = 0; k < i; ++k) v = __builtin_fma(-l[o + i][o + k], y[k], v);
      y[i] = v * rd[o + i];
    }
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (i >= lane) x[o + i][o + lane] = y[i];
  }
  __syncthreads();
  trtri_corner<16>(l, x, &t[16 * (w & 1)][0], 32 * (w & 1), 0, 0, w < 2);
  trtri_corner<32>(l, x, &t[0][0], 0, 16 * (w >> 1), 16 * (w & 1), true);
}

// 1 / sqrt(d) to about an ulp: the hardware estimate and three Newton steps.
__device__ __forceinline__ double rsqrt_newton(double d) {
  double y = __builtin_amdgcn_rsq(d);
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const double h = 0.5 * y;
    y = __builtin_fma(h, __builtin_fma(-d * y, y, 1.0), y);
  }
  return y;
}

// Diagonal block at (k0, k0): its Cholesky factor L_kk and the inverse of that (into Li), err
// bit 64 on a pivot <= 0.  Four panels of 16 columns: wavefront 0 holds a row per lane, 16
// columns of it in registers, and takes the columns one by one (the pivot and the pivot
// row's entries are read across lanes); the columns to the right of the panel are updated on
// the matrix cores, 16 x 16 tiles.  What bounds it is the chain of 64 pivots, about 150 cycles
// each.  The inverse turns the panel solve below into a product and is what the triangular
// inverse starts from.  (Column by column over the whole block in LDS, three barriers each,
// took 73 us, and the inverse, a column per thread, 50 us in a launch of its own; both now
// 26.0 us, of which the corners' corrections are 2.3.)
__global__ __launch_bounds__(256) void k_potrf_inv(int32_t ld, int32_t k0, double *D, double *Li,
                                                   int32_t *err) {
  __shared__ double a[kNB][kNB + 1], x[kNB][kNB + 1];
  __shared__ double t[32][33];
  __shared__ double rd[kNB];
  constexpr int LD = kNB + 1;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  for (int q = tid; q < kNB * kNB; q += 256) {
    const int i = q / kNB, j = q % kNB;
    a[i][j] = (j <= i) ? D[(int64_t)(k0 + i) * ld + k0 + j] : 0.0;
  }
  __syncthreads();
  for (int p = 0; p < kNB; p += 16) {
    if (w == 0) {
      double r[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) r[j] = a[lane][p + j];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const double d = __shfl(r[j], p + j, 64);
        const double y = rsqrt_newton(d);
        if (lane == p + j) {
          if (!(d > 0.0)) atomicOr(err, 64);
          rd[p + j] = y;
        }
        r[j] = r[j] * y;
#pragma unroll
        for (int k = j + 1; k < 16; ++k)
          r[k] = __builtin_fma(-r[j], __shfl(r[j], p + k, 64), r[k]);
      }
#pragma unroll
      for (int j = 0; j < 16; ++j)
        if (lane >= p + j) a[lane][p + j] = r[j];
    }
    __syncthreads();
    // tiles (ti, tj) of the columns to the right, ti >= tj > p / 16
    int q = 0;
    for (int ti = p + 16; ti < kNB; ti += 16)
      for (int tj = p + 16; tj <= ti; tj += 16)
        if ((q++ & 3) == w) {
          const v4d acc = mfma_16<16>(&a[ti][p], LD, &a[tj][p], 1, LD, v4d{0.0, 0.0, 0.0, 0.0});
          put_16(&a[ti][tj], LD, acc, -1.0, true);
        }
    __syncthreads();
  }
  // (the updates of the diagonal tiles wrote above the diagonal too)
  for (int q = tid; q < kNB * kNB; q += 256)
    if (q % kNB > q / kNB) a[q / kNB][q % kNB] = 0.0;
  trtri_64(a, x, rd, t);
  for (int q = tid; q < kNB * kNB; q += 256) {
    const int i = q / kNB, j = q % kNB;
    if (j <= i) D[(int64_t)(k0 + i) * ld + k0 + j] = a[i][j];
    Li[(int64_t)(k0 + i) * ld + k0 + j] = x[i][j];
  }
}

// A 16 x 64 strip times the transpose of a lower-triangular 64 x 64 block, out[ct] = a b^T for
// the column tiles ct, each as deep as the triangle (leading dimensions kNB + 1).
__device__ __forceinline__ void strip_times_lower_t(const double *a, const double (*b)[kNB + 1],
                                                    v4d (&out)[4]) {
  constexpr int LD = kNB + 1;
  const v4d zero = {0.0, 0.0, 0.0, 0.0};
  out[0] = mfma_16<16>(a, LD, &b[0][0], 1, LD, zero);
  out[1] = mfma_16<32>(a, LD, &b[16][0], 1, LD, zero);
  out[2] = mfma_16<48>(a, LD, &b[32][0], 1, LD, zero);
  out[3] = mfma_16<64>(a, LD, &b[48][0], 1, LD, zero);
}

// Panel below the diagonal block: L_ik = A_ik L_kk^{-T}, a 64 x 64 block per workgroup on the
// matrix cores, in place.  The product with the explicit inverse alone leaves a residual that
// grows with the condition of L_kk (the factor's backward error 1e-15 to 3e-12 on Gaussian
// kernels, and pivots lost from a condition of about 1e12 on), so one correction follows:
// Q = A X^T with X = L_kk^{-1}, then Q += (A - Q L_kk^T) X^T, which brings the backward error
// to forward substitution's (2e-16).  A wavefront works on its own 16 rows throughout.  The step's
// launch takes 15.1 us (9 blocks), 9.2 without the correction; substitution, a row per thread,
// took 31.
__device__ __forceinline__ void panel_tile(int32_t blk, int32_t ld, int32_t k0, const double *Li,
                                           double *D, double (*As)[kNB + 1],
                                           double (*Xs)[kNB + 1], double (*Ls)[kNB + 1]) {
  constexpr int LD = kNB + 1;
  const int tid = threadIdx.x, w = tid >> 6;
  const int64_t r0 = (int64_t)k0 + (int64_t)kNB * (1 + blk);
  for (int q = tid; q < kNB * kNB; q += 256) {
    const int r = q / kNB, k = q % kNB;
    As[r][k] = D[(r0 + r) * ld + k0 + k];
    Xs[r][k] = Li[(int64_t)(k0 + r) * ld + k0 + k];
    Ls[r][k] = k <= r ? D[(int64_t)(k0 + r) * ld + k0 + k] : 0.0;
  }
  __syncthreads();
  const int lr = tid & 15, lk = (tid & 63) >> 4;
  double *strip = &As[16 * w][0];
  v4d a[4], l[4], d[4];
#pragma unroll
  for (int ct = 0; ct < 4; ++ct)
#pragma unroll
    for (int v = 0; v < 4; ++v) a[ct][v] = strip[(4 * v + lk) * LD + 16 * ct + lr];
  strip_times_lower_t(strip, Xs, l);
  __syncthreads();
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) put_16(strip + 16 * ct, LD, l[ct], 1.0, false);
  __syncthreads();
  strip_times_lower_t(strip, Ls, d);
  __syncthreads();
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) put_16(strip + 16 * ct, LD, a[ct] - d[ct], 1.0, false);
  __syncthreads();
  strip_times_lower_t(strip, Xs, d);
#pragma unroll
  for (int ct = 0; ct < 4; ++ct)
#pragma unroll
    for (int v = 0; v < 4; ++v)
      D[(r0 + 16 * w + 4 * v + lk) * ld + k0 + 16 * ct + lr] = l[ct][v] + d[ct][v];
}

// Trailing update after step kb: D[ib][jb] -= L[ib][kb] L[jb][kb]^T for every block pair
// kb < jb <= ib < nbk (workgroup t = the t-th pair, row-major over the lower triangle).  The
// two 64 x 64 panels are staged in LDS; each of the 4 wavefronts computes a 16 x 64 strip
// as four 16 x 16 tiles with v_mfma_f64_16x16x4f64 (lane l supplies A[l%16][l/16] and
// B[l/16][l%16] and receives D[4v + l/16][l%16] in result register v).  Diagonal blocks are
// updated whole; their upper parts are never read.
__device__ __forceinline__ void syrk_tile(int64_t t, int32_t ld, int32_t kb, int32_t nbk, double *D,
                                          double (*As)[kNB + 1], double (*Bs)[kNB + 1]) {
  int32_t a = (int32_t)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
  while ((int64_t)a * (a + 1) / 2 > t) --a;
  while ((int64_t)(a + 1) * (a + 2) / 2 <= t) ++a;
  const int32_t b = (int32_t)(t - (int64_t)a * (a + 1) / 2);
  const int32_t ib = kb + 1 + a, jb = kb + 1 + b;
  if (ib >= nbk || jb > ib) return;  // block-uniform; the grid holds exactly the pairs
  const int64_t r0 = (int64_t)ib * kNB, c0 = (int64_t)jb * kNB, k0 = (int64_t)kb * kNB;
  const int tid = threadIdx.x;
  for (int q = tid; q < kNB * kNB; q += 256) {
    const int r = q / kNB, k = q % kNB;
    As[r][k] = D[(r0 + r) * ld + k0 + k];
    Bs[r][k] = D[(c0 + r) * ld + k0 + k];
  }
  __syncthreads();
  const int w = tid >> 6, lane = tid & 63;
  const int lr = lane & 15, lk = lane >> 4;
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) {
    v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int kk = 0; kk < kNB; kk += 4) {
      const double av = As[16 * w + lr][kk + lk];
      const double bv = Bs[16 * ct + lr][kk + lk];
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t row = r0 + 16 * w + 4 * v + lk;
      const int64_t col = c0 + 16 * ct + lr;
      D[row * ld + col] -= acc[v];
    }
  }
}

// ---- blocked inverse of the triangular factor, Li = L^{-1} ------------------------------------
// Step 0 inverts every 64 x 64 diagonal block.  Then L X = I is solved by right-looking block
// forward substitution with the whole identity as right-hand side, in place in Li (zero
// below the diagonal blocks to start with): for block row ib = 0, 1, ..., its tiles are
// finalised, X[ib][kb] = Li[ib][ib] B[ib][kb] (kb < ib), and every later block row is
// updated, B[i][kb] -= L[i][ib] X[ib][kb] (i > ib, kb <= ib).  Each launch is one tile
// product deep, so the dependent chain is two launches per block row.

// 64 x 64 product on the matrix cores: wavefront w accumulates rows 16w..16w+15 of As * Bs
// (As[r][k] = A[r][k], Bs[k][c] = B[k][c]) into acc[ct] for column tile ct.
__device__ __forceinline__ void mfma_64(const double (*As)[kNB + 1], const double (*Bs)[kNB + 1],
                                        v4d *acc) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int lr = lane & 15, lk = lane >> 4;
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) {
#pragma unroll
    for (int kk = 0; kk < kNB; kk += 4) {
      const double av = As[16 * w + lr][kk + lk];
      const double bv = Bs[kk + lk][16 * ct + lr];
      acc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc[ct], 0, 0, 0);
    }
  }
}

__global__ __launch_bounds__(256) void k_trtri_diag(int32_t ld, const double *L, double *Li,
                                                    bool unit) {
  __shared__ double l[kNB][kNB + 1];
  __shared__ double x[kNB][kNB + 1];
  const int tid = threadIdx.x;
  const int64_t k0 = (int64_t)blockIdx.x * kNB;
  for (int q = tid; q < kNB * kNB; q += 256) {
    const int i = q / kNB, j = q % kNB;
    l[i][j] = (j < i || (j == i && !unit)) ? L[(k0 + i) * ld + k0 + j] : (j == i ? 1.0 : 0.0);
    x[i][j] = 0.0;
  }
  __syncthreads();
  if (tid < kNB) {  // column c of the block's inverse by forward substitution
    const int c = tid;
    x[c][c] = 1.0 / l[c][c];
    for (int i = c + 1; i < kNB; ++i) {
      double t = 0.0;
      for (int k = c; k < i; ++k) t += l[i][k] * x[k][c];
      x[i][c] = -t / l[i][i];
    }
  }
  __syncthreads();
  for (int q = tid; q < kNB * kNB; q += 256) {
    const int i = q / kNB, j = q % kNB;
    Li[(k0 + i) * ld + k0 + j] = x[i][j];
  }
}

// X[ib][kb] = Li[ib][ib] B[ib][kb] for kb = blk < ib.
__device__ __forceinline__ void trinv_finalize_tile(int32_t blk, int32_t ld, int32_t ib, double *Li,
                                                    double (*As)[kNB + 1],
                                                    double (*Bs)[kNB + 1]) {
  const int tid = threadIdx.x;
  const int64_t r0 = (int64_t)ib * kNB, c0 = (int64_t)blk * kNB;
  for (int q = tid; q < kNB * kNB; q += 256) {
    const int r = q / kNB, k = q % kNB;
    As[r][k] = Li[(r0 + r) * ld + r0 + k];  // Li[ib][ib] (zero above its diagonal)
    Bs[r][k] = Li[(r0 + r) * ld + c0 + k];  // B[ib][kb]
  }
  __syncthreads();
  v4d acc[4];
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) acc[ct] = v4d{0.0, 0.0, 0.0, 0.0};
  mfma_64(As, Bs, acc);
  const int w = tid >> 6, lane = tid & 63;
  const int lr = lane & 15, lk = lane >> 4;
#pragma unroll
  for (int ct = 0; ct < 4; ++ct)
#pragma unroll
    for (int v = 0; v < 4; ++v)
      Li[(r0 + 16 * w + 4 * v + lk) * ld + c0 + 16 * ct + lr] = acc[ct][v];
}

// B[i][kb] -= L[i][ib] X[ib][kb] for every tile i > ib, kb <= ib (block t: i = ib+1+t/(ib+1),
// kb = t mod (ib+1)); each tile has one writer per launch.
__device__ __forceinline__ void trinv_update_tile(int64_t blk, int32_t ld, int32_t ib,
                                                  const double *L, double *Li,
                                                  double (*As)[kNB + 1], double (*Bs)[kNB + 1]) {
  const int tid = threadIdx.x;
  const int32_t i = ib + 1 + (int32_t)(blk / (ib + 1));
  const int32_t kb = (int32_t)(blk % (ib + 1));
  const int64_t r0 = (int64_t)i * kNB, j0 = (int64_t)ib * kNB, c0 = (int64_t)kb * kNB;
  for (int q = tid; q < kNB * kNB; q += 256) {
    const int r = q / kNB, k = q % kNB;
    As[r][k] = L[(r0 + r) * ld + j0 + k];   // L[i][ib]
    Bs[r][k] = Li[(j0 + r) * ld + c0 + k];  // X[ib][kb]
  }
  __syncthreads();
  v4d acc[4];
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) acc[ct] = v4d{0.0, 0.0, 0.0, 0.0};
  mfma_64(As, Bs, acc);
  const int w = tid >> 6, lane = tid & 63;
  const int lr = lane & 15, lk = lane >> 4;
#pragma unroll
  for (int ct = 0; ct < 4; ++ct)
#pragma unroll
    for (int v = 0; v < 4; ++v)
      Li[(r0 + 16 * w + 4 * v + lk) * ld + c0 + 16 * ct + lr] -= acc[ct][v];
}

__global__ __launch_bounds__(256) void k_trinv_finalize(int32_t ld, int32_t ib, double *Li) {
  __shared__ double As[kNB][kNB + 1], Bs[kNB][kNB + 1];
  trinv_finalize_tile((int32_t)blockIdx.x, ld, ib, Li, As, Bs);
}
__global__ __launch_bounds__(256) void k_trinv_update(int32_t ld, int32_t ib, const double *L,
                                                      double *Li) {
  __shared__ double As[kNB][kNB + 1], Bs[kNB][kNB + 1];
  trinv_update_tile(blockIdx.x, ld, ib, L, Li, As, Bs);
}

// Li = L^{-1} (Li zero outside the diagonal blocks, which k_trtri_diag has filled).
static void trinv_blocks(int32_t ld, int32_t nbk, const double *L, double *Li, hipStream_t s) {
  for (int32_t ib = 0; ib < nbk; ++ib) {
    if (ib > 0) k_trinv_finalize<<<(unsigned)ib, 256, 0, s>>>(ld, ib, Li);
    const int64_t tiles = (int64_t)(nbk - ib - 1) * (ib + 1);
    if (tiles > 0) k_trinv_update<<<(unsigned)tiles, 256, 0, s>>>(ld, ib, L, Li);
  }
  SA_LAUNCH_CHECK();
}

// Cholesky and the triangular inverse in step: block row kb of the inverse needs nothing
// beyond step kb of the factorisation, so each step is three launches, the diagonal block
// (k_potrf_inv), then the panel tiles L[i][kb] with the inverse's tiles X[kb][j] (j < kb), then
// the trailing updates with the updates B[i][j] -= L[i][kb] X[kb][j] of the rows below.  The
// launches are a few microseconds of work each (13-26 us for nbk = 9), so fewer of them is what
// counts.
__global__ __launch_bounds__(256) void k_step_panels(int32_t ld, int32_t kb, int32_t nbk,
                                                     double *D, double *Li) {
  __shared__ double As[kNB][kNB + 1], Bs[kNB][kNB + 1], Cs[kNB][kNB + 1];
  const int32_t m = nbk - kb - 1, t = (int32_t)blockIdx.x;
  if (t < m) panel_tile(t, ld, kb * kNB, Li, D, As, Bs, Cs);
  else trinv_finalize_tile(t - m, ld, kb, Li, As, Bs);
}
__global__ __launch_bounds__(256) void k_step_updates(int32_t ld, int32_t kb, int32_t nbk,
                                                      double *D, double *Li) {
  __shared__ double As[kNB][kNB + 1], Bs[kNB][kNB + 1];
  const int64_t m = nbk - kb - 1, pairs = m * (m + 1) / 2, t = blockIdx.x;
  if (t < pairs) syrk_tile(t, ld, kb, nbk, D, As, Bs);
  else trinv_update_tile(t - pairs, ld, kb, D, Li, As, Bs);
}
static void chol_inverse(int32_t ld, int32_t nbk, double *D, double *Li, int32_t *err,
                         hipStream_t s) {
  for (int32_t kb = 0; kb < nbk; ++kb) {
    k_potrf_inv<<<1, 256, 0, s>>>(ld, kb * kNB, D, Li, err);
    const int64_t m = nbk - kb - 1;
    if (m + kb > 0) k_step_panels<<<(unsigned)(m + kb), 256, 0, s>>>(ld, kb, nbk, D, Li);
    const int64_t tiles = m * (m + 1) / 2 + m * (kb + 1);
    if (tiles > 0) k_step_updates<<<(unsigned)tiles, 256, 0, s>>>(ld, kb, nbk, D, Li);
  }
  SA_LAUNCH_CHECK();
}

// C = X^T Y for lower-triangular X and Y (ld x ld, zero above the diagonal; Cholesky:
// X = Y = L^{-1}; LU: X = (U^T)^{-1}, Y = L^{-1}), n x n row-major output.  Tile (ib, jb)
// of 64 x 64 sums X[kb][ib]^T Y[kb][jb] over kb >= max(ib, jb) (the other tiles are zero),
// both tiles staged in LDS (X transposed on the way in) and multiplied on the matrix cores.
// sym: X = Y, so only tiles ib >= jb are computed and the off-diagonal ones are also written
// transposed.
// Block t enumerates the tile pairs row-major (the lower triangle when sym).
__global__ __launch_bounds__(256) void k_gram_tiles(int32_t n, int32_t ld, int32_t nbk,
                                                    const double *X, const double *Y,
                                                    double *C, bool sym) {
  __shared__ double As[kNB][kNB + 1];
  __shared__ double Bs[kNB][kNB + 1];
  const int64_t t = blockIdx.x;
  int32_t ib, jb;
  if (sym) {
    int32_t a = (int32_t)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
    while ((int64_t)a * (a + 1) / 2 > t) --a;
    while ((int64_t)(a + 1) * (a + 2) / 2 <= t) ++a;
    ib = a;
    jb = (int32_t)(t - (int64_t)a * (a + 1) / 2);
  } else {
    ib = (int32_t)(t / nbk);
    jb = (int32_t)(t % nbk);
  }
  const int tid = threadIdx.x;
  const int64_t i0 = (int64_t)ib * kNB, j0 = (int64_t)jb * kNB;
  v4d acc[4];
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) acc[ct] = v4d{0.0, 0.0, 0.0, 0.0};
  for (int32_t kb = ib > jb ? ib : jb; kb < nbk; ++kb) {
    const int64_t k0 = (int64_t)kb * kNB;
    for (int q = tid; q < kNB * kNB; q += 256) {
      const int k = q / kNB, c = q % kNB;
      As[c][k] = X[(k0 + k) * ld + i0 + c];  // A[r][k] = X[k][r]
      Bs[k][c] = Y[(k0 + k) * ld + j0 + c];
    }
    __syncthreads();
    mfma_64(As, Bs, acc);
    __syncthreads();
  }
  const int w = tid >> 6, lane = tid & 63;
  const int lr = lane & 15, lk = lane >> 4;
#pragma unroll
  for (int ct = 0; ct < 4; ++ct)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t row = i0 + 16 * w + 4 * v + lk, col = j0 + 16 * ct + lr;
      if (row < n && col < n) {
        C[row * n + col] = acc[ct][v];
        // a diagonal tile holds both (r, c) and (c, r): each is written once, by its own lane
        if (sym && ib != jb) C[col * n + row] = acc[ct][v];
      }
    }
}

static void gram(int32_t n, int32_t ld, int32_t nbk, const double *X, const double *Y,
                 double *C, bool sym, hipStream_t s) {
  const int64_t tiles = sym ? (int64_t)nbk * (nbk + 1) / 2 : (int64_t)nbk * nbk;
  k_gram_tiles<<<(unsigned)tiles, 256, 0, s>>>(n, ld, nbk, X, Y, C, sym);
  SA_LAUNCH_CHECK();
}

// ---- blocked right-looking LU without pivoting, 64 x 64 blocks --------------------------------
// D holds the whole matrix (identity pad).  Step kb factors the diagonal block (unit L below,
// U on and above), solves the row panel U12 = L11^{-1} A12 and the column panel
// L21 = A21 U11^{-1}, and updates the whole trailing matrix A22 -= L21 U12 on the matrix
// cores.  err bit 64 on a zero or non-finite pivot.
__global__ __launch_bounds__(256) void k_getrf_diag(int32_t ld, int32_t k0, double *D,
                                                    int32_t *err) {
  __shared__ double a[kNB][kNB + 1];
  const int tid = threadIdx.x;
  for (int q = tid; q < kNB * kNB; q += 256) {
    const int i = q / kNB, j = q % kNB;
    a[i][j] = D[(int64_t)(k0 + i) * ld + k0 + j];
  }
  __syncthreads();
  for (int j = 0; j < kNB; ++j) {
    const double piv = a[j][j];
    if (tid == 0 && (!(piv != 0.0) || !isfinite(piv))) atomicOr(err, 64);
    for (int i = j + 1 + tid; i < kNB; i += 256) a[i][j] /= piv;
    __syncthreads();
    for (int q = tid; q < kNB * kNB; q += 256) {
      const int i = q / kNB, k = q % kNB;
      if (i > j && k > j) a[i][k] -= a[i][j] * a[j][k];
    }
    __syncthreads();
  }
  for (int q = tid; q < kNB * kNB; q += 256) {
    const int i = q / kNB, j = q % kNB;
    D[(int64_t)(k0 + i) * ld + k0 + j] = a[i][j];
  }
}

// Row panel right of the diagonal block: column c of U12 solves L11 x = a by forward
// substitution with the unit diagonal (one thread per column, the 64 unknowns in registers).
__global__ __launch_bounds__(256) void k_trsm_row_panel(int32_t ld, int32_t k0, double *D) {
  __shared__ double lk[kNB][kNB + 1];
  const int tid = threadIdx.x;
  for (int q = tid; q < kNB * kNB; q += 256) {
    const int i = q / kNB, j = q % kNB;
    lk[i][j] = (j < i) ? D[(int64_t)(k0 + i) * ld + k0 + j] : 0.0;
  }
  __syncthreads();
  const int64_t c = (int64_t)k0 + kNB + (int64_t)blockIdx.x * 256 + tid;
  if (c >= ld) return;
  double x[kNB];
#pragma unroll
  for (int j = 0; j < kNB; ++j) x[j] = D[((int64_t)k0 + j) * ld + c];
#pragma unroll
  for (int j = 0; j < kNB; ++j) {
    double t = x[j];
#pragma unroll
    for (int m = 0; m < j; ++m) t -= lk[j][m] * x[m];
    x[j] = t;
  }
#pragma unroll
  for (int j = 0; j < kNB; ++j) D[((int64_t)k0 + j) * ld + c] = x[j];
}

// Column panel below the diagonal block: row i of L21 solves x U11 = a (one thread per row).
__global__ __launch_bounds__(256) void k_trsm_col_panel(int32_t ld, int32_t k0, double *D) {
  __shared__ double uk[kNB][kNB + 1];
  const int tid = threadIdx.x;
  for (int q = tid; q < kNB * kNB; q += 256) {
    const int i = q / kNB, j = q % kNB;
    uk[i][j] = (j >= i) ? D[(int64_t)(k0 + i) * ld + k0 + j] : 0.0;
  }
  __syncthreads();
  const int64_t i = (int64_t)k0 + kNB + (int64_t)blockIdx.x * 256 + tid;
  if (i >= ld) return;
  double *row = D + i * ld + k0;
  double x[kNB];
#pragma unroll
  for (int j = 0; j < kNB; ++j) x[j] = row[j];
#pragma unroll
  for (int j = 0; j < kNB; ++j) {
    double t = x[j];
#pragma unroll
    for (int m = 0; m < j; ++m) t -= x[m] * uk[m][j];
    x[j] = t / uk[j][j];
  }
#pragma unroll
  for (int j = 0; j < kNB; ++j) row[j] = x[j];
}

// Trailing update after step kb: D[ib][jb] -= L[ib][kb] U[kb][jb] for every block pair
// kb < ib, jb < nbk (workgroup t: ib = kb+1 + t/m, jb = kb+1 + t%m, m = nbk-kb-1).
__global__ __launch_bounds__(256) void k_gemm_update(int32_t ld, int32_t kb, int32_t nbk,
                                                     double *D) {
  __shared__ double As[kNB][kNB + 1];
  __shared__ double Bs[kNB][kNB + 1];
  const int32_t m = nbk - kb - 1;
  const int32_t ib = kb + 1 + (int32_t)(blockIdx.x / m), jb = kb + 1 + (int32_t)(blockIdx.x % m);
  const int64_t r0 = (int64_t)ib * kNB, c0 = (int64_t)jb * kNB, k0 = (int64_t)kb * kNB;
  const int tid = threadIdx.x;
  for (int q = tid; q < kNB * kNB; q += 256) {
    const int r = q / kNB, k = q % kNB;
    As[r][k] = D[(r0 + r) * ld + k0 + k];  // L21 block (row r, column k)
    Bs[r][k] = D[(k0 + r) * ld + c0 + k];  // U12 block (row r, column k)
  }
  __syncthreads();
  v4d acc[4];
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) acc[ct] = v4d{0.0, 0.0, 0.0, 0.0};
  mfma_64(As, Bs, acc);
  const int w = tid >> 6, lane = tid & 63;
  const int lr = lane & 15, lk = lane >> 4;
#pragma unroll
  for (int ct = 0; ct < 4; ++ct)
#pragma unroll
    for (int v = 0; v < 4; ++v)
      D[(r0 + 16 * w + 4 * v + lk) * ld + c0 + 16 * ct + lr] -= acc[ct][v];
}

// Lower forms of the two factors: Lb = unit lower part of D, Ut = U^T (lower).
__global__ void k_split_lu(int32_t ld, const double *D, double *Lb, double *Ut) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= (int64_t)ld * ld) return;
  const int64_t i = q / ld, j = q % ld;
  Lb[q] = (j < i) ? D[q] : (j == i ? 1.0 : 0.0);
  Ut[q] = (j <= i) ? D[j * ld + i] : 0.0;
}

// Symmetry of the coarsest operator before a Cholesky solve (which reads only the lower
// triangle): mx[0] = max |a_ij|, mx[1] = max |a_ij - a_ji| as the bit patterns of
// non-negative doubles (ordered like the values); err bit 256 when mx[1] > 1e-10 mx[0].
constexpr int kSymBlocks = 128;
__global__ __launch_bounds__(kBlock) void k_sym_max(int32_t ld, const double *D,
                                                    unsigned long long *mx) {
  __shared__ double sa[kBlock / 64], sd[kBlock / 64];
  double a = 0.0, d = 0.0;  // (a NaN entry never raises them; the factor's pivots catch it)
  for (int64_t q = (int64_t)blockIdx.x * kBlock + threadIdx.x; q < (int64_t)ld * ld;
       q += (int64_t)gridDim.x * kBlock) {
    const int64_t i = q / ld, j = q % ld;
    const double x = fabs(D[q]), y = fabs(D[q] - D[j * ld + i]);
    if (x > a) a = x;
    if (y > d) d = y;
  }
  for (int off = 32; off >= 1; off >>= 1) {
    a = fmax(a, __shfl_xor(a, off, 64));
    d = fmax(d, __shfl_xor(d, off, 64));
  }
  if ((threadIdx.x & 63) == 0) {
    sa[threadIdx.x >> 6] = a;
    sd[threadIdx.x >> 6] = d;
  }
  __syncthreads();
  if (threadIdx.x == 0) {  // one atomic per workgroup (one per entry took 80 us for 576^2)
    for (int w = 1; w < kBlock / 64; ++w) {
      a = fmax(a, sa[w]);
      d = fmax(d, sd[w]);
    }
    if (a > 0.0) atomicMax(&mx[0], (unsigned long long)__double_as_longlong(a));
    if (d > 0.0) atomicMax(&mx[1], (unsigned long long)__double_as_longlong(d));
  }
}
__global__ void k_sym_flag(const unsigned long long *mx, int32_t *err) {
  const double amax = __longlong_as_double((long long)mx[0]);
  const double asym = __longlong_as_double((long long)mx[1]);
  if (!(asym <= 1e-10 * amax)) atomicOr(err, 256);
}

// LU path of coarse_inverse: D (ld x ld, padded) is factored in place; Li (ld x ld) is
// scratch.  Ainv = W^T L^{-1} with W = (U^T)^{-1}.
static void lu_inverse(int32_t ld, int32_t nbk, int32_t n, double *D, double *Li, double *Ainv,
                       int32_t *err, hipStream_t s) {
  for (int32_t kb = 0; kb < nbk; ++kb) {
    const int32_t k0 = kb * kNB;
    k_getrf_diag<<<1, 256, 0, s>>>(ld, k0, D, err);
    const int32_t rest = ld - k0 - kNB;
    if (rest > 0) {
      k_trsm_row_panel<<<(unsigned)ceil_div(rest, 256), 256, 0, s>>>(ld, k0, D);
      k_trsm_col_panel<<<(unsigned)ceil_div(rest, 256), 256, 0, s>>>(ld, k0, D);
      const int64_t m = nbk - kb - 1;
      k_gemm_update<<<(unsigned)(m * m), 256, 0, s>>>(ld, kb, nbk, D);
    }
    SA_LAUNCH_CHECK();
  }
  const int64_t cnt = (int64_t)ld * ld;
  double *Lb = (double *)dev_alloc(sizeof(double) * (size_t)cnt, s);
  double *Ut = (double *)dev_alloc(sizeof(double) * (size_t)cnt, s);
  k_split_lu<<<grid_for(cnt), kBlock, 0, s>>>(ld, D, Lb, Ut);
  SA_LAUNCH_CHECK();
  // Li = Lb^{-1}; then W = Ut^{-1} into D (the factor is no longer needed)
  fill_f64(Li, 0.0, cnt, s);
  k_trtri_diag<<<(unsigned)nbk, 256, 0, s>>>(ld, Lb, Li, true);
  trinv_blocks(ld, nbk, Lb, Li, s);
  fill_f64(D, 0.0, cnt, s);
  k_trtri_diag<<<(unsigned)nbk, 256, 0, s>>>(ld, Ut, D, false);
  trinv_blocks(ld, nbk, Ut, D, s);
  SA_LAUNCH_CHECK();
  gram(n, ld, nbk, D, Li, Ainv, false, s);
  dev_free(Lb, s);
  dev_free(Ut, s);
}

void coarse_inverse(const Csr &A, double *Ainv, int32_t *err, bool lu, hipStream_t s) {
  const int32_t n = A.n;
  if (n <= 0) return;
  const int32_t ld = (int32_t)ceil_div(n, kNB) * kNB;
  const int32_t nbk = ld / kNB;
  const int64_t cnt = (int64_t)ld * ld;
  double *D = (double *)dev_alloc(sizeof(double) * (size_t)cnt, s);
  double *Li = (double *)dev_alloc(sizeof(double) * (size_t)cnt, s);
  fill_f64(D, 0.0, cnt, s);
  fill_f64(Li, 0.0, cnt, s);
  k_dense_scatter<<<grid_for((int64_t)n * 64), kBlock, 0, s>>>(n, ld, A.rp, A.col, A.val, D);
  SA_LAUNCH_CHECK();
  if (ld > n) {
    k_pad_identity<<<grid_for(ld - n), kBlock, 0, s>>>(n, ld, D);
    SA_LAUNCH_CHECK();
  }
  if (lu) {
    lu_inverse(ld, nbk, n, D, Li, Ainv, err, s);
    dev_free(D, s);
    dev_free(Li, s);
    return;
  }
  {
    unsigned long long *mx = (unsigned long long *)dev_alloc(2 * sizeof(unsigned long long), s);
    SA_HIP(hipMemsetAsync(mx, 0, 2 * sizeof(unsigned long long), s));
    k_sym_max<<<kSymBlocks, kBlock, 0, s>>>(ld, D, mx);
    k_sym_flag<<<1, 1, 0, s>>>(mx, err);
    SA_LAUNCH_CHECK();
    dev_free(mx, s);
  }
  chol_inverse(ld, nbk, D, Li, err, s);
  gram(n, ld, nbk, Li, Li, Ainv, true, s);
  dev_free(D, s);
  dev_free(Li, s);
}

}  // namespace sa
