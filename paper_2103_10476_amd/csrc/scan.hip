// Fills and exclusive prefix sums.
#include "common.hpp"

namespace sa {

template <class T>
__global__ void k_fill(T *p, T v, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = v;
}

template <class T>
static void fill(T *p, T v, int64_t n, hipStream_t s) {
  if (n <= 0) return;
  unsigned g = grid_for(n);
  if (g > 65536) g = 65536;
  k_fill<T><<<g, kBlock, 0, s>>>(p, v, n);
  SA_LAUNCH_CHECK();
}

void fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t s) { fill(p, v, n, s); }
void fill_f64(double *p, double v, int64_t n, hipStream_t s) { fill(p, v, n, s); }
void fill_u8(uint8_t *p, uint8_t v, int64_t n, hipStream_t s) { fill(p, v, n, s); }

// ---- exclusive scan -----------------------------------------------------------------
// Per-block totals (each block covers kScanTile elements), then a per-block scan seeded with the
// sum of the totals before it; past kScanSum blocks (8.4M elements) the totals are scanned first.
constexpr int kScanItems = 8;
constexpr int kScanTile = kBlock * kScanItems;

// Exclusive prefix sums of the 256 threads' values: within the wavefronts, then over their four
// totals (sh: 4 words).
template <class T>
__device__ T block_exclusive(T v, T *sh, T &total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  T incl = v;
  if constexpr (sizeof(T) == 4) {
    incl = (T)group_prefix<64>((int32_t)v, lane);
  } else {
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const T o = __shfl_up(incl, off, 64);
      if (lane >= off) incl += o;
    }
  }
  __syncthreads();  // an earlier call's reads come before
  if (lane == 63) sh[wave] = incl;
  __syncthreads();
  T before = 0;
  total = 0;
#pragma unroll
  for (int q = 0; q < kBlock / 64; ++q) {
    if (q < wave) before += sh[q];
    total += sh[q];
  }
  return before + incl - v;
}

template <class T>
__global__ void k_scan_totals(const T *in, int64_t n, T *totals) {
  __shared__ T sh[kBlock / 64];
  int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  T s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k)
    if (base + k < n) s += in[base + k];
  T tot;
  block_exclusive<T>(s, sh, tot);
  if (threadIdx.x == 0) totals[blockIdx.x] = tot;
}

// SUM: offsets are the tiles' totals, of which every block adds up those before its own (up to
// kScanSum of them) in place of a launch that scans them: a launch less in each of the 36 scans
// of a 60^3 mesh's setup, 420 -> 290 us of kernels and the gaps.
constexpr int64_t kScanSum = 4096;
template <class T, bool SUM>
__global__ void k_scan_apply(const T *in, T *out, int64_t n, const T *offsets) {
  __shared__ T sh[kBlock / 64];
  T before = 0;
  if constexpr (SUM) {
    for (int32_t b = threadIdx.x; b < (int32_t)blockIdx.x; b += kBlock) before += offsets[b];
    T all;
    block_exclusive<T>(before, sh, all);
    before = all;
  } else {
    before = offsets[blockIdx.x];
  }
  int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  T vals[kScanItems];
  T s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    vals[k] = (base + k < n) ? in[base + k] : T(0);
    s += vals[k];
  }
  T tot;
  T run = block_exclusive<T>(s, sh, tot) + before;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    if (base + k < n) out[base + k] = run;
    run += vals[k];
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == kBlock - 1) out[n] = run;
}

// n <= kScanTile: the whole scan in one block (out may equal in: every thread reads its items
// before the block scan's barriers, and writes after them).
template <class T>
__global__ void k_scan_single(const T *in, T *out, int64_t n) {
  __shared__ T sh[kBlock / 64];
  const int64_t base = (int64_t)threadIdx.x * kScanItems;
  T vals[kScanItems];
  T s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    vals[k] = (base + k < n) ? in[base + k] : T(0);
    s += vals[k];
  }
  T tot;
  T run = block_exclusive<T>(s, sh, tot);
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    if (base + k < n) out[base + k] = run;
    run += vals[k];
  }
  if (threadIdx.x == 0) out[n] = tot;
}

template <class T>
static void scan_impl(const T *in, T *out, int64_t n, hipStream_t s) {
  if (n <= 0) {
    fill(out, T(0), 1, s);
    return;
  }
  if (n <= kScanTile) {
    k_scan_single<T><<<1, kBlock, 0, s>>>(in, out, n);
    SA_LAUNCH_CHECK();
    return;
  }
  int64_t nb = ceil_div(n, kScanTile);
  T *tot = (T *)dev_alloc(sizeof(T) * (nb + 1), s);
  k_scan_totals<T><<<(unsigned)nb, kBlock, 0, s>>>(in, n, tot);
  SA_LAUNCH_CHECK();
  if (nb <= kScanSum) {
    k_scan_apply<T, true><<<(unsigned)nb, kBlock, 0, s>>>(in, out, n, tot);
  } else {
    scan_impl<T>(tot, tot, nb, s);  // in place: tot has nb+1 slots (nb >= 2 here)
    k_scan_apply<T, false><<<(unsigned)nb, kBlock, 0, s>>>(in, out, n, tot);
  }
  SA_LAUNCH_CHECK();
  dev_free(tot, s);
}

void exclusive_scan_i32(const int32_t *in, int32_t *out, int64_t n, hipStream_t s) {
  scan_impl<int32_t>(in, out, n, s);
}
void exclusive_scan_i64(const int64_t *in, int64_t *out, int64_t n, hipStream_t s) {
  scan_impl<int64_t>(in, out, n, s);
}

}  // namespace sa
