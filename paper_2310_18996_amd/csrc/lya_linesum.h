// Sums over lines of the per-line k-bin sums, in a fixed order (so that they do
// not depend on scheduling), shared by the 1D-power and tuning kernels.  Stage
// 1: R blocks (times the draws) each add the bins of a contiguous range of
// lines, rows [line][bin] read whole, and count the lines per length class (exact
// integers); stage 2 adds the R partial sums in order, and gets each bin's modes
// from the class counts and the table of first modes.  (A block per bin over
// [bin][line] rows took 58 us for 50,000 lines and 32 bins, and each line's 32
// sums went to as many cache lines.)  Below 256 lines R is 1, and the two stages are
// one launch (the 1D power of one line and 1, 22, 64 bins: 17.2, 18.2, 20.0 us with two
// and the table of first modes in both kernels, 15.4, 15.2, 15.1 us with one).
#pragma once

#include "lya_internal.h"
#include "lya_wavefft.h"

namespace lya {

struct LineSumArgs {
  int64_t n;              // lines
  int nk, R;
  const int32_t* npix;
  const double* rows;     // [draw][n][nk]
  const double* fs;       // [draw][n], or null
  double* part;           // [draw][R][nk + 1]: bins, then fs
  long long* hist;        // [R, or draws if R = 1][kLenClasses + 1]: lines per class, then pixels
};

// stage 1: block (r, draw) of 256 threads; the counts by the first draw's blocks,
// or each draw's own where R = 1
__device__ __forceinline__ void line_sum_block(const LineSumArgs& a, int r, int g) {
  __shared__ double ss[256];
  __shared__ int sh[kLenClasses];
  __shared__ unsigned long long spix;
  const int t = threadIdx.x, cols = a.nk <= 32 ? 32 : 64, nrow = 256 / cols, c = t % cols, row = t / cols;
  const int64_t q0 = a.n * r / a.R, q1 = a.n * (r + 1) / a.R;
  if (t < kLenClasses) sh[t] = 0;
  if (t == 0) spix = 0ull;
  double s = 0.0;
  if (c < a.nk) {
    const double* p = a.rows + static_cast<size_t>(g) * a.n * a.nk + c;
#pragma unroll 8
    for (int64_t q = q0 + row; q < q1; q += nrow) s += p[q * a.nk];
  }
  ss[t] = s;
  __syncthreads();
  double* out = a.part + (static_cast<size_t>(g) * a.R + r) * (a.nk + 1);
  if (t < a.nk) {
    for (int k = 1; k < nrow; ++k) s += ss[k * cols + t];
    out[t] = s;
  }
  if (a.fs) {
    __syncthreads();
    double f = 0.0;
    for (int64_t q = q0 + t; q < q1; q += 256) f += a.fs[static_cast<size_t>(g) * a.n + q];
    ss[t] = f;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
      if (t < w) ss[t] += ss[t + w];
      __syncthreads();
    }
    if (t == 0) out[a.nk] = ss[0];
  }
  if (g == 0 || a.R == 1) {
    unsigned long long pix = 0ull;
    for (int64_t q = q0 + t; q < q1; q += 256) {
      const int np = a.npix[q];
      atomicAdd(&sh[len_class(np)], 1);
      pix += static_cast<unsigned long long>(static_cast<long long>(np));
    }
    atomicAdd(&spix, pix);
    __syncthreads();
    long long* h = a.hist + static_cast<size_t>(r + g) * (kLenClasses + 1);   // (one of them is 0)
    if (t < kLenClasses) h[t] = sh[t];
    if (t == 0) h[kLenClasses] = static_cast<long long>(spix);
  }
}

// Sum of x(0) .. x(R - 1) in order, the loads of 32 of them in flight at once.
template <typename T, typename X>
__device__ __forceinline__ T sum_parts(int R, X x) {
  T s = 0;
  for (int r0 = 0; r0 < R; r0 += 32) {
    T v[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) v[i] = x(r0 + i < R ? r0 + i : R - 1);
#pragma unroll
    for (int i = 0; i < 32; ++i) s += r0 + i < R ? v[i] : T(0);
  }
  return s;
}
// stage 2 (a block of at least 64 threads): class counts and pixels into cls
// [kLenClasses + 1] (shared), valid after the caller's barrier
__device__ __forceinline__ void line_counts(const LineSumArgs& a, int g, long long* cls) {
  const int t = threadIdx.x;
  const long long* h = a.hist + (a.R == 1 ? static_cast<size_t>(g) * (kLenClasses + 1) : 0);
  if (t <= kLenClasses)
    cls[t] = sum_parts<long long>(a.R, [&](int r) { return h[static_cast<size_t>(r) * (kLenClasses + 1) + t]; });
}
__device__ __forceinline__ double line_total(const LineSumArgs& a, int g, int b) {
  const double* p = a.part + static_cast<size_t>(g) * a.R * (a.nk + 1) + b;
  return sum_parts<double>(a.R, [&](int r) { return p[static_cast<size_t>(r) * (a.nk + 1)]; });
}

// blocks of stage 1, and the bytes of part and hist for G draws
inline int line_sum_blocks(int64_t n) { return n < 256 ? 1 : n >= 128 * 128 ? 128 : static_cast<int>(n / 128); }
inline size_t line_sum_bytes(int64_t n, int nk, int G) {
  const size_t R = line_sum_blocks(n), counts = R == 1 ? G : R;
  return sizeof(double) * (R * G * (nk + 1) + counts * (kLenClasses + 1));
}

}  // namespace lya
