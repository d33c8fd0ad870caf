// Lines of sight, small-scale field and FGPA (gfx950).
//
// For every quasar line of sight (section "Gaussian fields along lines of
// sight" and eq:gfield, eq:FGPA):
//   * pixel j sits at the int64 fixed-point position origin + j*step (cell
//     units x 2^32); delta_L and eta_par come from periodic trilinear
//     interpolation of the packed {delta, eta} box;
//   * delta_S: Philox normals (stream 1, counter (q<<33)+m) on modes
//     m = 0..N_S/2 of a length N_S = next_pow2(n_q) line, scaled by
//     sqrt(P_s(k_m)/(N_S dpix)), P_s = amp exp(-(k/kcut)^2), then the real
//     inverse DFT, computed as one complex inverse FFT of length N_S/2 whose
//     output holds the even pixels in its real part and the odd pixels in
//     its imaginary part;
//   * wide-angle variant: eta_par = u_p u_q eta^pq at each corner voxel from
//     four packed boxes ({delta, eta_zz}, {eta_xx, eta_yy}, {eta_xy, eta_xz},
//     {eta_yz, 0}), u the skewer's direction, then interpolated like delta;
//   * Gaussian-kernel variant: the paper's average over the 7^3 voxels around
//     the pixel (standard deviation one voxel) in place of trilinear;
//   * g = delta_L + delta_S + c(z) eta_par, F = exp(-a(z) exp(b(z) g)), with
//     a, b, c quadratics in (1+z) and z the unperturbed redshift of
//     chi_j = chi0 - j*dchi (section "FGPA");
//   * per redshift bin, the sum of F and the pixel count, accumulated as
//     exact 64-bit integers of round(F 2^32), so the result does not depend on
//     the order in which work is scheduled.
// One persistent launch; each wavefront pulls chunks of skewers from an
// atomic queue and owns a skewer at a time (its small-scale FFT lives in the
// wave's slice of LDS, so no block-wide barrier is needed per skewer).
#include <algorithm>
#include <type_traits>

#include "lya_internal.h"
#include "lya_pull.h"
#include "lya_wavefft.h"

namespace lya {

constexpr int kSkWaves = 4;
constexpr int kSkNT = 64 * kSkWaves;

__global__ void __launch_bounds__(256) k_skewer_finalize(int n_bins, const unsigned long long* bsum,
                                                         const unsigned long long* bcnt, double* fsum,
                                                         int64_t* cnt) {
  const int t = threadIdx.x;
  if (t < n_bins) {
    unsigned long long s = 0ull, c = 0ull;
#pragma unroll
    for (int i = 0; i < kBinCopies; ++i) {
      s += bsum[i * kMaxZBins + t];
      c += bcnt[i * kMaxZBins + t];
    }
    if (fsum) fsum[t] = static_cast<double>(s) * 2.3283064365386963e-10;  // 2^-32
    if (cnt) cnt[t] = static_cast<int64_t>(c);
  }
}

// Box element loads, the storage type fixed at compile time (a run-time test
// per corner splits the gathers into separate blocks that each wait for their
// load, instead of issuing all of a pixel's gathers together).
template <bool B16>
__device__ __forceinline__ float2 ld_field(const SkewerArgs& a, size_t i) {
  if constexpr (B16) return unpack_bf16x2(a.field_bf16[i]);
  else return a.field[i];
}

// Interpolation modes of the skewer kernel.
enum { kSkTri = 0, kSkWide = 1, kSkGauss = 2 };

// Gaussian-kernel average over the 7^3 voxels around the pixel's nearest grid
// point c (standard deviation one voxel, section "Gaussian fields along lines
// of sight"): the weights separate into 7 per axis, exp(-(o - t)^2/2) with
// t = u - c in [-1/2, 1/2), and the average divides by their product sum.
// The general form, a pixel per lane, for lines with steps of a third of a cell or
// more (gauss_geo), whose neighbouring pixels share little; x and y weights where
// they are needed.  row(i, jy): where the z run of plane i and y row jy starts;
// cell(r, k): its k-th voxel.
template <class ROW, class CELL>
__device__ __forceinline__ void gauss7_sum(const float (&t)[3], ROW row, CELL cell, float& d, float& e) {
  auto weight = [](int o, float tt) {
    const float dd = static_cast<float>(o - 3) - tt;
    return __expf(-0.5f * dd * dd);
  };
  float gz[7], sz = 0.0f, sx = 0.0f, sy = 0.0f;
#pragma unroll
  for (int o = 0; o < 7; ++o) {
    gz[o] = weight(o, t[2]);
    sz += gz[o];
  }
  float ax_ = 0.0f, ay_ = 0.0f;
#pragma unroll 1
  for (int i = 0; i < 7; ++i) {
    float bx = 0.0f, by = 0.0f;
    sy = 0.0f;
#pragma unroll
    for (int jy = 0; jy < 7; ++jy) {
      const auto r = row(i, jy);
      float rx_ = 0.0f, ry_ = 0.0f;
#pragma unroll
      for (int k = 0; k < 7; ++k) {
        const float2 f = cell(r, k);
        rx_ += gz[k] * f.x;
        ry_ += gz[k] * f.y;
      }
      const float w = weight(jy, t[1]);
      sy += w;
      bx += w * rx_;
      by += w * ry_;
    }
    const float w = weight(i, t[0]);
    sx += w;
    ax_ += w * bx;
    ay_ += w * by;
  }
  const float inv = 1.0f / (sx * sy * sz);
  d = ax_ * inv;
  e = ay_ * inv;
}
// the pixel's nearest grid point and its offset from it
__device__ __forceinline__ void gauss_centre(const int64_t (&p)[3], int (&c)[3], float (&t)[3]) {
#pragma unroll
  for (int ax = 0; ax < 3; ++ax) {
    const uint32_t fr = static_cast<uint32_t>(p[ax]);
    const int up = static_cast<int>(fr >> 31);
    c[ax] = static_cast<int>((p[ax] >> 32) + up);
    t[ax] = static_cast<float>(fr) * 2.3283064365386963e-10f - static_cast<float>(up);
  }
}
// straight from the box
template <bool B16>
__device__ __forceinline__ void gauss7_at(const SkewerArgs& a, const int64_t (&p)[3], int N, size_t NN, float& d,
                                          float& e) {
  int c[3];
  float t[3];
  gauss_centre(p, c, t);
  gauss7_sum(
      t,
      [&](int i, int jy) {
        return static_cast<size_t>((c[0] + i - 3) & (N - 1)) * NN + static_cast<size_t>((c[1] + jy - 3) & (N - 1)) * N;
      },
      [&](size_t r, int k) { return ld_field<B16>(a, r + ((c[2] + k - 3) & (N - 1))); }, d, e);
}

// The Gaussian-kernel average of 64 consecutive pixels on the matrix cores.
// The lanes of a quad hold four neighbouring pixels (steps below a third of a
// cell per axis, so their nearest grid points differ by at most one), which
// share a window of 8 cells in y and z: each pixel's 7 weights go into 8 slots,
// the unused one 0.  For a plane x, one MFMA 4x4x1 (16 blocks: one per quad)
// adds, for one z slot, the products of the quad's four z weights with four
// columns: the two components of two neighbouring y rows; eight of them give
// the z sums of all four pixels over two rows, which the y and x weights then
// add up.  A voxel is so read from LDS once per quad and not once per pixel, as
// single words, and the z sums' 686 multiply-adds per pixel (one fused
// multiply-add each: K = 1) run at twice the rate of the vector unit.
// The wave's cells lie in LDS as z runs of 16 (or 32) words, the components
// apart: at half a run's shift of eight banks, the four columns of all quads
// read different banks.  Almost always they are 8 planes of 8-12 rows at most,
// and their loads go to registers while the previous 64 pixels are summed (at
// two waves per SIMD nothing else hides them), with a plane's address in
// scalar registers.
// 35M pixels of 50,000 lines in a 512^3 box: 3.11 ms when each pixel read its
// 343 voxels from LDS, 1.78 ms now (the same from a 64^3
// box: bound by vector issue and the latencies two waves per SIMD leave open.
// Reading a plane ahead took 2.26 against 2.07 ms under the profiler: spills).
constexpr int kGaussRows = 84;                            // z runs of 16 in a wave's slice (42 of 32)
constexpr int kGaussEta = 16 * kGaussRows + 8;            // start of the second component
constexpr int kGaussWords = kGaussEta + 16 * kGaussRows;
constexpr int kGaussPre = 24;                             // 8 planes x 3 groups of 4 rows
struct GaussGeo {
  int m1, m2;        // the quad's window start in y and z, relative to the wave's first cell
  int sh1, sh2;      // the pixel's shift within it, 0 or 1
  int c0;            // the pixel's nearest plane x, relative to the wave's first
  float t[3];        // offset from the pixel's nearest grid point, [-1/2, 1/2)
  int lo[3];         // the wave's first cell, to be taken modulo N (uniform, as the rest)
  int nx, ny, zs;    // planes and y rows of the wave; z runs of 2^zs cells
  bool fast;         // the cells fit the registers and the slice together
};

template <int CTRL>
__device__ __forceinline__ int dpp_i32(int v) {
  return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
  return __int_as_float(dpp_i32<CTRL>(__float_as_int(v)));
}

// Pixels j1 .. j1 + 63 of a line of np (those past the end repeat the last
// one); st: steps below a third of a cell.
__device__ __forceinline__ GaussGeo gauss_geo(const int64_t (&o)[3], const int32_t (&st)[3], int j1, int np, int lane) {
  GaussGeo g;
  const int last = min(63, np - 1 - j1), dj = min(lane, last);
  int c[3], span[3];
#pragma unroll
  for (int ax = 0; ax < 3; ++ax) {
    // nearest grid points (floor(u + 1/2)) of the first and the last pixel:
    // along a straight line the others lie between them
    constexpr int64_t kHalf = int64_t(1) << 31;
    const int64_t pf = o[ax] + static_cast<int64_t>(j1) * st[ax] + kHalf, pl = pf + static_cast<int64_t>(last) * st[ax];
    const int64_t cf = pf >> 32, cl = pl >> 32;
    const int64_t lo = cf < cl ? cf : cl;
    span[ax] = static_cast<int>(cf < cl ? cl - cf : cf - cl);   // <= 21
    g.lo[ax] = static_cast<int>(lo - 3);
    const int64_t p = (pf - (lo << 32)) + static_cast<int64_t>(dj) * st[ax];
    c[ax] = static_cast<int>(p >> 32);
    // p's fraction is that of u + 1/2: t = u - c = fraction - 1/2
    const uint32_t fr = static_cast<uint32_t>(p) ^ 0x80000000u;
    g.t[ax] = static_cast<float>(fr) * 2.3283064365386963e-10f - static_cast<float>(fr >> 31);
  }
  auto quad_min = [](int v) {
    v = min(v, dpp_i32<0xB1>(v));    // quad_perm [1, 0, 3, 2]
    return min(v, dpp_i32<0x4E>(v));  // quad_perm [2, 3, 0, 1]
  };
  g.c0 = c[0] + 3;
  g.m1 = quad_min(c[1]);
  g.sh1 = c[1] - g.m1;
  g.m2 = quad_min(c[2]);
  g.sh2 = c[2] - g.m2;
  g.nx = span[0] + 7;
  g.ny = span[1] + 8;
  g.zs = span[2] + 8 <= 16 ? 4 : 5;
  g.fast = g.zs == 4 && g.nx <= 8 && g.ny <= 12 && g.nx * g.ny <= kGaussRows;
  return g;
}

template <bool B16>
struct GaussCell {
  typedef float2 type;
};
template <>
struct GaussCell<true> {
  typedef uint32_t type;
};
__device__ __forceinline__ float2 gauss_cell(float2 v) { return v; }
__device__ __forceinline__ float2 gauss_cell(uint32_t v) { return unpack_bf16x2(v); }

// All cells of a fast geometry into registers: row group r (4 rows x 16 z, a
// lane each) of plane p in pre[3 p + r].  Every address is in the box (the cell
// indices are taken modulo N), also those of rows past the last.
template <bool B16, int P0, int P1, int RG>
__device__ __forceinline__ void gauss_load_planes(const typename GaussCell<B16>::type* fb, const GaussGeo& g,
                                                  uint32_t msk, size_t NN, const uint32_t (&off)[3],
                                                  typename GaussCell<B16>::type (&pre)[kGaussPre]) {
#pragma unroll
  for (int p = P0; p < P1; ++p) {
    const auto* plane = fb + static_cast<size_t>(static_cast<uint32_t>(g.lo[0] + p) & msk) * NN;
#pragma unroll
    for (int r = 0; r < RG; ++r) pre[3 * p + r] = plane[off[r]];
  }
}
template <bool B16>
__device__ __forceinline__ void gauss_load(const typename GaussCell<B16>::type* fb, const GaussGeo& g, int N, size_t NN,
                                           int lane, typename GaussCell<B16>::type (&pre)[kGaussPre]) {
  const uint32_t msk = static_cast<uint32_t>(N - 1);
  const uint32_t z = static_cast<uint32_t>(g.lo[2] + (lane & 15)) & msk;
  uint32_t off[3];
#pragma unroll
  for (int r = 0; r < 3; ++r)
    off[r] = (static_cast<uint32_t>(g.lo[1] + (lane >> 4) + 4 * r) & msk) * static_cast<uint32_t>(N) + z;
  if (g.ny <= 8) {
    gauss_load_planes<B16, 0, 7, 2>(fb, g, msk, NN, off, pre);
    if (g.nx > 7) gauss_load_planes<B16, 7, 8, 2>(fb, g, msk, NN, off, pre);
  } else {
    gauss_load_planes<B16, 0, 7, 3>(fb, g, msk, NN, off, pre);
    if (g.nx > 7) gauss_load_planes<B16, 7, 8, 3>(fb, g, msk, NN, off, pre);
  }
}

// and on into the slice
template <typename C>
__device__ __forceinline__ void gauss_store(const GaussGeo& g, const C (&pre)[kGaussPre], float* lds, int lane) {
  const bool third = (lane >> 4) + 8 < g.ny;
  float* at = lds + lane;
#pragma unroll
  for (int p = 0; p < 8; ++p) {
    if (p == 7 && g.nx <= 7) break;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const float2 v = gauss_cell(pre[3 * p + r]);
      at[64 * r] = v.x;
      at[kGaussEta + 64 * r] = v.y;
    }
    if (g.ny > 8) {
      const float2 v = gauss_cell(pre[3 * p + 2]);
      if (third) {
        at[128] = v.x;
        at[kGaussEta + 128] = v.y;
      }
    }
    at += 16 * g.ny;
  }
}

// Planes x0 .. x0 + planes - 1 of any geometry straight into the slice.
template <bool B16>
__device__ __forceinline__ void gauss_stage(const typename GaussCell<B16>::type* fb, const GaussGeo& g, int x0,
                                            int planes, int N, size_t NN, int lane, float* lds) {
  const uint32_t msk = static_cast<uint32_t>(N - 1);
  const uint32_t z = static_cast<uint32_t>(g.lo[2] + (lane & ((1 << g.zs) - 1))) & msk;
  const int dy = 64 >> g.zs, cells = (planes * g.ny) << g.zs;
  int x = g.lo[0] + x0, y = lane >> g.zs;   // dy <= 4 < ny
#pragma unroll 4
  for (int i = lane; i < cells; i += 64) {
    const float2 v = gauss_cell(fb[static_cast<size_t>(static_cast<uint32_t>(x) & msk) * NN +
                                   (static_cast<uint32_t>(g.lo[1] + y) & msk) * static_cast<uint32_t>(N) + z]);
    lds[i] = v.x;
    lds[kGaussEta + i] = v.y;
    y += dy;
    const bool wrap = y >= g.ny;
    y -= wrap ? g.ny : 0;
    x += wrap ? 1 : 0;
  }
}

// The cells around pixels j1 .. j1 + last of a line without shared windows, where
// all of them fit the wave's slice at once (steps of a third of a cell and more: up to
// some 30 pixels, so short lines and the ends of others): loaded once, then read by
// every pixel.  50,000 lines of 8-64 pixels at 0.35 cells per pixel: 1.97 ms straight
// from the box, 0.96 ms so.
struct GaussBox {
  int lo[3], ny, nz, cells;   // first cell (to be taken modulo N), y rows, z cells, cells in all; 0: they do not fit
};
__device__ __forceinline__ GaussBox gauss_box(const int64_t (&o)[3], const int64_t (&st)[3], int j1, int last) {
  constexpr int kCap = kGaussWords / 2;
  constexpr int64_t kHalf = int64_t(1) << 31, kFar = int64_t(1) << 62, kStep = int64_t(1) << 37;
  GaussBox g;
  int n[3];
  bool fits = true;
#pragma unroll
  for (int ax = 0; ax < 3; ++ax) {
    // as in gauss_geo; below 2^5 cells a step from within +-2^30 cells nothing wraps
    const int64_t pf = o[ax] + static_cast<int64_t>(j1) * st[ax] + kHalf;
    fits = fits && st[ax] < kStep && st[ax] > -kStep && pf >= -kFar && pf < kFar;
    const int64_t cf = pf >> 32, cl = (pf + static_cast<int64_t>(last) * st[ax]) >> 32;
    const int64_t lo = cf < cl ? cf : cl, span = cf < cl ? cl - cf : cf - cl;
    fits = fits && span < kCap;
    g.lo[ax] = static_cast<int>(lo - 3);
    n[ax] = static_cast<int>(span < kCap ? span : 0) + 7;
  }
  g.ny = n[1];
  g.nz = n[2];
  fits = fits && n[1] * n[2] <= kCap;   // (each below 2^11)
  g.cells = fits && n[0] * (n[1] * n[2]) <= kCap ? n[0] * (n[1] * n[2]) : 0;
  return g;
}
template <bool B16>
__device__ __forceinline__ void gauss7_staged(const typename GaussCell<B16>::type* fb, const GaussBox& g,
                                              const int64_t (&p)[3], int N, size_t NN, int lane, float2* lds, float& d,
                                              float& e) {
  const uint32_t msk = static_cast<uint32_t>(N - 1);
  const int plane = g.ny * g.nz;
  for (int v = lane; v < g.cells; v += 64) {
    const int x = v / plane, r = v - x * plane, y = r / g.nz, z = r - y * g.nz;
    lds[v] = gauss_cell(fb[static_cast<size_t>(static_cast<uint32_t>(g.lo[0] + x) & msk) * NN +
                           (static_cast<uint32_t>(g.lo[1] + y) & msk) * static_cast<uint32_t>(N) +
                           (static_cast<uint32_t>(g.lo[2] + z) & msk)]);
  }
  wave_sync();
  int c[3];
  float t[3];
  gauss_centre(p, c, t);
  const float2* at = lds + ((c[0] - 3 - g.lo[0]) * plane + (c[1] - 3 - g.lo[1]) * g.nz + (c[2] - 3 - g.lo[2]));
  gauss7_sum(
      t, [&](int i, int jy) { return at + i * plane + jy * g.nz; }, [](const float2* r, int k) { return r[k]; }, d, e);
  wave_sync();   // the slice is loaded again
}

typedef float v4f __attribute__((ext_vector_type(4)));

// Adds planes x0 .. x0 + planes - 1 to the quad's sums acc[pixel] (this lane's
// column: component lane & 1 of every second row) and the x weights to sx.
__device__ __forceinline__ void gauss_planes_add(const GaussGeo& g, int x0, int planes, const float (&wz)[8],
                                                 const float (&wy)[4][4], const float* lds, int lane, float (&acc)[4],
                                                 float& sx) {
  const float* row = lds + ((lane & 1) ? kGaussEta : 0) + ((g.m1 + ((lane >> 1) & 1)) << g.zs) + g.m2;
  const int two_rows = 2 << g.zs, plane = g.ny << g.zs;
#pragma unroll 1
  for (int x = x0; x < x0 + planes; ++x, row += plane) {
    const int o = x - g.c0;
    const float dd = static_cast<float>(o) - g.t[0];
    const float w = o >= -3 && o <= 3 ? __expf(-0.5f * dd * dd) : 0.0f;
    sx += w;
    const float wx[4] = {dpp_f32<0x00>(w), dpp_f32<0x55>(w), dpp_f32<0xAA>(w), dpp_f32<0xFF>(w)};
    float f[4][8];
#pragma unroll
    for (int jj = 0; jj < 4; ++jj)
#pragma unroll
      for (int k = 0; k < 8; ++k) f[jj][k] = row[jj * two_rows + k];
    v4f D[4];
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) D[jj] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int k = 0; k < 8; ++k)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) D[jj] = __builtin_amdgcn_mfma_f32_4x4x1f32(wz[k], f[jj][k], D[jj], 0, 0, 0);
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const float ty = fmaf(wy[3][p], D[3][p], fmaf(wy[2][p], D[2][p], fmaf(wy[1][p], D[1][p], wy[0][p] * D[0][p])));
      acc[p] = fmaf(wx[p], ty, acc[p]);
    }
  }
}

// The pixel's weights of one axis in its quad's window slots; returns their sum.
__device__ __forceinline__ float gauss_slots(float t, int sh, float (&w)[8]) {
  float g[7], s = 0.0f;
#pragma unroll
  for (int o = 0; o < 7; ++o) {
    const float dd = static_cast<float>(o - 3) - t;
    g[o] = __expf(-0.5f * dd * dd);
    s += g[o];
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) w[k] = sh ? (k > 0 ? g[k - 1] : 0.0f) : (k < 7 ? g[k] : 0.0f);
  return s;
}

// eta_par of a voxel from its four boxes; explicit fused multiply-adds, so that
// every path rounds alike.
struct WideWeights {
  float xx, yy, zz, xy, xz, yz;
  __device__ __forceinline__ float eta(float2 a0, float2 a1, float2 a2, float2 a3) const {
    float e = __builtin_fmaf(zz, a0.y, xx * a1.x);
    e = __builtin_fmaf(yy, a1.y, e);
    e = __builtin_fmaf(xy, a2.x, e);
    e = __builtin_fmaf(xz, a2.y, e);
    return __builtin_fmaf(yz, a3.x, e);
  }
};

// c: values at the pixel's z in the columns (x0, y0), (x0, y1), (x1, y0), (x1, y1)
__device__ __forceinline__ float bilerp(float tx, float ty, const float (&c)[4]) {
  const float c0 = c[0] + ty * (c[1] - c[0]);
  const float c1 = c[2] + ty * (c[3] - c[2]);
  return c0 + tx * (c1 - c0);
}
__device__ __forceinline__ float trilerp(float tx, float ty, float tz, float c000, float c001, float c010, float c011,
                                         float c100, float c101, float c110, float c111) {
  const float c[4] = {c000 + tz * (c001 - c000), c010 + tz * (c011 - c010), c100 + tz * (c101 - c100),
                      c110 + tz * (c111 - c110)};
  return bilerp(tx, ty, c);
}

// Sum over the wave, in lane 63: an inclusive scan by DPP moves (a shuffle per
// step would be an LDS round trip).
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned long long dpp_add_u64(unsigned long long v) {
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, ROWS, 0xf, true);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(v >> 32), CTRL, ROWS, 0xf, true);
  return v + ((static_cast<unsigned long long>(hi) << 32) | lo);
}
__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v) {
  v = dpp_add_u64<0x111, 0xf>(v);   // row_shr 1, 2, 4, 8
  v = dpp_add_u64<0x112, 0xf>(v);
  v = dpp_add_u64<0x114, 0xf>(v);
  v = dpp_add_u64<0x118, 0xf>(v);
  v = dpp_add_u64<0x142, 0xa>(v);   // row_bcast 15 into rows 1 and 3
  return dpp_add_u64<0x143, 0xc>(v);   // row_bcast 31 into rows 2 and 3
}

// Bin sums along one line for the cell walk.  The bin is the wave's, not a lane's:
// nearly every 64 consecutive pixels lie in one bin as a whole (two scalar
// comparisons), and where one ends its lanes are added first and leave by one LDS
// addition.  With a bin per lane every pixel reads its bounds from LDS and 64 lanes
// add to one address, twice per bin (LDS conflicts 570M -> 140M cycles on the 2048^3
// lines); the other modes keep that, it needs fewer scalar registers (7^3 mode
// 1.80 against 1.83 ms).  Pixel counts follow from the bounds.
struct BinWalk {
  int bin, lo, hi;           // uniform; bin < 0: past the last
  unsigned long long acc;    // this lane's pixels of the bin, F 2^32
  __device__ __forceinline__ void bounds(const int* jb) {
    lo = bin < 0 ? 0x7fffffff : __builtin_amdgcn_readfirstlane(jb[bin + 1]);
    hi = bin < 0 ? 0x7fffffff : __builtin_amdgcn_readfirstlane(jb[bin]);
  }
  __device__ __forceinline__ void start(const int* jb, int n_bins) {
    bin = n_bins - 1;
    acc = 0ull;
    bounds(jb);
  }
  __device__ __forceinline__ void flush(unsigned long long* s_sum, int lane) {
    const unsigned long long t = wave_sum_u64(acc);
    if (lane == 63 && t) atomicAdd(&s_sum[bin], t);   // t = 0 past the last bin
    acc = 0ull;
  }
  // pixels j0 .. j0 + 63 of np, j this lane's
  __device__ __forceinline__ void add(const int* jb, int j0, int np, int j, float F, unsigned long long* s_sum,
                                      int lane) {
    const int end = j0 + 64 < np ? j0 + 64 : np;
    const unsigned long long f = __float2ull_rn(F * 4294967296.0f);
    if (j0 >= lo && j0 + 64 <= hi) {   // hi <= np
      acc += f;
      return;
    }
    while (bin >= 0) {
      if (j >= lo && j < hi) acc += f;
      if (hi >= end) break;
      flush(s_sum, lane);
      --bin;
      bounds(jb);
    }
  }
  __device__ __forceinline__ void end(const int* jb, int n_bins, unsigned long long* s_sum,
                                      unsigned long long* s_cnt, int lane) {
    flush(s_sum, lane);
    for (int b = lane; b < n_bins; b += 64)
      if (jb[b] > jb[b + 1]) atomicAdd(&s_cnt[b], static_cast<unsigned long long>(jb[b] - jb[b + 1]));
  }
};

// Trilinear interpolation through the wave's cells.  64 consecutive pixels of a
// line (steps of a tenth of a cell, say) lie in some 10 cells, so the eight corner
// gathers of each pixel read the same few voxels over and over.  Instead a lane
// takes one (x, y) corner column of one cell: it loads both its voxels (two
// gathers in place of eight, in flight during the 64 pixels before), and leaves
// {delta, its z difference, eta, its z difference} in LDS, from where a pixel
// reads its cell's four columns.  The arithmetic is the same to the bit.
// Cells are numbered by the boundaries crossed since the wave's first pixel, all
// axes together; a number that no pixel has stays unused.  Lines with steps that
// may cross more than 15 boundaries in 64 pixels (steps above about a fifth of a cell
// summed over the axes: 0.206 along one, 0.079 along each of three) gather pixel by
// pixel.
// What bounded the gathers: the address unit (20 cycles each, 70% busy) and that
// every step waited for the stores of the step before (loads and stores complete
// in order).  1.1e9 pixels of 1M lines in a 2048^3 box without delta_S and FGPA
// 6.7 -> 5.6 ms, with both and bins 11.9 -> 10.6 ms (0.77 vector
// instructions per CU cycle); 35M wide-angle pixels in 512^3 (four BF16 boxes) 592 -> 481
// us (vector unit 72% busy), (FP32) 788 -> 643 us.  The columns alone, without the order of loads and stores, took 13.1 ms.
constexpr int kCells = 16;
__device__ __forceinline__ bool cells_fit(int64_t sx, int64_t sy, int64_t sz) {
  // 63 steps cross at most floor(63 |s|) + 1 boundaries of an axis
  const uint64_t a = static_cast<uint64_t>(sx < 0 ? -sx : sx), b = static_cast<uint64_t>(sy < 0 ? -sy : sy),
                 c = static_cast<uint64_t>(sz < 0 ? -sz : sz);
  return a < (1u << 30) && b < (1u << 30) && c < (1u << 30) &&
         ((63 * a) >> 32) + ((63 * b) >> 32) + ((63 * c) >> 32) + 3 < kCells;
}
// A line from here whose steps reach less than 2^62 in all (2^28 pixels of a quarter
// of a cell, 2^31 of a third) stays within 64 bits.  Positions that wrap, at +-2^31
// cells, are right modulo the box, but their cells are no longer in the order that
// the cell walk and the 7^3 windows count them in.
__device__ __forceinline__ bool no_wrap(int64_t ox, int64_t oy, int64_t oz) {
  // (from -2^62 up to 2^62 the two highest bits are alike)
  const auto top = [](int64_t v) {
    const uint32_t h = static_cast<uint32_t>(static_cast<uint64_t>(v) >> 32);
    return h ^ (h << 1);
  };
  return static_cast<int32_t>(top(ox) | top(oy) | top(oz)) >= 0;
}
__device__ __forceinline__ uint32_t abs_diff(uint32_t a, uint32_t uniform) {
  uint32_t r;
  asm("v_sad_u32 %0, %1, %2, 0" : "=v"(r) : "v"(a), "s"(uniform));
  return r;
}

template <int MODE, bool B16>
struct CellWalk {
  static constexpr int F = MODE == kSkWide ? 4 : 1;   // boxes
  typedef typename GaussCell<B16>::type V;
  uint64_t p[3];       // this lane's pixel of the step on its way, biased by 2^63 (cell order without signs)
  uint32_t fr[3], k;   // its fractions and cell number
  V v[F][2];           // the lane's column

  __device__ __forceinline__ void start(int64_t ox, int64_t oy, int64_t oz, int64_t sx, int64_t sy, int64_t sz,
                                        int lane) {
    constexpr uint64_t kBias = uint64_t(1) << 63;
    p[0] = kBias + static_cast<uint64_t>(ox) + static_cast<uint64_t>(sx) * static_cast<uint32_t>(lane);
    p[1] = kBias + static_cast<uint64_t>(oy) + static_cast<uint64_t>(sy) * static_cast<uint32_t>(lane);
    p[2] = kBias + static_cast<uint64_t>(oz) + static_cast<uint64_t>(sz) * static_cast<uint32_t>(lane);
  }

  // The cells of the 64 pixels at p: their columns are sent for, p goes on.  All lanes.
  __device__ __forceinline__ void send(const SkewerArgs& a, int64_t sx, int64_t sy, int64_t sz, int N, size_t NN,
                                       int lane) {
    const int64_t s[3] = {sx, sy, sz};
    uint32_t first[3], r[3];
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
      const uint32_t cell = static_cast<uint32_t>(p[ax] >> 32);
      first[ax] = __builtin_amdgcn_readfirstlane(cell);
      r[ax] = abs_diff(cell, first[ax]);
      fr[ax] = static_cast<uint32_t>(p[ax]);
      p[ax] += static_cast<uint64_t>(s[ax]) * 64u;
    }
    k = r[0] + r[1] + r[2];   // < kCells
    // the cell to its number's quad of lanes (any of its pixels: the last one stays)
    const uint32_t pack = r[0] | r[1] << 8 | r[2] << 16;
    const uint32_t c = dpp_i32<0x00>(__builtin_amdgcn_ds_permute(static_cast<int>(k << 4), static_cast<int>(pack)));
    const int dir[3] = {sx < 0 ? -1 : 1, sy < 0 ? -1 : 1, sz < 0 ? -1 : 1};
    const uint32_t msk = static_cast<uint32_t>(N - 1);
    const uint32_t x = (first[0] + dir[0] * static_cast<int>(c & 255u) + ((lane >> 1) & 1)) & msk;
    const uint32_t y = (first[1] + dir[1] * static_cast<int>(c >> 8 & 255u) + (lane & 1)) & msk;
    const uint32_t z = (first[2] + dir[2] * static_cast<int>(c >> 16 & 255u)) & msk;
    const uint32_t row = y * static_cast<uint32_t>(N);
    const uint64_t plane = static_cast<uint64_t>(x) * static_cast<uint32_t>(NN);   // n^2 + padding < 2^32
    const uint64_t i0 = plane + (row + z), i1 = plane + (row + ((z + 1) & msk));
#pragma unroll
    for (int f = 0; f < F; ++f) {
      const V* b;
      if constexpr (B16) b = f == 0 ? a.field_bf16 : a.wide_bf16[f - 1];
      else b = f == 0 ? a.field : a.wide[f - 1];
      v[f][0] = b[i0];
      v[f][1] = b[i1];
    }
  }
};

// A line's pixels of one output as a bounded buffer: lanes past the end, and all
// of an output that is not wanted, are dropped by the bounds check, so that a
// step's stores need no branch.  Loads and stores complete in order here, and
// where a branch may skip a store the wait for a later load is a wait for
// everything before it.
struct LineOut {
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ LineOut(float* p, int64_t off, int np)
      : r(__builtin_amdgcn_make_buffer_rsrc(p ? p + off : p, 0, p ? 4 * np : 0, 0x00020000)) {}
  __device__ __forceinline__ void put(int j, float v) const {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, 4 * j, 0, 0);
  }
};

// Position of a line's pixels in the z(chi) table, in table steps times 2^32:
// chi_j / kZTabH = chi0 / kZTabH - j dchi / kZTabH, each term rounded to 2^-32
// steps (at most 2^-22 Mpc/h off at j = 2048).
__device__ __forceinline__ int64_t z_start(double chi0) { return llrint(chi0 * (4294967296.0 / kZTabH)); }
__device__ __forceinline__ int64_t z_step(double dchi) { return llrint(dchi * (4294967296.0 / kZTabH)); }
// The two nodes of the z(chi) table around a position in table steps times 2^32,
// and the place between them.
struct ZNodes {
  float z0, z1, t;
  // inside (uniform): the position is known to lie in the table
  __device__ __forceinline__ void send(const float* ztab, int64_t zp, bool inside = false) {
    const int64_t ip = zp >> 32;
    int iu;
    if (inside || (ip >= 0 && ip <= kZTabN - 2)) {
      iu = static_cast<int>(ip);
      t = static_cast<float>(static_cast<uint32_t>(zp)) * 2.3283064365386963e-10f;
    } else {  // beyond the table: the end interval continued linearly
      iu = ip < 0 ? 0 : kZTabN - 2;
      t = static_cast<float>(static_cast<double>(zp - (static_cast<int64_t>(iu) << 32)) * 2.3283064365386963e-10);
    }
    z0 = ztab[iu];
    z1 = ztab[iu + 1];
  }
};
__device__ __forceinline__ float fgpa_flux(const SkewerArgs& a, const ZNodes& z, float d, float e) {
  const float x = (z.z0 + z.t * (z.z1 - z.z0)) + (1.0f - kFgpaX0);   // (1+z) - x0
  const float ca = a.cf[0][0] + x * (a.cf[0][1] + x * a.cf[0][2]);
  const float cb = a.cf[1][0] + x * (a.cf[1][1] + x * a.cf[1][2]);
  const float cc = a.cf[2][0] + x * (a.cf[2][1] + x * a.cf[2][2]);
  return __expf(-ca * __expf(cb * (d + cc * e)));
}

// What small_scale_wave reads of the arguments.
struct LineNoise {
  static constexpr bool kPsTab = true;
  uint64_t seed;
  const float* ps_tab;
  int ps_fixed_amp;
};

// (the Gaussian mode's LDS leaves two waves per SIMD)
template <int U, int MODE, bool B16>
__global__ void __launch_bounds__(kSkNT, MODE == kSkGauss ? 2 : U == 1 ? 4 : 1) k_skewers(SkewerArgs a) {
  __shared__ float2 sbuf[kSkWaves][kHalfBuf];
  __shared__ __align__(8) float sgauss[MODE == kSkGauss ? kSkWaves : 1][MODE == kSkGauss ? kGaussWords : 1];
  constexpr bool kCellWalk = U == 1 && MODE != kSkGauss;
  __shared__ float4 scell[kCellWalk ? kSkWaves : 1][kCellWalk ? 4 * kCells : 1];
  __shared__ int sjb[kSkWaves][kMaxZBins + 1];
  __shared__ unsigned long long s_sum[kMaxZBins], s_cnt[kMaxZBins];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  for (int b = tid; b < kMaxZBins; b += kSkNT) {
    s_sum[b] = 0ull;
    s_cnt[b] = 0ull;
  }
  __syncthreads();
  const int N = a.n;
  const size_t NN = plane_pitch(N);
  const bool gather = a.in_dens == nullptr;
  const bool want_bins = a.n_bins > 0 && a.do_flux;
  float2* buf = sbuf[wv];
  int* jb = sjb[wv];
  LinePull<SkewerArgs, kSkWaves> pull;
  for (int64_t c = pull.first(lane); c < a.chunks; c = pull.next(lane)) {
    const auto* ca0 = kernarg_here<SkewerArgs>();
    const int64_t q0 = c * ca0->chunk;
    const int64_t q1 = q0 + ca0->chunk < ca0->n_sk ? q0 + ca0->chunk : ca0->n_sk;
    for (int64_t q = q0; q < q1; ++q) {
      if (q == q1 - 1) pull.ask(lane);
      const auto* la = kernarg_here<SkewerArgs>();   // what a line reads once
      const int np = la->npix[q];
      const int64_t off = la->offset[q];
      const double chi0 = la->chi0[q];
      int ns = 1;
      while (ns < np) ns <<= 1;
      const bool with_ds = (gather || la->ds_in_apply) && la->ps_amp > 0.0 && ns >= 2;
      // delta_S is drawn on lines of next_pow2(npix) <= 2048 pixels (the wave's
      // LDS line): a longer skewer is an input error, marked by NaN in every
      // output and left out of the bins
      if (with_ds && ns > 2 * kHalfMax) {
        const float qnan = __builtin_nanf("");
        for (int j = lane; j < np; j += 64) {
          if (la->dens) la->dens[off + j] = qnan;
          if (la->eta) la->eta[off + j] = qnan;
          if (la->flux) la->flux[off + j] = qnan;
        }
        continue;
      }
      // twiddles from global memory: a copy in LDS would cost this kernel its fourth block per CU
      int dl_lane = lane;
      if constexpr (MODE == kSkGauss) asm volatile("" : "+v"(dl_lane));
      if (with_ds) {
        const LineNoise ps{la->seed, la->ps_tab, la->ps_fixed_amp};
        small_scale_wave(ps, 0.0, 0.0, la->id_base + q, ns, buf, static_cast<const float2*>(la->tw2048), dl_lane);
      }
      // bin boundaries: jb[b] = first pixel with chi_j < edges[b] (chi_j decreases with j)
      if (want_bins) {
        bin_bounds(la->chi_edges, la->n_bins, chi0, la->dchi, np, jb, lane);
        wave_sync();
      }
      int64_t ox = 0, oy = 0, oz = 0, sx = 0, sy = 0, sz = 0;
      if (gather) {
        ox = la->origin_fx[3 * q];
        oy = la->origin_fx[3 * q + 1];
        oz = la->origin_fx[3 * q + 2];
        sx = la->step_fx[3 * q];
        sy = la->step_fx[3 * q + 1];
        sz = la->step_fx[3 * q + 2];
      }
      // wide-angle weights u_p u_q (off-diagonal ones doubled), u = step/|step|
      WideWeights ww{};
      if (MODE == kSkWide) {
        const double ux = static_cast<double>(sx), uy = static_cast<double>(sy), uz = static_cast<double>(sz);
        const double r2 = ux * ux + uy * uy + uz * uz;
        const double ir2 = r2 > 0.0 ? 1.0 / r2 : 0.0;
        ww.xx = static_cast<float>(ux * ux * ir2);
        ww.yy = static_cast<float>(uy * uy * ir2);
        ww.zz = static_cast<float>(uz * uz * ir2);
        ww.xy = static_cast<float>(2.0 * ux * uy * ir2);
        ww.xz = static_cast<float>(2.0 * ux * uz * ir2);
        ww.yz = static_cast<float>(2.0 * uy * uz * ir2);
      }
      if constexpr (kCellWalk) {
        if (gather && cells_fit(sx, sy, sz) && no_wrap(ox, oy, oz) && np > 0 && np < (1 << 28)) {
          // all loads of the next 64 pixels are sent for before the stores of these
          const int64_t uoff = lane_i64(off, 0);
          const LineOut dens(la->dens, uoff, np), eta(la->eta, uoff, np), flux(la->flux, uoff, np);
          BinWalk bins;
          if (want_bins) bins.start(jb, la->n_bins);
          const float* ds = reinterpret_cast<const float*>(buf) + lane + 2 * (lane >> 5);   // pixel j at j + 2 (j / 32)
          CellWalk<MODE, B16> walk;
          ZNodes zn;
          const int64_t zstep = z_step(la->dchi);
          int64_t zp = z_start(chi0) - lane * zstep;
          // the line, and the step sent for past its end, within the z(chi) table (a
          // line that is shorter than the table, so that zlast cannot wrap back into it)
          const int64_t zfirst = lane_i64(zp, 0), zlast = zfirst - static_cast<int64_t>(np + 127) * zstep;
          constexpr int64_t kZEnd = static_cast<int64_t>(kZTabN - 1) << 32;
          const bool inside = static_cast<double>(np + 127) * la->dchi < kZTabN * kZTabH && zfirst >= 0 &&
                              zfirst < kZEnd && zlast >= 0 && zlast < kZEnd;
          walk.start(ox, oy, oz, sx, sy, sz, lane);
          walk.send(a, sx, sy, sz, N, NN, lane);
          float4* rec = scell[wv];
          // (as two loops: a branch around the nodes' loads would hide their number)
          auto line = [&](auto with_flux) {
          constexpr bool FLUX = decltype(with_flux)::value;
          if (FLUX) zn.send(a.ztab, zp, inside);
          for (int it = 0; it < np; it += 64) {
            const int j = it + lane;
            float2 v0 = gauss_cell(walk.v[0][0]), v1 = gauss_cell(walk.v[0][1]);
            if constexpr (MODE == kSkWide) {
              v0.y = ww.eta(v0, gauss_cell(walk.v[1][0]), gauss_cell(walk.v[2][0]), gauss_cell(walk.v[3][0]));
              v1.y = ww.eta(v1, gauss_cell(walk.v[1][1]), gauss_cell(walk.v[2][1]), gauss_cell(walk.v[3][1]));
            }
            rec[lane] = make_float4(v0.x, v1.x - v0.x, v0.y, v1.y - v0.y);
            const float tx = static_cast<float>(walk.fr[0]) * 2.3283064365386963e-10f;
            const float ty = static_cast<float>(walk.fr[1]) * 2.3283064365386963e-10f;
            const float tz = static_cast<float>(walk.fr[2]) * 2.3283064365386963e-10f;
            const int k = static_cast<int>(walk.k);
            const ZNodes z = zn;
            wave_sync();
            walk.send(a, sx, sy, sz, N, NN, lane);   // (past the line's end too: every address is in the box)
            if (FLUX) {
              zp -= 64 * zstep;
              zn.send(a.ztab, zp, inside);
            }
            float col[2][4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              const float4 r = rec[4 * k + c];
              col[0][c] = r.x + tz * r.y;
              col[1][c] = r.z + tz * r.w;
            }
            float d = bilerp(tx, ty, col[0]);
            const float e = bilerp(tx, ty, col[1]);
            if (with_ds) d += ds[it + (it >> 4)];   // (past the line's end: unused slots of the buffer)
            wave_sync();   // the records are written again
            dens.put(j, d);
            eta.put(j, e);
            if (FLUX) {
              const float F = fgpa_flux(a, z, d, e);
              flux.put(j, F);
              if (want_bins) bins.add(jb, it, np, j, F, s_sum, lane);
            }
          }
          };
          if (la->do_flux) line(std::true_type{});
          else line(std::false_type{});
          if (want_bins) bins.end(jb, la->n_bins, s_sum, s_cnt, lane);
          wave_sync();  // the wave's LDS slice is reused by its next skewer
          continue;
        }
      }
      // fixed-point positions of the lane's pixels j = lane + 64 u, advanced by
      // one addition per step of 64 U pixels (pixels past the end wrap like any
      // other and are dropped)
      int64_t pos[U][3];
      const int64_t adv[3] = {64 * U * sx, 64 * U * sy, 64 * U * sz};
      int64_t zpos[U];   // the lane's pixels in the z(chi) table
      const int64_t zstep = z_step(la->dchi);
      if (a.do_flux) {
        const int64_t z0 = z_start(chi0);
#pragma unroll
        for (int u = 0; u < U; ++u) zpos[u] = z0 - (lane + 64 * u) * zstep;
      }
      if (MODE != kSkGauss) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int64_t j = lane + 64 * u;
          pos[u][0] = ox + j * sx;
          pos[u][1] = oy + j * sy;
          pos[u][2] = oz + j * sz;
        }
      }
      // pixel j is in bin b when jb[b+1] <= j < jb[b]; each lane walks j upward
      // and therefore the bins downward, accumulating one bin at a time.  U
      // pixels per lane per step: all their gathers are issued before any is used.
      int bin = la->n_bins - 1;
      int cur = -1;
      unsigned long long acc = 0ull, cnt = 0ull;
      // Gaussian mode: the geometry of the next 64 pixels, and their cells on the way
      [[maybe_unused]] GaussGeo geo;
      [[maybe_unused]] typename GaussCell<B16>::type pre[MODE == kSkGauss ? kGaussPre : 1];
      [[maybe_unused]] const int64_t o3[3] = {ox, oy, oz};
      [[maybe_unused]] const int32_t s3[3] = {static_cast<int32_t>(sx), static_cast<int32_t>(sy),
                                              static_cast<int32_t>(sz)};
      [[maybe_unused]] const int64_t st3[3] = {sx, sy, sz};
      [[maybe_unused]] const typename GaussCell<B16>::type* fb = nullptr;
      [[maybe_unused]] bool shared = false;   // quads share their window (steps below a third of a cell)
      if constexpr (MODE == kSkGauss) {
        if constexpr (B16) fb = a.field_bf16;
        else fb = a.field;
        constexpr int64_t kThird = (int64_t(1) << 32) / 3;
        shared = sx < kThird && sx > -kThird && sy < kThird && sy > -kThird && sz < kThird && sz > -kThird &&
                 no_wrap(ox, oy, oz);
        if (shared && np > 0) {
          geo = gauss_geo(o3, s3, 0, np, lane);
          if (geo.fast) gauss_load<B16>(fb, geo, N, NN, lane, pre);
        }
      }
      // the Gaussian mode runs every lane through every 64-pixel chunk (its
      // wave reductions need all lanes); lanes past the end are not stored
      for (int it = (MODE == kSkGauss ? 0 : lane); it < np; it += 64 * U) {
        const int j0 = MODE == kSkGauss ? it + lane : it;
        float dd[U], ee[U];
        if (gather) {
          float dl[U], el[U];
          if constexpr (MODE == kSkGauss) {
            static_assert(U == 1, "one pixel per lane");
            bool done = false;   // uniform
            if (shared) {
              const GaussGeo g = geo;
              float* lds = sgauss[wv];
              // planes in the slice together
              const int most = g.fast ? g.nx : min(g.nx, ((16 * kGaussRows) >> g.zs) / g.ny);
              if (g.fast) gauss_store(g, pre, lds, lane);
              else gauss_stage<B16>(fb, g, 0, most, N, NN, lane, lds);
              wave_sync();
              if (it + 64 < np) {  // the next pixels' cells
                geo = gauss_geo(o3, s3, it + 64, np, lane);
                if (geo.fast) gauss_load<B16>(fb, geo, N, NN, lane, pre);
              }
              float w[8], wz[8], wy[4][4], acc[4] = {0.0f, 0.0f, 0.0f, 0.0f}, wsum = 0.0f;
              const float ws = gauss_slots(g.t[1], g.sh1, w) * gauss_slots(g.t[2], g.sh2, wz);
              // lane l of a quad takes column l: component l & 1 of y row 2 jj + (l >> 1)
#pragma unroll
              for (int jj = 0; jj < 4; ++jj) {
                // (both rows' values first: a DPP move under a lane's condition
                // would not see the other lanes)
                const float a0 = w[2 * jj], a1 = w[2 * jj + 1];
                const float e0[4] = {dpp_f32<0x00>(a0), dpp_f32<0x55>(a0), dpp_f32<0xAA>(a0), dpp_f32<0xFF>(a0)};
                const float e1[4] = {dpp_f32<0x00>(a1), dpp_f32<0x55>(a1), dpp_f32<0xAA>(a1), dpp_f32<0xFF>(a1)};
#pragma unroll
                for (int p = 0; p < 4; ++p) wy[jj][p] = (lane & 2) ? e1[p] : e0[p];
              }
              for (int x0 = 0;;) {
                gauss_planes_add(g, x0, min(most, g.nx - x0), wz, wy, lds, lane, acc, wsum);
                wave_sync();  // the slice is loaded again
                x0 += most;
                if (x0 >= g.nx) break;
                gauss_stage<B16>(fb, g, x0, min(most, g.nx - x0), N, NN, lane, lds);
                wave_sync();
              }
              // the two row parities, then pixel p's components (columns 0 and 1) to lane p
#pragma unroll
              for (int p = 0; p < 4; ++p) acc[p] += dpp_f32<0x4E>(acc[p]);
              const int p = lane & 3;
              const float inv = 1.0f / (wsum * ws);
              const float d0 = dpp_f32<0x00>(acc[0]), d1 = dpp_f32<0x00>(acc[1]), d2 = dpp_f32<0x00>(acc[2]),
                          d3 = dpp_f32<0x00>(acc[3]);
              const float e0 = dpp_f32<0x55>(acc[0]), e1 = dpp_f32<0x55>(acc[1]), e2 = dpp_f32<0x55>(acc[2]),
                          e3 = dpp_f32<0x55>(acc[3]);
              dl[0] = (p == 0 ? d0 : p == 1 ? d1 : p == 2 ? d2 : d3) * inv;
              el[0] = (p == 0 ? e0 : p == 1 ? e1 : p == 2 ? e2 : e3) * inv;
              // a cell that is not finite spreads by the zero weights: such pixels
              // are taken again one by one
              done = !__any(!(fabsf(dl[0]) < HUGE_VALF) || !(fabsf(el[0]) < HUGE_VALF));
            }
            if (!done) {
              const int last = min(63, np - 1 - it), j = it + min(lane, last);
              const int64_t p3[3] = {ox + j * sx, oy + j * sy, oz + j * sz};
              GaussBox box;
              box.cells = 0;
              if (!shared) box = gauss_box(o3, st3, it, last);
              if (box.cells) gauss7_staged<B16>(fb, box, p3, N, NN, lane, reinterpret_cast<float2*>(sgauss[wv]), dl[0], el[0]);
              else gauss7_at<B16>(a, p3, N, NN, dl[0], el[0]);
            }
          } else {
          float2 c[U][MODE == kSkWide ? 4 : 8];   // columns or corners
          float t3[U][3];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int64_t px = pos[u][0], py = pos[u][1], pz = pos[u][2];
            pos[u][0] = px + adv[0];
            pos[u][1] = py + adv[1];
            pos[u][2] = pz + adv[2];
            const uint32_t msk = static_cast<uint32_t>(N - 1);
            const uint32_t ix = static_cast<uint32_t>(px >> 32) & msk;
            const uint32_t iy = static_cast<uint32_t>(py >> 32) & msk;
            const uint32_t iz = static_cast<uint32_t>(pz >> 32) & msk;
            const uint32_t jx = (ix + 1) & msk, jy = (iy + 1) & msk, jz = (iz + 1) & msk;
            t3[u][0] = static_cast<float>(static_cast<uint32_t>(px)) * 2.3283064365386963e-10f;
            t3[u][1] = static_cast<float>(static_cast<uint32_t>(py)) * 2.3283064365386963e-10f;
            t3[u][2] = static_cast<float>(static_cast<uint32_t>(pz)) * 2.3283064365386963e-10f;
            if constexpr (MODE == kSkWide) {
              // Lines come here whose steps are too long for the cell walk.  The four
              // columns, z taken, box by box: most of a voxel's cache line is a
              // neighbouring corner's, and with the four boxes in turn at each corner
              // the 64 lanes' lines left the L1 in between (1.2e8 FP32 pixels in
              // directions all over, 0.3 and 1 cells a step: 12.0 and 31.5 ms by two
              // corners, all four boxes each; 8.9 and 26.7 so; BF16 10.7 and 29.9, 8.1
              // and 24.5).  Three waves per SIMD, without FP32's spills, take 8.6 and 24.8,
              // but short lines there are 2-5% slower than on four.
              // plane offsets in 64 bits, offsets within a plane (< n^2) in 32
              const size_t x0 = static_cast<size_t>(ix) * NN, x1 = static_cast<size_t>(jx) * NN;
              const uint32_t y0 = iy * static_cast<uint32_t>(N), y1 = jy * static_cast<uint32_t>(N);
              const size_t col[4] = {x0 + y0, x0 + y1, x1 + y0, x1 + y1};
              typename GaussCell<B16>::type w[4][4][2];
#pragma unroll
              for (int f = 0; f < 4; ++f) {
                const typename GaussCell<B16>::type* b;
                if constexpr (B16) b = f == 0 ? a.field_bf16 : a.wide_bf16[f - 1];
                else b = f == 0 ? a.field : a.wide[f - 1];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                  w[f][k][0] = b[col[k] + iz];
                  w[f][k][1] = b[col[k] + jz];
                }
              }
#pragma unroll
              for (int k = 0; k < 4; ++k) {
                const float2 v0 = gauss_cell(w[0][k][0]), v1 = gauss_cell(w[0][k][1]);
                const float e0 = ww.eta(v0, gauss_cell(w[1][k][0]), gauss_cell(w[2][k][0]), gauss_cell(w[3][k][0]));
                const float e1 = ww.eta(v1, gauss_cell(w[1][k][1]), gauss_cell(w[2][k][1]), gauss_cell(w[3][k][1]));
                c[u][k] = make_float2(v0.x + t3[u][2] * (v1.x - v0.x), e0 + t3[u][2] * (e1 - e0));
              }
            } else {
              // byte addresses: each x plane's start as one 32 x 32 -> 64-bit
              // multiply-add on the box pointer, the corner's offset within the
              // plane (below 2^25 bytes) added to it
              constexpr uint32_t ES = B16 ? 4u : 8u;
              const char* fb = B16 ? reinterpret_cast<const char*>(a.field_bf16) : reinterpret_cast<const char*>(a.field);
              const uint32_t pb = static_cast<uint32_t>(NN) * ES;  // plane pitch in bytes (< 2^32)
              const char* p0 = fb + static_cast<uint64_t>(ix) * pb;
              const char* p1 = fb + static_cast<uint64_t>(jx) * pb;
              const uint32_t y0 = iy * (static_cast<uint32_t>(N) * ES), y1 = jy * (static_cast<uint32_t>(N) * ES);
              const uint32_t z0 = iz * ES, z1 = jz * ES;
              const uint32_t o[4] = {y0 + z0, y0 + z1, y1 + z0, y1 + z1};
#pragma unroll
              for (int k = 0; k < 8; ++k) {
                const char* pk = (k < 4 ? p0 : p1) + o[k & 3];
                if constexpr (B16)
                  c[u][k] = unpack_bf16x2(*reinterpret_cast<const uint32_t*>(pk));
                else
                  c[u][k] = *reinterpret_cast<const float2*>(pk);
              }
            }
          }
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const float tx = t3[u][0], ty = t3[u][1], tz = t3[u][2];
            if constexpr (MODE == kSkWide) {
              const float cd[4] = {c[u][0].x, c[u][1].x, c[u][2].x, c[u][3].x};
              const float ce[4] = {c[u][0].y, c[u][1].y, c[u][2].y, c[u][3].y};
              dl[u] = bilerp(tx, ty, cd);
              el[u] = bilerp(tx, ty, ce);
            } else {
              dl[u] = trilerp(tx, ty, tz, c[u][0].x, c[u][1].x, c[u][2].x, c[u][3].x, c[u][4].x, c[u][5].x,
                              c[u][6].x, c[u][7].x);
              el[u] = trilerp(tx, ty, tz, c[u][0].y, c[u][1].y, c[u][2].y, c[u][3].y, c[u][4].y, c[u][5].y,
                              c[u][6].y, c[u][7].y);
            }
          }
          }
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int j = j0 + 64 * u;
            float d = dl[u];
            const float e = el[u];
            if (j < np) {
              if (with_ds) {
                const float2 z2 = buf[pidx(j >> 1)];
                d += (j & 1) ? z2.y : z2.x;
              }
              if (a.dens) a.dens[off + j] = d;
              if (a.eta) a.eta[off + j] = e;
            }
            dd[u] = d;
            ee[u] = e;
          }
        } else {
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int j = j0 + 64 * u;
            dd[u] = j < np ? a.in_dens[off + j] : 0.0f;
            ee[u] = j < np ? a.in_eta[off + j] : 0.0f;
            if (with_ds && j < np) {
              const float2 z2 = buf[pidx(j >> 1)];
              dd[u] += (j & 1) ? z2.y : z2.x;
            }
          }
        }
        if (a.do_flux) {
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int j = j0 + 64 * u;
            if (j >= np) break;
            const float d = dd[u], e = ee[u];
            ZNodes z;
            z.send(a.ztab, zpos[u]);
            const float F = fgpa_flux(a, z, d, e);
            if (a.flux) a.flux[off + j] = F;
            if (want_bins) {
              while (bin >= 0 && j >= jb[bin]) --bin;  // pixel j lies below bin's upper edge
              const int key = (bin >= 0 && j >= jb[bin + 1]) ? bin : -1;
              if (key != cur) {
                if (cnt) {
                  atomicAdd(&s_sum[cur], acc);
                  atomicAdd(&s_cnt[cur], cnt);
                }
                acc = 0ull;
                cnt = 0ull;
                cur = key;
              }
              if (key >= 0) {
                acc += __float2ull_rn(F * 4294967296.0f);
                cnt += 1ull;
              }
            }
          }
#pragma unroll
          for (int u = 0; u < U; ++u) zpos[u] -= 64 * U * zstep;
        }
      }
      if (cnt) {
        atomicAdd(&s_sum[cur], acc);
        atomicAdd(&s_cnt[cur], cnt);
      }
      wave_sync();  // the wave's LDS slice is reused by its next skewer
    }
  }
  if (want_bins) {
    __syncthreads();
    const int copy = static_cast<int>(blockIdx.x % kBinCopies) * kMaxZBins;
    for (int b = tid; b < a.n_bins; b += kSkNT) {
      if (s_cnt[b]) {
        atomicAdd(&a.bin_sum[copy + b], s_sum[b]);
        atomicAdd(&a.bin_cnt[copy + b], s_cnt[b]);
      }
    }
  }
}

int device_cus() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (!cached[dev]) {
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) cus = 256;
    cached[dev] = cus;
  }
  return cached[dev];
}

template <bool B16>
void launch_skewer_kernel(const SkewerArgs& a, int u, dim3 grid, hipStream_t st) {
  if (a.is_gauss) {
    // 343 gathers per pixel: one pixel per lane at a time
    LYA_TIMED("skewers_gauss", st, hipLaunchKernelGGL((k_skewers<1, kSkGauss, B16>), grid, dim3(kSkNT), 0, st, a));
  } else if (a.is_wide) {
    // four boxes per pixel: one pixel per lane at a time, whatever the unroll
    LYA_TIMED("skewers_wide", st, hipLaunchKernelGGL((k_skewers<1, kSkWide, B16>), grid, dim3(kSkNT), 0, st, a));
  } else if (u == 1) {
    LYA_TIMED(a.in_dens ? "apply_fgpa" : "skewers", st,
              hipLaunchKernelGGL((k_skewers<1, kSkTri, B16>), grid, dim3(kSkNT), 0, st, a));
  } else if (u == 2) {
    LYA_TIMED(a.in_dens ? "apply_fgpa" : "skewers", st,
              hipLaunchKernelGGL((k_skewers<2, kSkTri, B16>), grid, dim3(kSkNT), 0, st, a));
  } else {
    LYA_TIMED(a.in_dens ? "apply_fgpa" : "skewers", st,
              hipLaunchKernelGGL((k_skewers<4, kSkTri, B16>), grid, dim3(kSkNT), 0, st, a));
  }
}

SkLaunch sk_launch(int64_t n_sk, int chunk, int blocks_per_cu, int unroll) {
  SkLaunch l{};
  l.blocks = static_cast<int64_t>(device_cus()) * (blocks_per_cu > 0 ? blocks_per_cu : 4);
  // no more skewers per pull than leave every wave of the grid eight pulls: longer
  // ones leave it uneven at the end (35M stored pixels of 50,000 skewers 568 us in
  // pulls of 4, 482 us one by one), and 500 skewers of 256 pixels in pulls of 4 ran
  // on 125 waves, four in a row each (39.5 us; one per wave 18.6 us)
  l.chunk = static_cast<int>(std::min<int64_t>(chunk, std::max<int64_t>(1, n_sk / (8 * l.blocks * kSkWaves))));
  l.chunks = (n_sk + l.chunk - 1) / l.chunk;
  if (l.blocks * kSkWaves > l.chunks) l.blocks = (l.chunks + kSkWaves - 1) / kSkWaves;
  if (l.blocks < 1) l.blocks = 1;
  // with at most a skewer per wave the trilinear pass is one skewer's latency: the
  // gathers of four steps of 64 pixels go out together, against one step's on the
  // cell walk (calls without FGPA in a 512^3 box, 250 and 1500 pixels: one line 9.8
  // and 21.8 us, walk 12.0 and 27.2; 500 lines 11.3 and 26.7, walk 13.0 and 30.6; with
  // FGPA 26.1 and 47.2, walk 26.6 and 45.3).  From about half the waves up the
  // walk would gain again (4000 lines 19.4 and 59.0 us, walk 17.4 and 51.1; 20-2000
  // pixels 42.4, walk 50.0).  Every unroll gives the same bits.
  const bool few = n_sk <= l.blocks * kSkWaves;
  l.unroll = few ? 4 : unroll == 1 || unroll == 4 ? unroll : 2;
  return l;
}

hipError_t launch_skewers(SkewerArgs a, hipStream_t st) {
  const SkLaunch l = sk_launch(a.n_sk, a.chunk, a.blocks_per_cu, a.unroll);
  a.chunk = l.chunk;
  a.chunks = l.chunks;
  const dim3 grid(static_cast<unsigned>(l.blocks));
  if (a.field_bf16)
    launch_skewer_kernel<true>(a, l.unroll, grid, st);
  else
    launch_skewer_kernel<false>(a, l.unroll, grid, st);
  if (a.n_bins > 0 && a.do_flux)
    LYA_TIMED("skewer_finalize", st,
              hipLaunchKernelGGL(k_skewer_finalize, dim3(1), dim3(256), 0, st, a.n_bins, a.bin_sum, a.bin_cnt,
                                 a.out_fsum, a.out_count));
  return hipGetLastError();
}

}  // namespace lya
