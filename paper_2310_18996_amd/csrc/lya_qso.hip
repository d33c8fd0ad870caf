// Lognormal quasar field (gfx950), section "Quasar generation" and Appendix A:
//   * xi_m(r) of the smoothed matter spectrum and the lognormal spectrum
//     P_q(k) = FT of ln(1 + b_0^2 xi_m), both in FP64;
//   * the variance of a box (a reduction over the grid);
//   * per comoving distance: z and the three-box coefficients c_i(z);
//   * the draw: every voxel is selected with probability
//     p = nbar(z) dx^3 sum_i c_i(z) exp(a_i(z) delta_i - a_i(z)^2 var_i / 2),
//     a_i(z) = b_q(z) (1 + z_i) / (b_q(z_i) (1 + z)) = ((1 + z)/(1 + z_i))^0.7
//     for b_q proportional to (1 + z)^1.7, and a selected voxel gets a
//     uniform position inside it;
//   * the catalogue: each quasar's redshift with its line-of-sight velocity
//     (eq:velocity) and its line of sight as a skewer-table row.
#include <algorithm>

#include "lya_internal.h"

namespace lya {

namespace {

// Sum over a 256-thread block; the result is valid in thread 0.
__device__ double block_sum256(double v, double* red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return threadIdx.x == 0 ? red[0] + red[1] + red[2] + red[3] : 0.0;
}

}  // namespace

// Both transforms are sums over uniform nodes, T(x) = sum_j f_j sin(j h x):
// xi_m(r) over k_j = j h, P_q(k) over r_i = i dr.  The nodes go in groups of
// kSineJ = 2 kSineB around a half-integer centre c: with beta = (b + 1/2) h x,
//   f+ sin(phi + beta) + f- sin(phi - beta)
//     = sin phi cos beta (f+ + f-) + cos phi sin beta (f+ - f-),  phi = c h x,
// so a pair of nodes costs two FMAs once cos beta and sin beta, the same in
// every group, sit in registers (one lane per x), and the sums and differences
// f+ +- f- (the same for every lane) come as scalar operands: one FP64 FMA per
// node and x, where a rotation per node takes five.  sin phi and cos phi turn
// by J h x per group, from an exact sincos every kSineSync groups.  Bound by
// FP64 FMA issue (4.4e9 nodes x r values, 0.11 ms of FMAs at 40001 r and 1.1e5
// k nodes): 2.18 -> 0.29 ms.  x = 0 (or below) takes the limit sum_j f_j (j h):
// sin y -> y / x, cos -> 1.
// Group a of sd: kSineB sums f+ + f-, then kSineB differences f+ - f-, with
// f+ = f[J a + B + b], f- = f[J a + B - 1 - b].
constexpr int kSineSync = 32;

__global__ void __launch_bounds__(256) k_sine_sum(const double* __restrict__ sd, int na, int per_seg, double h,
                                                  const double* __restrict__ xv, double dx, int nx,
                                                  double* __restrict__ part) {
  constexpr int B = kSineB, J = kSineJ;
  const int i = blockIdx.x * 256 + threadIdx.x;
  const double x = i >= nx ? 0.0 : xv ? xv[i] : dx * i;
  const bool lim = !(x > 0.0);
  // a turn by (h x), an exact start at h x / 2 and B - 1 turns; limit: sin -> the
  // angle over x, cos -> 1, which the turns keep
  double cb[B], sb[B], st, ct, sr, cr;
  sincos(0.5 * h * x, &sb[0], &cb[0]);
  sincos(h * x, &st, &ct);
  sincos(J * h * x, &sr, &cr);
  if (lim) {
    sb[0] = 0.5 * h;
    st = h;
    sr = J * h;
    cb[0] = ct = cr = 1.0;
  }
  const double st0 = lim ? 0.0 : st, sr0 = lim ? 0.0 : sr;  // no sin sin term in the limit
#pragma unroll
  for (int b = 1; b < B; ++b) {
    sb[b] = fma(sb[b - 1], ct, cb[b - 1] * st);
    cb[b] = fma(cb[b - 1], ct, -(sb[b - 1] * st0));
  }
  const int a0 = blockIdx.y * per_seg, a1 = min(a0 + per_seg, na);
  double tot = 0.0;
  for (int as = a0; as < a1; as += kSineSync) {
    const double kc = h * (static_cast<double>(J) * as + (B - 0.5));
    double sp, cp;
    sincos(kc * x, &sp, &cp);
    if (lim) {
      sp = kc;
      cp = 1.0;
    }
    const int ae = min(as + kSineSync, a1);
    for (int a = as; a < ae; ++a) {
      const double* __restrict__ f = sd + static_cast<size_t>(a) * J;
      double u0 = 0.0, u1 = 0.0, v0 = 0.0, v1 = 0.0;
#pragma unroll
      for (int b = 0; b < B; b += 2) {
        u0 = fma(f[b], cb[b], u0);
        u1 = fma(f[b + 1], cb[b + 1], u1);
        v0 = fma(f[B + b], sb[b], v0);
        v1 = fma(f[B + b + 1], sb[b + 1], v1);
      }
      tot = fma(sp, u0 + u1, fma(cp, v0 + v1, tot));
      const double t = fma(sp, cr, cp * sr);
      cp = fma(cp, cr, -(sp * sr0));
      sp = t;
    }
  }
  if (i < nx) part[static_cast<size_t>(blockIdx.y) * nx + i] = tot;
}

// Segments of the groups (blockIdx.y): enough for about kSineWaves waves in
// all (four per SIMD), at least eight groups each.
SineShape sine_shape(int n_nodes, int nx) {
  constexpr int kMaxSegs = 64;
  SineShape s{};
  s.na = (n_nodes + kSineJ - 1) / kSineJ;
  const int waves = (nx + 255) / 256 * 4;
  int segs = std::max(1, std::min(kMaxSegs, kSineWaves / std::max(1, waves)));
  segs = std::min(segs, (s.na + 7) / 8);
  s.per_seg = (s.na + segs - 1) / segs;
  s.segs = (s.na + s.per_seg - 1) / s.per_seg;
  return s;
}

// in order, the loads of 16 segments in flight at once (one after another they
// were most of k_lognormal_pq's 17 us)
__device__ __forceinline__ double sine_total(const double* part, int segs, int nx, int i) {
  double s = 0.0;
  for (int k0 = 0; k0 < segs; k0 += 16) {
    double v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = part[static_cast<size_t>(min(k0 + k, segs - 1)) * nx + i];
#pragma unroll
    for (int k = 0; k < 16; ++k) s += k0 + k < segs ? v[k] : 0.0;
  }
  return s;
}

// xi_i = (the sum at r_i = i dr) / (2 pi^2 r_i), then g_i = Simpson weight
// (dr/3) ln(1 + b2 xi_i) r_i (n_r odd) in the groups of k_sine_sum.  part may
// be xi itself (one segment): a thread writes only the values it has read.
__global__ void __launch_bounds__(256) k_lognormal_g(const double* part, int segs, int n_r, double dr, double b2,
                                                     double* xi, double* __restrict__ sd, int na) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  const int a = t / kSineB, b = t % kSineB;
  if (a >= na) return;
  auto g = [&](int i) {
    if (i >= n_r) return 0.0;
    const double r = dr * i, tot = sine_total(part, segs, n_r, i);
    const double x = (i == 0 ? tot : tot / r) / (2.0 * M_PI * M_PI);
    xi[i] = x;
    const double w = (i == 0 || i == n_r - 1) ? 1.0 : ((i & 1) ? 4.0 : 2.0);
    return w * dr / 3.0 * log1p(b2 * x) * r;
  };
  const double fp = g(a * kSineJ + kSineB + b), fm = g(a * kSineJ + kSineB - 1 - b);
  sd[static_cast<size_t>(a) * kSineJ + b] = fp + fm;
  sd[static_cast<size_t>(a) * kSineJ + kSineB + b] = fp - fm;
}

// P_q(k) = 4 pi / k times the sum over r (k = 0: 4 pi times the limit), then
// values below 1e-12 of the largest raised to that floor, so that the result
// can serve as a tabulated spectrum (ln P interpolation).  One block; part may
// be pq itself (one segment).
__global__ void __launch_bounds__(1024) k_lognormal_pq(const double* part, int segs, int n_k,
                                                       const double* __restrict__ kv, double* pq) {
  __shared__ double red[16];
  double mx = 0.0;
  for (int i = threadIdx.x; i < n_k; i += 1024) {
    const double k = kv[i], tot = sine_total(part, segs, n_k, i);
    const double v = 4.0 * M_PI * (k <= 0.0 ? tot : tot / k);
    pq[i] = v;
    mx = fmax(mx, v);
  }
  for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_down(mx, o, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
  __syncthreads();
  mx = 0.0;
  for (int w = 0; w < 16; ++w) mx = fmax(mx, red[w]);
  const double fl = 1e-12 * mx;
  if (fl <= 0.0) return;
  for (int i = threadIdx.x; i < n_k; i += 1024) pq[i] = fmax(pq[i], fl);  // each thread its own values
}

hipError_t launch_lognormal(const PkParams& p, const LognormalArgs& a, hipStream_t st) {
  hipError_t e = launch_xi_weights(p, a.smooth, a.h, a.m, a.partial, a.f, st);
  if (e != hipSuccess) return e;
  const SineShape sx = sine_shape(a.m + 1, a.n_r), sk = sine_shape(a.n_r, a.n_k);
  double* px = sx.segs == 1 ? a.xi : a.part;  // the caller's array where one segment holds the sums
  double* pk = sk.segs == 1 ? a.pq : a.part;
  LYA_TIMED("xi_r", st,
            hipLaunchKernelGGL(k_sine_sum, dim3((a.n_r + 255) / 256, sx.segs), dim3(256), 0, st, a.f, sx.na,
                               sx.per_seg, a.h, static_cast<const double*>(nullptr), a.dr, a.n_r, px));
  LYA_TIMED("lognormal_g", st,
            hipLaunchKernelGGL(k_lognormal_g, dim3((sk.na * kSineB + 255) / 256), dim3(256), 0, st, px, sx.segs,
                               a.n_r, a.dr, a.b2, a.xi, a.g, sk.na));
  if (a.n_k > 0) {
    LYA_TIMED("lognormal_sum", st,
              hipLaunchKernelGGL(k_sine_sum, dim3((a.n_k + 255) / 256, sk.segs), dim3(256), 0, st, a.g, sk.na,
                                 sk.per_seg, a.dr, a.k, 0.0, a.n_k, pk));
    LYA_TIMED("lognormal_pq", st,
              hipLaunchKernelGGL(k_lognormal_pq, dim3(1), dim3(1024), 0, st, pk, sk.segs, a.n_k, a.k, a.pq));
  }
  return hipGetLastError();
}

// ---- box moments ----
// Per block: sums of re, re^2, im, im^2 over segments of 1024 cells (each in one
// plane: n^2 is a multiple), two cells per 16-byte load (planes start 16-byte
// aligned), kMomSegs segments' loads in flight.  Bound by reading the box: 1024^3 in
// 1.49 ms, with NT (non-temporal loads) 1.27 ms.
constexpr int kMomSeg = 1024, kMomSegs = 4;
// NT where a box is beyond the 256 MB last-level cache: no read of it would find
// anything there, and not allocating there is faster.
bool box_streams(int n) { return sizeof(float2) * box_elems(n) > (size_t(256) << 20); }
template <bool NT>
__global__ void __launch_bounds__(256) k_box_moments(const float2* __restrict__ box, int log2n2, size_t pitch,
                                                     int64_t segs, double* __restrict__ part) {
  constexpr int SEGS = kMomSegs;
  typedef float f4 __attribute__((ext_vector_type(4)));
  __shared__ double red[4];
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  const size_t pad = pitch - (static_cast<size_t>(1) << log2n2);
  for (int64_t g = blockIdx.x; g < segs; g += static_cast<int64_t>(gridDim.x) * SEGS) {
    f4 v[SEGS][2];
#pragma unroll
    for (int k = 0; k < SEGS; ++k) {
      const int64_t gk = g + static_cast<int64_t>(gridDim.x) * k;
      const size_t c = static_cast<size_t>(gk < segs ? gk : g) * kMomSeg;
      const f4* q = reinterpret_cast<const f4*>(box + c + (c >> log2n2) * pad) + threadIdx.x;
#pragma unroll
      for (int h = 0; h < 2; ++h) v[k][h] = NT ? __builtin_nontemporal_load(q + 256 * h) : q[256 * h];
    }
#pragma unroll
    for (int k = 0; k < SEGS; ++k) {
      if (g + static_cast<int64_t>(gridDim.x) * k >= segs) break;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const f4 w = v[k][h];
        s[0] += static_cast<double>(w.x) + w.z;
        s[1] += static_cast<double>(w.x) * w.x + static_cast<double>(w.z) * w.z;
        s[2] += static_cast<double>(w.y) + w.w;
        s[3] += static_cast<double>(w.y) * w.y + static_cast<double>(w.w) * w.w;
      }
    }
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const double t = block_sum256(s[c], red);
    if (threadIdx.x == 0) part[blockIdx.x * 4 + c] = t;
    __syncthreads();
  }
}

// out = {mean re, var re, mean im, var im} over the n^3 grid points.
__global__ void __launch_bounds__(256) k_box_moments_final(const double* __restrict__ part, int nblocks,
                                                           double inv_count, double* __restrict__ out) {
  __shared__ double red[4];
  double t[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    double s = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += 256) s += part[b * 4 + c];
    t[c] = block_sum256(s, red);
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double m0 = t[0] * inv_count, m1 = t[2] * inv_count;
    out[0] = m0;
    out[1] = t[1] * inv_count - m0 * m0;
    out[2] = m1;
    out[3] = t[3] * inv_count - m1 * m1;
  }
}

hipError_t launch_box_moments(const float2* box, int n, double* part, double* out, hipStream_t st) {
  int log2n2 = 0;
  while ((int64_t(1) << log2n2) < static_cast<int64_t>(n) * n) ++log2n2;
  const int64_t segs = static_cast<int64_t>(n) * n * n / kMomSeg;
  LYA_TIMED("box_moments", st,
            hipLaunchKernelGGL(box_streams(n) ? k_box_moments<true> : k_box_moments<false>, dim3(kQsoMomBlocks), dim3(256),
                               0, st, box, log2n2, plane_pitch(n), segs, part));
  const double inv = 1.0 / (static_cast<double>(n) * n * n);
  LYA_TIMED("box_moments_final", st,
            hipLaunchKernelGGL(k_box_moments_final, dim3(1), dim3(256), 0, st, part, kQsoMomBlocks, inv, out));
  return hipGetLastError();
}

// ---- per-distance table: {z, c_1, c_2, c_3} at chi = i kZTabH ----
__device__ __forceinline__ double bias_qso(double z) { return 3.7 * pow((1.0 + z) / 3.33, 1.7); }

__global__ void __launch_bounds__(256) k_qso_coef(const float* __restrict__ ztab, QsoCoef c, float4* __restrict__ tab,
                                                  unsigned long long* count) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i == 0) *count = 0ull;  // of the draw that follows
  if (i >= kZTabN) return;
  const double z = ztab[i];
  double cf[3] = {1.0, 0.0, 0.0};
  if (c.nb == 3) {
    double xi[3];
    for (int j = 0; j < 3; ++j) {
      const double al = pow((1.0 + z) / (1.0 + c.z[j]), 0.7);
      xi[j] = pow(1.0 + c.b2[j] * c.xi5, al * al) - 1.0;
    }
    const double gq = c.g_ref * (1.0 + c.z_ref) / (1.0 + z);
    const double bz = bias_qso(z) * gq;
    const double xi_mod = bz * bz * c.xi5;
    const double t12 = (z - c.z[0]) / (c.z[1] - c.z[0]);
    const double t23 = (z - c.z[1]) / (c.z[2] - c.z[1]);
    const double xi12 = (1.0 - t12) * xi[0] + t12 * xi[1];
    const double xi23 = (1.0 - t23) * xi[1] + t23 * xi[2];
    const double den = xi12 - xi23;
    const double w = fabs(den) <= 1e-12 * fabs(xi[1]) ? 0.5 : fmin(fmax((xi_mod - xi23) / den, 0.0), 1.0);
    cf[0] = w * (1.0 - t12);
    cf[1] = w * t12 + (1.0 - w) * (1.0 - t23);
    cf[2] = (1.0 - w) * t23;
  }
  tab[i] = make_float4(static_cast<float>(z), static_cast<float>(cf[0]), static_cast<float>(cf[1]),
                       static_cast<float>(cf[2]));
}

// ---- the draw ----
// A thread takes VPT consecutive voxels along z at a time (one Philox call gives
// the decision uniforms of four), a wave `tiles` times 64 VPT of them.  Selected
// voxels wait in the wave's LDS list and leave it with one atomic on the count per
// flush (one per tile was an atomic per quasar, and additions to one cache line
// take 11.5 ns each); a slot at or beyond cap is counted but not written.
// The transcendentals run on the hardware units (v_sqrt_f32, v_log_f32,
// v_exp_f32: about 1 ulp each); the exponent's own rounding, |x| 2^-24 for
// |x| up to about 10, dominates the error of p (a few 1e-7 relative).
//
// Almost every voxel is rejected (p about 1e-4), so p itself is formed only where
// an upper bound does not already reject (qso_bound): Philox, two FMAs, a maximum
// and a comparison per box and voxel in place of 8 transcendentals and two table
// gathers.  1024^3, three boxes: 6.52 ms bound by vector issue and by the L1, 3.07 ms
// (reading the boxes takes 2.6).
constexpr float kLog2e = 1.4426950408889634f;
constexpr int kQsoVpt = 8;      // voxels per thread and tile (consecutive along z)
constexpr int kQsoBlock = 256;
constexpr int kQsoMaxTiles = 64;
constexpr int kQsoFlush = 256;
constexpr int kQsoList = 768;   // per wave: flushed above kQsoFlush, a tile adds at most 512

// Voxel (ix, iy, iz0) .. + VPT - 1 along z.
struct QsoCell {
  int ix, iy, iz0;
  __device__ __forceinline__ QsoCell(const QsoDrawArgs& a, uint64_t v0) {
    // n is a power of two: shifts and masks instead of 64-bit divisions
    const uint64_t row = v0 >> a.log2n;
    iz0 = static_cast<int>(v0 & static_cast<uint64_t>(a.n - 1));
    ix = static_cast<int>(row >> a.log2n);
    iy = static_cast<int>(row & static_cast<uint64_t>(a.n - 1));
  }
  __device__ __forceinline__ float r2xy(const QsoDrawArgs& a) const {
    const float rx = static_cast<float>(ix * a.dx_d - a.o[0]);
    const float ry = static_cast<float>(iy * a.dx_d - a.o[1]);
    return rx * rx + ry * ry;
  }
};

// Bound of VPT voxels: p = nb dx^3 sum_i c_i 2^(x_i), x_i = log2(e) (al_i d_i -
// al_i^2 var_i / 2), is below u wherever log2 u >= max(lo_i d_i, hi_i d_i) + add_i
// for every box i, since the voxels' al_i lie between lo_i and hi_i (over log2 e),
// their c_i below the largest that any weight 0 <= w <= 1 gives between the ends'
// redshifts, and nb below nb_top.  Redshift ends: the table nodes around the
// voxels' distances; all else is widened by a few parts in 10^6 (above every
// rounding of the exact evaluation) and 1e-3 in the exponent.  A NaN anywhere makes
// a comparison false, which keeps the voxel.
template <int NB>
struct QsoBound {
  float lo[NB], hi[NB], add[NB];
};
template <int VPT>
__device__ __forceinline__ float2 qso_ends(const QsoDrawArgs& a, float r2xy, int iz0) {
  const float ra = static_cast<float>(iz0) * a.dx - a.oz, rb = static_cast<float>(iz0 + VPT - 1) * a.dx - a.oz;
  const float r_lo = ra <= 0.0f && rb >= 0.0f ? 0.0f : fminf(ra * ra, rb * rb), r_hi = fmaxf(ra * ra, rb * rb);
  const float per_h = 1.0f / static_cast<float>(kZTabH);
  const float t_lo = __builtin_amdgcn_sqrtf(r2xy + r_lo) * per_h * (1.0f - 4e-6f);
  const float t_hi = __builtin_amdgcn_sqrtf(r2xy + r_hi) * per_h * (1.0f + 4e-6f);
  // from where the table may fall or hold no number (towards the horizon) nothing
  // bounds the voxels between its nodes: they are all kept
  if (!(t_hi < a.t_rise)) return make_float2(__builtin_nanf(""), __builtin_nanf(""));
  return make_float2(a.tab[min(static_cast<int>(t_lo), kZTabN - 2)].x,
                     a.tab[min(static_cast<int>(t_hi), kZTabN - 2) + 1].x);
}
template <int NB>
__device__ __forceinline__ QsoBound<NB> qso_bound(const QsoDrawArgs& a, float2 ends, const float (&hv)[NB], float nb_top) {
  const float z_lo = ends.x - 2e-5f, z_hi = ends.y + 2e-5f;
  const float l_lo = __log2f(1.0f + z_lo), l_hi = __log2f(1.0f + z_hi);
  float c = 1.0f;
  if (NB == 3) {
    const float i12 = 1.0f / (a.zb[1 % NB] - a.zb[0]), i23 = 1.0f / (a.zb[2 % NB] - a.zb[1 % NB]);
    const float c0 = (a.zb[1 % NB] - z_lo) * i12, c2 = (z_hi - a.zb[1 % NB]) * i23;
    const float c1 = fmaxf((z_hi - a.zb[0]) * i12, (a.zb[2 % NB] - z_lo) * i23);
    c = fmaxf(c0, 0.0f) + fmaxf(c1, 0.0f) + fmaxf(c2, 0.0f);
  }
  // (not below 2^-127: there a p that overflows its factors is kept as well)
  const float top = fmaxf(__log2f(nb_top * a.dx3 * c) + 1e-3f, -127.0f);
  QsoBound<NB> b;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const float al_lo = __builtin_amdgcn_exp2f(0.7f * (l_lo - a.l2z[i])) * (1.0f - 4e-6f);
    const float al_hi = __builtin_amdgcn_exp2f(0.7f * (l_hi - a.l2z[i])) * (1.0f + 4e-6f);
    b.lo[i] = kLog2e * al_lo;
    b.hi[i] = kLog2e * al_hi;
    b.add[i] = top - kLog2e * (hv[i] >= 0.0f ? al_lo * al_lo : al_hi * al_hi) * hv[i];
  }
  return b;
}

// p of one voxel against u, the field values d.
template <int NB>
__device__ __forceinline__ bool qso_selected(const QsoDrawArgs& a, float r2xy, int iz, const float (&d)[NB],
                                             const float (&hv)[NB], float nb_top, float u, const float* snz,
                                             const float* snb) {
  const float rz = static_cast<float>(iz) * a.dx - a.oz;
  const float chi = __builtin_amdgcn_sqrtf(r2xy + rz * rz);
  const float t = chi * (1.0f / static_cast<float>(kZTabH));
  const int i0 = min(static_cast<int>(t), kZTabN - 2);
  const float fr = t - static_cast<float>(i0);
  const float4 c0 = a.tab[i0], c1 = a.tab[i0 + 1];
  const float z = c0.x + fr * (c1.x - c0.x);
  const float cf[3] = {c0.y + fr * (c1.y - c0.y), c0.z + fr * (c1.z - c0.z), c0.w + fr * (c1.w - c0.w)};
  const float lz = __log2f(1.0f + z);
  float acc;
  if (NB == 1) {
    const float al = __builtin_amdgcn_exp2f(0.7f * (lz - a.l2z[0]));
    acc = __builtin_amdgcn_exp2f(kLog2e * (al * d[0] - al * al * hv[0]));
  } else {
    acc = 0.0f;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const float al = __builtin_amdgcn_exp2f(0.7f * (lz - a.l2z[i]));
      acc += cf[i] * __builtin_amdgcn_exp2f(kLog2e * (al * d[i] - al * al * hv[i]));
    }
  }
  // p <= nb_top dx^3 acc (rounding is monotone): most are rejected on that
  // bound before nbar(z) is looked up
  if (!(u < fminf(nb_top * a.dx3 * acc, 1.0f))) return false;
  // nbar(z): linear between the nodes, zero outside
  float nb = 0.0f;
  if (z >= snz[0] && z <= snz[a.n_nbar - 1]) {
    int lo = 0, hi = a.n_nbar - 1;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (snz[mid] <= z) lo = mid; else hi = mid;
    }
    const float span = snz[hi] - snz[lo];
    nb = span > 0.0f ? snb[lo] + (snb[hi] - snb[lo]) * ((z - snz[lo]) / span) : snb[lo];
  }
  return u < fminf(nb * a.dx3 * acc, 1.0f);
}

// Two cells (16 bytes) per lane from memory to LDS, lane after lane from dst (the same
// in all lanes).  DMA: straight there, for boxes that start 16-byte aligned (and
// so do their rows and planes); other boxes cell by cell through registers.
template <bool NT, bool DMA>
__device__ __forceinline__ void to_lds(const float2* src, float4* dst, int lane) {
  if constexpr (DMA) {
    __builtin_amdgcn_global_load_lds((__attribute__((address_space(1))) const void*)src,
                                     (__attribute__((address_space(3))) void*)dst, 16, 0, NT ? 2 : 0);
  } else {
    const float2 a = src[0], b = src[1];
    dst[lane] = make_float4(a.x, a.y, b.x, b.y);
  }
}

template <int NB, int VPT, bool NT, bool DMA>
__global__ void __launch_bounds__(kQsoBlock) k_qso_draw(QsoDrawArgs a) {
  static_assert(VPT % 4 == 0 && 64 * VPT + kQsoFlush <= kQsoList && 64 * VPT * kQsoMaxTiles <= 65536, "list entries");
  __shared__ float snz[kQsoMaxNbar], snb[kQsoMaxNbar];
  __shared__ uint16_t slist[kQsoBlock / 64][kQsoList];
  __shared__ float4 sbox[kQsoBlock / 64][NB == 3 ? 2 : 1][64 * VPT / 2];
  const int lane = threadIdx.x & 63;
  uint16_t* list = slist[threadIdx.x >> 6];
  for (int i = threadIdx.x; i < a.n_nbar; i += kQsoBlock) {
    snz[i] = static_cast<float>(a.nbar_z[i]);
    snb[i] = static_cast<float>(a.nbar[i]);
  }
  float hv[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) hv[i] = 0.5f * static_cast<float>(*a.var[i]);
  __syncthreads();
  // the largest density, raised by a margin over the rounding of the
  // interpolation between two nodes
  float nb_top = 0.0f;
  for (int i = lane; i < a.n_nbar; i += 64) nb_top = fmaxf(nb_top, snb[i]);
#pragma unroll
  for (int w = 32; w >= 1; w >>= 1) nb_top = fmaxf(nb_top, __shfl_xor(nb_top, w));  // over the wave
  nb_top *= 1.0f + 1.0e-6f;

  const uint64_t wave = static_cast<uint64_t>(blockIdx.x) * (kQsoBlock / 64) + (threadIdx.x >> 6);
  const uint64_t w0 = wave * static_cast<uint64_t>(a.tiles) * (64 * VPT);   // the wave's first voxel
  // A tile comes through LDS, its loads issued while the one before is worked on:
  // lanes take neighbouring 16-byte pieces of the box there (a thread's own 64 bytes
  // would be four loads that each touch 64 cache lines), in an order that lets the
  // threads read theirs back without bank conflicts: piece h of thread l in slot
  // 4 l + (h ^ (l / 2 mod 4)).  A tile lies in one x plane (n^2 is a multiple of it).
  static_assert(VPT == 8, "four pieces per thread");
  const int swz = (lane >> 1) & 3;
  float4* sa = sbox[threadIdx.x >> 6][0];
  float4* sb = sbox[threadIdx.x >> 6][NB == 3 ? 1 : 0];
  const int mine = 8 * (lane >> 2) + 2 * ((lane & 3) ^ ((lane >> 3) & 3));
  const auto fetch = [&](int tile) {
    const uint64_t vt = w0 + static_cast<uint64_t>(tile) * (64 * VPT);
    const size_t et = static_cast<size_t>(vt) +
                      static_cast<size_t>(vt >> (2 * a.log2n)) * (a.pitch - static_cast<size_t>(a.n) * a.n) + mine;
#pragma unroll
    for (int i = 0; i < VPT / 2; ++i) {
      to_lds<NT, DMA>(a.box_a + et + 128 * i, sa + 64 * i, lane);
      if (NB == 3) to_lds<NT, DMA>(a.box_b + et + 128 * i, sb + 64 * i, lane);
    }
  };
  fetch(0);
  int cnt = 0;   // list entries (uniform)
  for (int tile = 0; tile < a.tiles; ++tile) {
    const uint32_t o0 = static_cast<uint32_t>((tile * 64 + lane) * VPT);
    const uint64_t v0 = w0 + o0;
    const QsoCell c(a, v0);
    const float r2xy = c.r2xy(a);
    const float2 ends = qso_ends<VPT>(a, r2xy, c.iz0);
    float d[NB][VPT];
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the tile is in LDS
#pragma unroll
    for (int h = 0; h < VPT / 2; ++h) {
      const int slot = lane * (VPT / 2) + (h ^ swz);
      const float4 v = sa[slot];
      d[0][2 * h] = v.x;
      d[0][2 * h + 1] = v.z;
      if (NB == 3) {
        const float4 w = sb[slot];
        d[1 % NB][2 * h] = v.y;
        d[1 % NB][2 * h + 1] = v.w;
        d[2 % NB][2 * h] = w.x;
        d[2 % NB][2 * h + 1] = w.z;
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (tile + 1 < a.tiles) fetch(tile + 1);
    const QsoBound<NB> b = qso_bound<NB>(a, ends, hv, nb_top);
    // decision words: voxel m takes word m & 3 of the call for counter m >> 2
    float u[VPT];
#pragma unroll
    for (int k = 0; k < VPT / 4; ++k) {
      const uint64_t ctr = (v0 >> 2) + k;
      const uint4 wd = philox10_x3(make_uint4(static_cast<uint32_t>(ctr), static_cast<uint32_t>(ctr >> 32), 2u, 0u),
                                   static_cast<uint32_t>(a.seed), static_cast<uint32_t>(a.seed >> 32));
      u[4 * k] = u01(wd.x);
      u[4 * k + 1] = u01(wd.y);
      u[4 * k + 2] = u01(wd.z);
      u[4 * k + 3] = u01(wd.w);
    }
    uint32_t left = 0;   // voxels that the bound does not reject
#pragma unroll
    for (int e = 0; e < VPT; ++e) {
      // a float's bits as a number: 2^23 (127 + log2 u) from below (at most 0.09 2^23)
      const float l2u = fmaf(static_cast<float>(__float_as_int(u[e])), 1.0f / 8388608.0f, -127.0f);
      bool reject = true;
#pragma unroll
      for (int i = 0; i < NB; ++i)
        reject = reject && l2u >= fmaxf(fmaf(b.lo[i], d[i][e], b.add[i]), fmaf(b.hi[i], d[i][e], b.add[i]));
      left |= reject ? 0u : 1u << e;
    }
    // one of each lane's at a time
    while (__any(left != 0u)) {
      const int e = __ffs(left) - 1;
      bool sel = false;
      if (left) {
        float de[NB], ue = u[0];
#pragma unroll
        for (int i = 0; i < NB; ++i) de[i] = d[i][0];
#pragma unroll
        for (int k = 1; k < VPT; ++k) {
          ue = e == k ? u[k] : ue;
#pragma unroll
          for (int i = 0; i < NB; ++i) de[i] = e == k ? d[i][k] : de[i];
        }
        sel = qso_selected<NB>(a, r2xy, c.iz0 + e, de, hv, nb_top, ue, snz, snb);
        left &= left - 1u;
      }
      const uint64_t m = __ballot(sel);
      if (sel) list[cnt + __popcll(m & ((1ull << lane) - 1ull))] = static_cast<uint16_t>(o0 + e);
      cnt += __popcll(m);
    }
    // (the list is read by other lanes than wrote it)
    if (cnt > kQsoFlush || (tile == a.tiles - 1 && cnt > 0)) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      unsigned long long base = 0;
      if (lane == 0) base = atomicAdd(a.count, static_cast<unsigned long long>(cnt));
      const uint32_t blo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(base));
      const uint32_t bhi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(base >> 32));
      base = (static_cast<unsigned long long>(bhi) << 32) | blo;
      for (int i = lane; i < cnt; i += 64) {
        const unsigned long long slot = base + i;
        if (slot >= static_cast<unsigned long long>(a.cap)) break;
        const uint64_t m = w0 + list[i];
        const QsoCell q(a, m);
        const uint4 pw = philox10_x3(make_uint4(static_cast<uint32_t>(m), static_cast<uint32_t>(m >> 32), 4u, 0u),
                                     static_cast<uint32_t>(a.seed), static_cast<uint32_t>(a.seed >> 32));
        int64_t* o = a.pos + 3 * slot;
        o[0] = (static_cast<int64_t>(q.ix) << 32) - (int64_t(1) << 31) + pw.x;
        o[1] = (static_cast<int64_t>(q.iy) << 32) - (int64_t(1) << 31) + pw.y;
        o[2] = (static_cast<int64_t>(q.iz0) << 32) - (int64_t(1) << 31) + pw.z;
      }
      cnt = 0;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
  }
}

hipError_t launch_qso_draw(const QsoCoef& c, const QsoDrawArgs& p, const float* ztab, float4* tab, hipStream_t st) {
  QsoDrawArgs a = p;
  for (int i = 0; i < 3; ++i) a.zb[i] = static_cast<float>(c.z[i]);
  LYA_TIMED("qso_coef", st,
            hipLaunchKernelGGL(k_qso_coef, dim3((kZTabN + 255) / 256), dim3(256), 0, st, ztab, c, tab,
                               a.count));
  // n^3 / (64 kQsoVpt) tiles, a power of two from 64 up (n >= 32): a wave takes as
  // many as leave the device about eight waves per SIMD, 64 at most, and every block
  // and wave is full
  const uint64_t all = static_cast<uint64_t>(a.n) * a.n * a.n / (64 * kQsoVpt);
  const uint64_t waves = static_cast<uint64_t>(device_cus()) * 32;
  a.tiles = 1;
  while (a.tiles < kQsoMaxTiles && all / (2 * a.tiles) >= waves) a.tiles *= 2;
  const uint64_t blocks = all / a.tiles / (kQsoBlock / 64);
  const bool nt = box_streams(a.n);
  const bool dma = (reinterpret_cast<uintptr_t>(a.box_a) | reinterpret_cast<uintptr_t>(a.box_b)) % 16 == 0;
  const auto kernel =
      a.nb == 3 ? (!dma ? k_qso_draw<3, kQsoVpt, false, false>
                   : nt ? k_qso_draw<3, kQsoVpt, true, true>
                        : k_qso_draw<3, kQsoVpt, false, true>)
                : (!dma ? k_qso_draw<1, kQsoVpt, false, false>
                   : nt ? k_qso_draw<1, kQsoVpt, true, true>
                        : k_qso_draw<1, kQsoVpt, false, true>);
  LYA_TIMED("qso_draw", st,
            hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(blocks)), dim3(kQsoBlock), 0, st, a));
  return hipGetLastError();
}

// ---- catalogue: redshift-space quasar redshifts and their lines of sight ----
// Flat LCDM in FP64.  I(a) = int_0^a da' / (a' E(a'))^3 by composite Simpson
// in t = sqrt(a') (a smooth integrand near 0), 512 intervals.
__device__ double growth_integral(double a, double om) {
  constexpr int kN = 512;
  const double tmax = sqrt(a), h = tmax / kN;
  double acc = 0.0;
  for (int i = 1; i <= kN; ++i) {
    const double t = h * i, ap = t * t;
    const double ae2 = om / ap + (1.0 - om) * ap * ap;  // (a E)^2
    acc += (i == kN ? 1.0 : (i & 1 ? 4.0 : 2.0)) * 2.0 * t / (ae2 * sqrt(ae2));
  }
  return acc * h / 3.0;
}

// chi(z) = c/H0 int_0^z dz' / E(z'), composite Simpson with 1024 intervals.
__device__ double chi_of_z_fine(double z, double om) {
  constexpr int kN = 1024;
  const double h = z / kN;
  double acc = 0.0;
  for (int i = 0; i <= kN; ++i) {
    const double x = 1.0 + h * i;
    acc += (i == 0 || i == kN ? 1.0 : (i & 1 ? 4.0 : 2.0)) / sqrt(om * x * x * x + (1.0 - om));
  }
  return kCOverH0 * acc * h / 3.0;
}

// Velocity factor G(z) f(z) E(z) / (1 + z) at chi = i kZTabH (z from ztab):
// the velocity boxes (z = 0, f = 1) to redshift z.  f = dln D / dln a =
// -3 Om / (2 a^3 E^2) + a / (I (a E)^3) for D = E I.
__global__ void __launch_bounds__(256) k_qso_vtab(const float* __restrict__ ztab, double om, float* __restrict__ vtab) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= kZTabN) return;
  const double z = ztab[i];
  const double a = 1.0 / (1.0 + z);
  const double e2 = om / (a * a * a) + 1.0 - om;
  const double I = growth_integral(a, om), I1 = growth_integral(1.0, om);
  const double g = sqrt(e2) * I / I1;
  const double ae2 = a * a * e2;
  const double f = -1.5 * om / (a * a * a * e2) + a / (I * ae2 * sqrt(ae2));
  vtab[i] = static_cast<float>(g * f * sqrt(e2) / (1.0 + z));
}

__device__ __forceinline__ double lerp_tab(const float* tab, double chi) {
  const double t = chi / kZTabH;
  const int i0 = min(static_cast<int>(t), kZTabN - 2);
  const double fr = t - i0;
  return tab[i0] + fr * (static_cast<double>(tab[i0 + 1]) - tab[i0]);
}

// One thread per quasar.
__global__ void __launch_bounds__(256) k_qso_los(QsoLosArgs a) {
  constexpr double kTwo32 = 4294967296.0;
  constexpr double kCKms = 299792.458;
  for (int64_t q = blockIdx.x * 256ll + threadIdx.x; q < a.n_q; q += static_cast<int64_t>(gridDim.x) * 256) {
    const int64_t p[3] = {a.pos[3 * q], a.pos[3 * q + 1], a.pos[3 * q + 2]};
    double d[3], chi2 = 0.0;
    for (int ax = 0; ax < 3; ++ax) {
      d[ax] = static_cast<double>(p[ax]) / kTwo32 * a.dx - a.o[ax];
      chi2 += d[ax] * d[ax];
    }
    const double chi = sqrt(chi2);
    double u[3] = {d[0] / chi, d[1] / chi, d[2] / chi};
    // z(chi): the table's value refined by Newton steps on chi(z) (FP64)
    double zc = lerp_tab(a.ztab, chi);
    for (int it = 0; it < 3; ++it) {
      const double x = 1.0 + zc;
      zc -= (chi_of_z_fine(zc, a.om) - chi) * sqrt(a.om * x * x * x + 1.0 - a.om) / kCOverH0;
    }
    double vpar = 0.0;
    if (a.vxy) {
      // periodic trilinear of {v_x, v_y} and v_z at the quasar
      int c0[3], c1[3];
      double w1[3];
      for (int ax = 0; ax < 3; ++ax) {
        const int64_t cell = p[ax] >> 32;
        c0[ax] = static_cast<int>(((cell % a.n) + a.n) % a.n);
        c1[ax] = c0[ax] + 1 == a.n ? 0 : c0[ax] + 1;
        w1[ax] = static_cast<double>(p[ax] & 0xffffffffll) / kTwo32;
      }
      double v[3] = {0.0, 0.0, 0.0};
      for (int cx = 0; cx < 2; ++cx)
        for (int cy = 0; cy < 2; ++cy)
          for (int cz = 0; cz < 2; ++cz) {
            const double w = (cx ? w1[0] : 1.0 - w1[0]) * (cy ? w1[1] : 1.0 - w1[1]) * (cz ? w1[2] : 1.0 - w1[2]);
            const size_t e = static_cast<size_t>(cx ? c1[0] : c0[0]) * a.pitch +
                             static_cast<size_t>(cy ? c1[1] : c0[1]) * a.n + (cz ? c1[2] : c0[2]);
            const float2 xy = a.vxy[e];
            v[0] += w * xy.x;
            v[1] += w * xy.y;
            v[2] += w * a.vz[e].x;
          }
      vpar = (v[0] * u[0] + v[1] * u[1] + v[2] * u[2]) * lerp_tab(a.vtab, chi);
    }
    const double zq = zc + (1.0 + zc) * vpar / kCKms;
    const double z_hi = (1.0 + zq) * a.r_hi - 1.0;
    const double z_lo = fmax((1.0 + zq) * a.r_lo - 1.0, a.z_min);
    const double c_hi = chi_of_z_fine(z_hi, a.om);
    int np = 0;
    if (z_hi > z_lo) np = static_cast<int>(fmin(floor((c_hi - chi_of_z_fine(z_lo, a.om)) / a.dchi), 2048.0));
    a.z_q[q] = zq;
    a.chi0[q] = c_hi;
    a.npix[q] = np;
    for (int ax = 0; ax < 3; ++ax) {
      a.origin[3 * q + ax] = llrint((a.o[ax] + u[ax] * c_hi) / a.dx * kTwo32);
      a.step[3 * q + ax] = llrint(-u[ax] * a.dchi / a.dx * kTwo32);
    }
  }
}

// Exclusive prefix sum of npix into offset, and the total (one block).
__global__ void __launch_bounds__(1024) k_qso_offsets(const int32_t* __restrict__ npix, int64_t n_q,
                                                      int64_t* __restrict__ offset, int64_t* __restrict__ total) {
  __shared__ int wsum[16];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  long long run = 0;
  for (int64_t base = 0; base < n_q; base += 1024) {
    const int64_t i = base + threadIdx.x;
    const int v = i < n_q ? npix[i] : 0;
    int x = v;  // inclusive scan in the wave (a chunk sums to at most 2^21)
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(x, o, 64);
      if (lane >= o) x += y;
    }
    if (lane == 63) wsum[wv] = x;
    __syncthreads();
    int before = 0, chunk = 0;
    for (int k = 0; k < 16; ++k) {
      if (k < wv) before += wsum[k];
      chunk += wsum[k];
    }
    if (i < n_q) offset[i] = run + before + x - v;
    run += chunk;
    __syncthreads();
  }
  if (threadIdx.x == 0) *total = run;
}

hipError_t launch_qso_los(const QsoLosArgs& a, float* ztab_w, float* vtab_w, hipStream_t st) {
  hipError_t e = launch_zchi_table(a.om, ztab_w, st);
  if (e != hipSuccess) return e;
  LYA_TIMED("qso_vtab", st, hipLaunchKernelGGL(k_qso_vtab, dim3((kZTabN + 255) / 256), dim3(256), 0, st, ztab_w,
                                               a.om, vtab_w));
  if (a.n_q > 0) {
    const int64_t blocks = std::min<int64_t>((a.n_q + 255) / 256, static_cast<int64_t>(device_cus()) * 16);
    LYA_TIMED("qso_los", st, hipLaunchKernelGGL(k_qso_los, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, a));
  }
  LYA_TIMED("qso_offsets", st,
            hipLaunchKernelGGL(k_qso_offsets, dim3(1), dim3(1024), 0, st, a.npix, a.n_q, a.offset, a.total));
  return hipGetLastError();
}

}  // namespace lya
