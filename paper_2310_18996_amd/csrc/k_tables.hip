// FP64 tables for the hot path (gfx950): the power-spectrum amplitude per
// integer n^2, the sigma8 normalisation, FFT twiddles, and z(chi) for pixel
// redshifts.  FP64 on the GPU is confined to these small tables.
//
// P(k) (stand-in for the paper's CAMB spectrum, eq:deltaL):
//   P = A k^ns T_BBKS(k/Gamma)^2 (1 + w sin(k r_w) exp(-(k/k_d)^2)),
//   T_BBKS(q) = ln(1+2.34q)/(2.34q) [1+3.89q+(16.1q)^2+(5.46q)^3+(6.71q)^4]^(-1/4)
//   (Bardeen, Bond, Kaiser & Szalay 1986);
//   A from sigma8: sigma_8^2 = 1/(2 pi^2) int k^3 P W_TH(8k)^2 dln k with the
//   sphere window W_TH(x) = 3 (sin x - x cos x)/x^3, composite Simpson in
//   ln k over [1e-5, 1e3] h/Mpc with 2^16+1 nodes.
// A tabulated P(k) (the paper's CAMB table) replaces the analytic form and its
// sigma8 normalisation when given.
// Amplitude per mode (eq:deltaL with unit-variance complex noise):
//   s(n^2) = sqrt(P(2 pi |n| / L) / L^3) * exp(-k^2 smooth^2 / 2), s(0) = 0.
// Pixel redshift (section "FGPA": unperturbed cosmological redshift), flat
// LCDM with E(z)^2 = Om (1+z)^3 + 1 - Om (Table cosmoparams), c/H0 in Mpc/h.
#include "lya_internal.h"
#include "lya_wavefft.h"

namespace lya {

__device__ __forceinline__ double t_bbks(double q) {
  const double x = 2.34 * q;
  const double lead = x > 0.0 ? log1p(x) / x : 1.0;
  const double a = 16.1 * q, b = 5.46 * q, c = 6.71 * q;
  const double poly = 1.0 + 3.89 * q + a * a + b * b * b + (c * c) * (c * c);
  return lead * pow(poly, -0.25);
}

__device__ __forceinline__ double pk_shape(double k, const PkParams& p) {
  const double t = t_bbks(k / p.gamma);
  const double kd = k / p.wig_kd;
  const double wig = 1.0 + p.wig_amp * sin(k * p.wig_r) * exp(-kd * kd);
  return pow(k, p.ns) * t * t * wig;
}

__device__ __forceinline__ double w_tophat(double x) {
  if (fabs(x) < 1e-2) {
    const double x2 = x * x;
    return 1.0 - x2 / 10.0 + x2 * x2 / 280.0;
  }
  return 3.0 * (sin(x) - x * cos(x)) / (x * x * x);
}

constexpr int kSimpsonNodes = 65537;
constexpr double kLnkMin = -11.512925464970229;  // ln 1e-5
constexpr double kLnkMax = 6.907755278982137;    // ln 1e3

// First launch of a table: the sigma8 integral's partial sums (kSigmaBlocks blocks,
// one node per thread and the last node with the first block: the nodes' FP64
// exp, pow, sin and log are the launch's time, 12.7 us at four nodes per thread,
// 5 at one), then ntw twiddles exp(+2 pi i k / ntw).  What reads the table's
// amplitude adds the partial sums itself (pk_amplitude); a launch of one block for
// that cost 5 us.
__global__ void __launch_bounds__(kSigmaBlocks) k_pk_start(PkParams p, int nsig, double* partial, float2* tw, int ntw) {
  __shared__ double red[kSigmaBlocks];
  if (static_cast<int>(blockIdx.x) >= nsig) {
    const int k = (blockIdx.x - nsig) * kSigmaBlocks + threadIdx.x;
    if (k >= ntw) return;
    double sn, cs;
    sincospi(2.0 * k / ntw, &sn, &cs);
    tw[k] = make_float2(static_cast<float>(cs), static_cast<float>(sn));
    return;
  }
  const double h = (kLnkMax - kLnkMin) / (kSimpsonNodes - 1);
  double acc = 0.0;
  for (int i = blockIdx.x * kSigmaBlocks + threadIdx.x; i < kSimpsonNodes; i += kSigmaBlocks * kSigmaBlocks) {
    const double lnk = kLnkMin + h * i;
    const double k = exp(lnk);
    const double w = w_tophat(8.0 * k);
    const double wt = (i == 0 || i == kSimpsonNodes - 1) ? 1.0 : ((i & 1) ? 4.0 : 2.0);
    acc += wt * k * k * k * pk_shape(k, p) * w * w;
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = kSigmaBlocks / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// Amplitude A of the analytic form from the partial sums, by a block of
// kSigmaBlocks threads in a fixed order (the same in every block).
__device__ __forceinline__ double pk_amplitude(const PkParams& p, const double* __restrict__ partial) {
  __shared__ double red[kSigmaBlocks / 64];
  double s = partial[threadIdx.x];
#pragma unroll
  for (int w = 32; w >= 1; w >>= 1) s += __shfl_xor(s, w);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  s = 0.0;
#pragma unroll
  for (int w = 0; w < kSigmaBlocks / 64; ++w) s += red[w];
  const double h = (kLnkMax - kLnkMin) / (kSimpsonNodes - 1);
  const double sig2 = h / 3.0 * s / (2.0 * M_PI * M_PI);
  return p.sigma8 * p.sigma8 / sig2;
}

// Tabulated P(k): ln P linear in ln k between the nodes; below the first and
// above the last node the end intervals' power laws continue.
__device__ __forceinline__ double pk_tabulated(double k, const PkParams& p) {
  const double* kt = p.k_tab;
  const int n = p.n_tab;
  int i;   // interval [kt[i], kt[i+1]]
  if (k <= kt[0]) {
    i = 0;
  } else if (k >= kt[n - 1]) {
    i = n - 2;
  } else {
    int lo = 0, hi = n - 1;   // kt[lo] <= k < kt[hi]
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (kt[mid] <= k) lo = mid; else hi = mid;
    }
    i = lo;
  }
  const double x0 = log(kt[i]), x1 = log(kt[i + 1]);
  const double y0 = log(p.p_tab[i]), y1 = log(p.p_tab[i + 1]);
  return exp(y0 + (y1 - y0) * (log(k) - x0) / (x1 - x0));
}

__global__ void __launch_bounds__(kSigmaBlocks) k_amp_table(const double* __restrict__ partial, PkParams p, double L,
                                                            int nentries, float* table) {
  const double amp = p.k_tab ? 1.0 : pk_amplitude(p, partial);
  const int e = blockIdx.x * kSigmaBlocks + threadIdx.x;
  if (e >= nentries) return;
  if (e == 0) {
    table[0] = 0.0f;
    return;
  }
  const double k = 2.0 * M_PI * sqrt(static_cast<double>(e)) / L;
  const double P = p.k_tab ? pk_tabulated(k, p) : amp * pk_shape(k, p);
  double s = sqrt(P / (L * L * L));
  if (p.smooth > 0.0) s *= exp(-0.5 * (k * p.smooth) * (k * p.smooth));
  table[e] = static_cast<float>(s);
}

// Integrand of the matter correlation function of the smoothed spectrum
// (section "Quasar generation"): xi(r) = 1/(2 pi^2 r) int_0^kmax P(k)
// exp(-k^2 s^2) k sin(k r) dk, composite Simpson on k_j = j h, j = 0..m
// (m even).  f_j is the Simpson weight times P(k_j) exp(-k_j^2 s^2) k_j (k = 0
// carries nothing), written as the sums and differences of the node pairs that
// k_sine_sum takes (nodes beyond m are 0).
__global__ void __launch_bounds__(kSigmaBlocks) k_xi_weights(const double* __restrict__ partial, PkParams p, double s,
                                                             double h, int m, int na, double* sd) {
  const double amp = p.k_tab ? 1.0 : pk_amplitude(p, partial);
  const int t = blockIdx.x * kSigmaBlocks + threadIdx.x;
  const int a = t / kSineB, b = t % kSineB;
  if (a >= na) return;
  auto f = [&](int j) {
    if (j == 0 || j > m) return 0.0;
    const double k = h * j;
    const double P = p.k_tab ? pk_tabulated(k, p) : amp * pk_shape(k, p);
    const double w = (j == m) ? 1.0 : ((j & 1) ? 4.0 : 2.0);
    return w * h / 3.0 * P * exp(-(k * s) * (k * s)) * k;
  };
  const double fp = f(a * kSineJ + kSineB + b), fm = f(a * kSineJ + kSineB - 1 - b);
  sd[static_cast<size_t>(a) * kSineJ + b] = fp + fm;
  sd[static_cast<size_t>(a) * kSineJ + kSineB + b] = fp - fm;
}

// ---- pixel redshift table: z at chi = i * kZTabH ----
__device__ __forceinline__ double inv_e(double z, double om) {
  const double zp = 1.0 + z;
  return rsqrt(om * zp * zp * zp + (1.0 - om));
}

// Sum over the 16 lanes of a group (one DPP row), the same bits in every
// lane, so that the lanes take the same branches: the empty asm keeps the
// compiler from fusing v's last product into a lane's own first addition.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const uint64_t u = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(u), CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(u >> 32), CTRL, 0xf, 0xf, false);
  return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<uint32_t>(lo));
}
__device__ __forceinline__ double group_sum(double v) {
  asm volatile("" : "+v"(v));
  v += dpp_f64<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  v += dpp_f64<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  v += dpp_f64<0x141>(v);  // row_half_mirror
  v += dpp_f64<0x140>(v);  // row_mirror
  return v;
}

// chi(z) by composite Simpson, 128 intervals on [0, z] (relative error ~1e-9
// for z < 5), the nodes dealt out over a group of 16 lanes: lane l takes the
// nodes l + 1 + 16 t, all of one parity (lane 15's last one is the end node).
__device__ __forceinline__ double chi_of_z_group(double z, double om, int l) {
  constexpr int m = 128;
  const double h = z / m, w = (l & 1) ? 2.0 : 4.0;
  double s = 0.0;
#pragma unroll
  for (int t = 0; t < m / 16; ++t) {
    const int i = l + 1 + 16 * t;
    s += (i == m ? 1.0 : w) * inv_e(h * i, om);
  }
  return kCOverH0 * h / 3.0 * (group_sum(s) + inv_e(0.0, om));
}

// Positive nodes and weights of the 16-point Gauss-Legendre rule on [-1, 1].
__constant__ double kGlX[8] = {0.09501250983763744, 0.2816035507792589,  0.45801677765722737, 0.6178762444026438,
                               0.755404408355003,   0.8656312023878318,  0.9445750230732326,  0.9894009349916499};
__constant__ double kGlW[8] = {0.1894506104550685,  0.18260341504492358, 0.16915651939500254, 0.14959598881657674,
                               0.12462897125553388, 0.09515851168249279, 0.062253523938647894, 0.027152459411754096};

// z(chi) by Newton on the Simpson chi(z), from z = chi H0/c, until a step is
// below 1e-11 (at most 20 steps), by a group of 16 lanes per node.  A thread
// per node with 129 square roots and divisions in each of its 5-20 steps was
// one serial chain of 0.23 ms on 79 blocks, whatever the size of the call.
// Split over 16 lanes, and with the first steps taken on the 16-point
// Gauss-Legendre chi(z) (one node per lane: it agrees with the Simpson rule
// to ~1e-9 for z < 5, so one or two Simpson steps remain), the table takes
// 0.018 ms.  Where the quick start has not settled below z = 60, or the
// Simpson steps from it do not (towards and beyond the horizon, where no z has
// that distance), the steps start again from z = chi H0/c; a NaN stays one.
__device__ __forceinline__ double z_of_chi_group(double chi, double om, int l) {
  const double x0 = (l & 1) ? kGlX[l >> 1] : -kGlX[l >> 1], w0 = kGlW[l >> 1];
  auto slope = [om](double z) { return sqrt(om * (1 + z) * (1 + z) * (1 + z) + 1 - om) / kCOverH0; };
  double z = chi / kCOverH0;
  bool quick = false;
  for (int it = 0; it < 10 && !quick && z < 60.0; ++it) {
    const double half = 0.5 * z;
    const double dz = (kCOverH0 * half * group_sum(w0 * inv_e(half * (x0 + 1.0), om)) - chi) * slope(z);
    z -= dz;
    quick = fabs(dz) < 1e-6;
  }
  quick = quick && z >= 0.0 && z < 60.0;
  for (int start = quick ? 0 : 1; start < 2; ++start) {
    if (start == 1) z = chi / kCOverH0;
    const int most = start == 0 ? 6 : 20;
    for (int it = 0; it < most; ++it) {
      const double dz = (chi_of_z_group(z, om, l) - chi) * slope(z);
      z -= dz;
      if (fabs(dz) < 1e-11 || z != z) return z;
    }
  }
  return z;
}

// What a call needs before its main kernel, in one launch (each of these was
// a launch of 4-5 us of its own): the z(chi) table (ztab), the 2048 twiddles
// (tw), the amplitudes of delta_S (ps_tab: in the line kernel a tabulated ratio took
// an FP64 search of dependent loads for each mode of each line; FGPA and 1D power of
// 35M stored pixels 630 -> 523 us), the first modes of the k bins (modes), and the work
// queue and bin sums cleared (queue, bsum, bcnt; ordinary stores, no memset node).  Null pointers are left out.  The table's
// blocks come first and in decreasing chi (the far nodes take the most steps).
constexpr int kPrepNT = 256;
constexpr int kPrepZBlocks = (kZTabN * 16 + kPrepNT - 1) / kPrepNT;
constexpr int kPrepTwBlocks = kTw2048 / kPrepNT;
constexpr int kPrepPsBlocks = (kPsTab + kPrepNT - 1) / kPrepNT;

__global__ void __launch_bounds__(kPrepNT) k_prep(PrepArgs a) {
  const int nz = a.ztab ? kPrepZBlocks : 0, nt = a.tw ? kPrepTwBlocks : 0;
  int b = blockIdx.x;
  const int t = threadIdx.x;
  if (b < nz) {
    // the lanes of a group share their node, so a group leaves as a whole
    const int i = kZTabN - 1 - (b * (kPrepNT / 16) + (t >> 4));
    if (i < 0) return;
    const double z = z_of_chi_group(kZTabH * i, a.omega_m, t & 15);
    if ((t & 15) == 0) a.ztab[i] = static_cast<float>(z);
    return;
  }
  b -= nz;
  if (b < nt) {
    const int k = b * kPrepNT + t;
    double sn, cs;
    sincospi(2.0 * k / kTw2048, &sn, &cs);
    a.tw[k] = make_float2(static_cast<float>(cs), static_cast<float>(sn));
    return;
  }
  b -= nt;
  if (b < (a.ps_tab ? kPrepPsBlocks : 0)) {
    const int i = b * kPrepNT + t;
    if (i >= kPsTab) return;
    const int ns = i < 2 ? 2 : 1 << (31 - __clz(i)), m = i - ns;   // (entries past ns/2 are not used)
    const float2 sc = ps_scales(a.ps_amp, a.ps_kcut, a.dpix, ns);
    a.ps_tab[i] = m > 0 ? ps_amplitude(a, m, ns, sc.x, sc.y) : 0.0f;
    return;
  }
  b -= a.ps_tab ? kPrepPsBlocks : 0;
  if (a.modes && b < kModeBlocks) {
    mode_table(a.modes, a.k_edges, a.nk, a.dv, b, t, kPrepNT);
    return;
  }
  if (t < kPullCounters && a.queue) a.queue[t * kPullStride] = 0u;
  for (int i = t; i < kBinCopies * kMaxZBins && a.bsum; i += kPrepNT) {
    a.bsum[i] = 0ull;
    a.bcnt[i] = 0ull;
  }
}

hipError_t launch_prep(const PrepArgs& a, hipStream_t st) {
  const int blocks = (a.ztab ? kPrepZBlocks : 0) + (a.tw ? kPrepTwBlocks : 0) +
                     (a.ps_tab ? kPrepPsBlocks : 0) + (a.modes ? kModeBlocks : 0) + (a.queue || a.bsum ? 1 : 0);
  if (blocks == 0) return hipSuccess;
  LYA_TIMED("prep", st, hipLaunchKernelGGL(k_prep, dim3(blocks), dim3(kPrepNT), 0, st, a));
  return hipGetLastError();
}

// ---- launchers ----
// sigma8 sums (none for a tabulated spectrum) and twiddles (ntw may be 0)
void launch_pk_start(const PkParams& p, double* partial, float2* tw, int ntw, hipStream_t st) {
  const int nsig = p.k_tab ? 0 : kSigmaBlocks, nt = (ntw + kSigmaBlocks - 1) / kSigmaBlocks;
  if (nsig + nt > 0)
    LYA_TIMED("pk_start", st,
              hipLaunchKernelGGL(k_pk_start, dim3(nsig + nt), dim3(kSigmaBlocks), 0, st, p, nsig, partial, tw, ntw));
}

hipError_t launch_pk_table(const PkParams& p, int n, double dx, TableWork& w, hipStream_t st) {
  const double L = n * dx;
  launch_pk_start(p, w.partial, w.tw, n, st);
  const int ne = amp_table_entries(n);
  LYA_TIMED("pk_table", st,
            hipLaunchKernelGGL(k_amp_table, dim3((ne + kSigmaBlocks - 1) / kSigmaBlocks), dim3(kSigmaBlocks), 0, st,
                               w.partial, p, L, ne, w.table));
  return hipGetLastError();
}

hipError_t launch_xi_weights(const PkParams& p, double s, double h, int m, double* partial, double* f,
                             hipStream_t st) {
  launch_pk_start(p, partial, nullptr, 0, st);
  const int na = sine_shape(m + 1, 1).na;
  LYA_TIMED("xi_weights", st,
            hipLaunchKernelGGL(k_xi_weights, dim3((na * kSineB + kSigmaBlocks - 1) / kSigmaBlocks),
                               dim3(kSigmaBlocks), 0, st, partial, p, s, h, m, na,
                               f));
  return hipGetLastError();
}

hipError_t launch_zchi_table(double omega_m, float* ztab, hipStream_t st) {
  PrepArgs a{};
  a.omega_m = omega_m;
  a.ztab = ztab;
  return launch_prep(a, st);
}

__global__ void __launch_bounds__(256) k_twiddles(float2* tw, int ntw) {
  for (int k = blockIdx.x * 256 + threadIdx.x; k < ntw; k += gridDim.x * 256) {
    double sn, cs;
    sincospi(2.0 * k / ntw, &sn, &cs);
    tw[k] = make_float2(static_cast<float>(cs), static_cast<float>(sn));
  }
}

hipError_t launch_twiddles(float2* tw, int ntw, hipStream_t st) {
  LYA_TIMED("twiddles", st, hipLaunchKernelGGL(k_twiddles, dim3((ntw + 255) / 256), dim3(256), 0, st, tw, ntw));
  return hipGetLastError();
}

}  // namespace lya
