// Per-line helpers shared by the skewer and 1D-power kernels: pixel distances,
// distance-bin boundaries, and a wavefront-level FFT in LDS (one wavefront owns
// a line of up to kHalfMax complex values in its slice of LDS and transforms it
// in place, without block barriers).
#pragma once

#include "lya_internal.h"

namespace lya {

constexpr int kHalfMax = 1024;                        // complex length <= 1024
constexpr int kHalfBuf = kHalfMax + kHalfMax / 16 - 1;   // a padding slot after every 16 but the last

__device__ __forceinline__ int pidx(int i) { return i + (i >> 4); }   // pidx(a + b) = pidx(a) + pidx(b) if a & b == 0

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Comoving distance of pixel j: chi0 - (j * dchi), each operation rounded in
// FP64 (no fused multiply-add), as the C-ABI defines it.
__device__ __forceinline__ double pixel_chi(double chi0, int j, double dchi) {
  return __dsub_rn(chi0, __dmul_rn(static_cast<double>(j), dchi));
}

// First pixel j in [0, np] with chi_j < edge (chi_j decreases with j); exact
// FP64 comparisons.
__device__ __forceinline__ int first_below(double edge, double chi0, double dchi, int np) {
  double j0 = dchi > 0.0 ? ceil((chi0 - edge) / dchi) : 0.0;
  j0 = j0 < 0.0 ? 0.0 : (j0 > np ? np : j0);
  int j = static_cast<int>(j0);
  while (j < np && pixel_chi(chi0, j, dchi) >= edge) ++j;
  while (j > 0 && pixel_chi(chi0, j - 1, dchi) < edge) --j;
  return j;
}

// jb[b] = first_below of edges[b], for b = 0..n_bins, so pixel j lies in
// distance bin b exactly when jb[b+1] <= j < jb[b].  Lanes split the edges.
__device__ __forceinline__ void bin_bounds(const double* __restrict__ edges, int n_bins, double chi0, double dchi,
                                           int np, int* jb, int lane) {
  for (int b = lane; b <= n_bins; b += 64) jb[b] = first_below(edges[b], chi0, dchi, np);
}

// The block's copy of the twiddle table tw2048 in LDS (read by every stage of
// every wavefront FFT; global reads would put an L2 round trip in each stage).
// Padded so that the stages' strides (8, 32, 128 and their multiples) spread over
// the banks: without it they met in one or two of them, half of all LDS cycles of
// a line (8 draws on 20,000 lines 326 -> 279 us).
__host__ __device__ constexpr int tidx(int i) { return i + (i >> 3) + (i >> 5); }
struct LdsTw {
  const float2* p;
  __device__ __forceinline__ float2 operator[](int i) const { return p[tidx(i)]; }
};
// N: 3/4 of the table is all that radix-4 stages and half-length spectra read.
template <int N = kTw2048>
__device__ __forceinline__ void load_twiddles(float2* stw, const float2* __restrict__ tw2048, int tid, int nt) {
  for (int i = tid; i < N; i += nt) stw[tidx(i)] = tw2048[i];
}
// entry n STEP of the table: one multiplication where the padding is linear in n
template <int STEP, class TW>
__device__ __forceinline__ float2 tw_at(TW tw, int n) { return tw[n * STEP]; }
template <int STEP>
__device__ __forceinline__ float2 tw_at(LdsTw tw, int n) {
  if constexpr (STEP % 32 == 0) return tw.p[n * tidx(STEP)];
  else return tw[n * STEP];
}

// First mode m >= 1 of a line of n_p pixels with k_m = 2 pi m / (n_p dv) >= edge
// (M + 1 if none, M = n_p / 2), decided in FP64.
__device__ __forceinline__ int first_mode(double edge, int n_p, double dv) {
  const int M = n_p / 2;
  const double kf = 2.0 * M_PI / (n_p * dv);
  double m0 = ceil(edge / kf);
  m0 = m0 < 1.0 ? 1.0 : (m0 > M + 1.0 ? M + 1.0 : m0);
  int m = static_cast<int>(m0);
  while (m <= M && (2.0 * M_PI * m) / (n_p * dv) < edge) ++m;
  while (m > 1 && (2.0 * M_PI * (m - 1)) / (n_p * dv) >= edge) --m;
  return m;
}

// Lines are transformed at the lengths 2^1 .. 2^11 only, so the first modes of
// the k bins are a table per length class (log2 of the length) and not an FP64
// search per line: row c holds the nk + 1 edges' first modes, then the smallest
// and the largest of them (the modes any bin wants).
constexpr int kLenClasses = 12;  // class 0: no transform
__device__ __forceinline__ int len_class(int np) {
  return np >= 2 ? 31 - __clz(np < 2 * kHalfMax ? np : 2 * kHalfMax) : 0;
}
__host__ __device__ constexpr int mode_row(int nk) { return nk + 3; }
// Part b of kModeBlocks, by a block of nt threads, into out; once per call, in the
// launch before the lines' (its FP64 divisions in every block of those were 3 us of
// each, and as one part 2 us more of that launch at 64 bins).
constexpr int kModeBlocks = 4;
template <typename T>
__device__ __forceinline__ void mode_table(T* __restrict__ out, const double* __restrict__ k_edges, int nk, double dv,
                                           int part, int tid, int nt) {
  constexpr int nc = kLenClasses / kModeBlocks;
  static_assert(kLenClasses % kModeBlocks == 0, "whole rows per part");
  __shared__ int lo[nc], hi[nc];
  const int row = mode_row(nk), c0 = part * nc;
  if (tid < nc) {
    lo[tid] = kHalfMax + 1;
    hi[tid] = 0;
  }
  __syncthreads();
  for (int i = tid; i < nc * (nk + 1); i += nt) {
    const int c = i / (nk + 1), b = i % (nk + 1), m = c0 + c > 0 ? first_mode(k_edges[b], 1 << (c0 + c), dv) : 1;
    out[(c0 + c) * row + b] = static_cast<T>(m);
    atomicMin(&lo[c], m);   // (one thread per row over the finished row took longer than the modes)
    atomicMax(&hi[c], m);
  }
  __syncthreads();
  if (tid < nc) {
    out[(c0 + tid) * row + nk + 1] = static_cast<T>(lo[tid]);
    out[(c0 + tid) * row + nk + 2] = static_cast<T>(hi[tid]);
  }
}

// |X_m|^2 scale of a transformed line for the modes lo <= m < hi (1 <= m <= M),
// from the transform Z of its pixel pairs in buf, left in the real part of
// slot m mod M: X_m = (Z_m + conj Z_{M-m})/2 + w^m (Z_m - conj Z_{M-m})/(2i).  A
// lane takes m and M - m, which read the same two values, so the powers can
// take their place without a second buffer.
__device__ __forceinline__ float line_power(float2 zm, float2 zc, float2 w, float scale) {
  const float2 E = make_float2(0.5f * (zm.x + zc.x), 0.5f * (zm.y - zc.y));
  const float2 O = make_float2(0.5f * (zm.y + zc.y), -0.5f * (zm.x - zc.x));
  const float2 X = cadd(E, cmul(w, O));
  return scale * (X.x * X.x + X.y * X.y);
}
template <class TW>
__device__ __forceinline__ void power_in_place(float2* buf, int M, int lo, int hi, float scale, TW tw, int lane) {
  const int twstep = kTw2048 / (2 * M);
  // pairs (m, M - m), 0 <= m <= M/2, of which one lies in [lo, hi); the pair
  // (0, M) stands for mode M alone
  const int first = hi > M / 2 ? min(lo, M - hi + 1) : lo, last = min(hi - 1, M / 2);
  const int end = lo > M / 2 ? M - lo : (hi > M / 2 ? M / 2 : last);
  for (int m = (first > 0 ? first : 0) + lane; m <= end; m += 64) {
    const float2 zm = buf[pidx(m)], zc = buf[pidx(m == 0 ? 0 : M - m)];
    if (m == 0) {
      if (M >= lo && M < hi) buf[pidx(0)].x = line_power(zm, zm, tw[M * twstep], scale);
      continue;
    }
    const int c = M - m;
    if (m >= lo && m < hi) buf[pidx(m)].x = line_power(zm, zc, tw[m * twstep], scale);
    if (c != m && c >= lo && c < hi) buf[pidx(c)].x = line_power(zc, zm, tw[c * twstep], scale);
  }
}

// FP64 sums of the powers power_in_place left, per k bin (first modes m0 <= m <
// m1 of the lane's bin): 64 >> lg lanes bins, each by 2^lg lanes taking every
// 2^lg-th mode, added in a fixed tree.
__device__ __forceinline__ double bin_sum(const float2* buf, int M, int m0, int m1, int lg, int lane) {
  double s = 0.0;
#pragma unroll 4
  for (int m = m0 + (lane & ((1 << lg) - 1)); m < m1; m += 1 << lg) s += buf[pidx(m == M ? 0 : m)].x;
  for (int w = 0; w < lg; ++w) s += __shfl_xor(s, 1 << w);
  return s;
}
__device__ __forceinline__ int bin_split(int nk) { return nk <= 8 ? 3 : nk <= 16 ? 2 : nk <= 32 ? 1 : 0; }

// Value of a lane, the lane uniform, as a scalar.
__device__ __forceinline__ int lane_i32(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ __forceinline__ int64_t lane_i64(int64_t v, int l) {
  const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(v), l);
  const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(v >> 32), l);
  return static_cast<int64_t>((static_cast<uint64_t>(hi) << 32) | lo);
}
__device__ __forceinline__ double lane_f64(double v, int l) {
  return __longlong_as_double(lane_i64(__double_as_longlong(v), l));
}

// Unnormalised inverse DFT (exp(+2 pi i k n / M)) of buf[pidx(0..M-1)], M =
// 2^LG <= kHalfMax, by an in-place Stockham radix-4/2 FFT: every stage first
// reads all of the lane's inputs, then writes (the wave runs in lockstep).
// tw2048[k] = exp(2 pi i k / 2048).
template <int LG, int LS = 0, class TW>
__device__ __forceinline__ void wave_ifft_n(float2* buf, TW tw2048, int lane) {
  if constexpr (LS < LG) {
    constexpr int LR = LG - LS >= 2 ? 2 : 1, R = 1 << LR, s = 1 << LS, nb = 1 << (LG - LR);
    constexpr int T = nb > 64 ? nb / 64 : 1, step = kTw2048 >> (LS + LR);
    float2 v[T][R];
    asm volatile("" : "+v"(lane));   // no stage's addresses are computed ahead of it and kept
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int j = lane + 64 * t;
      if (nb >= 64 || j < nb) {
#pragma unroll
        for (int r = 0; r < R; ++r) v[t][r] = buf[pidx(j) + pidx(r * nb)];
      }
    }
    wave_sync();
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int j = lane + 64 * t;
      if (nb >= 64 || j < nb) {
        const int k = j & (s - 1);
        if constexpr (s > 1) {
#pragma unroll
          for (int r = 1; r < R; ++r) v[t][r] = cmul(v[t][r], tw_at<step>(tw2048, r * k));
        }
        dft<R>(v[t]);
        const int base = (j - k) * R + k;
#pragma unroll
        for (int r = 0; r < R; ++r) buf[pidx(base) + pidx(r * s)] = v[t][r];
      }
    }
    wave_sync();
    wave_ifft_n<LG, LS + LR>(buf, tw2048, lane);
  }
}
// The length as a constant: no division by a stage's stride, no pass over the
// butterflies that a shorter line does not have, and addresses as one base and
// immediates (1D power of 50,000 lines 255 -> 216 us).
template <class TW>
__device__ __forceinline__ void wave_ifft(float2* buf, int M, TW tw2048, int lane) {
  switch (31 - __clz(M)) {
    case 1: return wave_ifft_n<1>(buf, tw2048, lane);
    case 2: return wave_ifft_n<2>(buf, tw2048, lane);
    case 3: return wave_ifft_n<3>(buf, tw2048, lane);
    case 4: return wave_ifft_n<4>(buf, tw2048, lane);
    case 5: return wave_ifft_n<5>(buf, tw2048, lane);
    case 6: return wave_ifft_n<6>(buf, tw2048, lane);
    case 7: return wave_ifft_n<7>(buf, tw2048, lane);
    case 8: return wave_ifft_n<8>(buf, tw2048, lane);
    case 9: return wave_ifft_n<9>(buf, tw2048, lane);
    case 10: return wave_ifft_n<10>(buf, tw2048, lane);
    default: return;   // M = 1
  }
}

// One radix-R stage of the in-place Stockham FFT wave_ifft8: s = product of the
// radices before it; every lane first reads all of its inputs, then writes.
template <int R, class TW>
__device__ __forceinline__ void wave_stage(float2* buf, int M, int ls, TW tw2048, int lane) {
  constexpr int LR = R == 16 ? 4 : R == 8 ? 3 : R == 4 ? 2 : 1;
  const int s = 1 << ls;   // shifts and masks: the compiler would not know that s divides as a power of two
  constexpr int TMAX = kHalfMax / R / 64 > 0 ? kHalfMax / R / 64 : 1;  // butterflies per lane at M = kHalfMax
  const int nb = M / R;
  float2 v[TMAX][R];
  asm volatile("" : "+v"(lane));   // as above
#pragma unroll
  for (int t = 0; t < TMAX; ++t) {
    const int j = lane + 64 * t;
    if (j < nb) {
#pragma unroll
      for (int r = 0; r < R; ++r) v[t][r] = buf[pidx(j) + pidx(r * nb)];
    }
  }
  wave_sync();
#pragma unroll
  for (int t = 0; t < TMAX; ++t) {
    const int j = lane + 64 * t;
    if (j < nb) {
      const int k = j & (s - 1);
      if (s > 1) {
        const int step = kTw2048 >> (ls + LR);
#pragma unroll
        for (int r = 1; r < R; ++r) v[t][r] = cmul(v[t][r], tw2048[r * k * step]);
      }
      dft<R>(v[t]);
      const int base = (j - k) * R + k;
#pragma unroll
      for (int r = 0; r < R; ++r) buf[pidx(base) + pidx(r * s)] = v[t][r];
    }
  }
  wave_sync();
}

// The same inverse DFT as wave_ifft by radix-8 stages (with radix-16 ones
// where they save a stage, then one radix-4 or radix-2 stage for what
// remains): fewer passes through LDS, more registers.
template <class TW>
__device__ __forceinline__ void wave_ifft8(float2* buf, int M, TW tw2048, int lane) {
  const int lg = 31 - __clz(M);
  int ls = 0;
  // radix-16 stages where they save a stage: 16 x 8^k for lg = 1 mod 3,
  // 16 x 16 x 8^k for lg = 2 mod 3 from 256 up
  const int n16 = (lg % 3 == 1 && lg >= 4) ? 1 : (lg % 3 == 2 && lg >= 8) ? 2 : 0;
  for (int i = 0; i < n16; ++i, ls += 4) wave_stage<16>(buf, M, ls, tw2048, lane);
  for (; lg - ls >= 3; ls += 3) wave_stage<8>(buf, M, ls, tw2048, lane);
  if (lg - ls == 2) wave_stage<4>(buf, M, ls, tw2048, lane);
  else if (lg - ls == 1) wave_stage<2>(buf, M, ls, tw2048, lane);
}


// ---- the small-scale field delta_S along one line (section "Gaussian fields
// along lines of sight"), shared by the skewer and tuning-evaluation kernels:
// Philox normals (stream 1, counter (qid << 33) + m) on the modes m = 1 ..
// ns/2 of a line of ns pixels, scaled by sqrt(P_s(k_m) / (ns dpix)), the DC
// mode zero, and one half-length complex inverse FFT.

// Amplitude sqrt(P_s(k_m) / (ns dpix)) of mode m of a line of ns pixels.
template <class A>
__device__ __forceinline__ float ps_amplitude(const A& a, int m, int ns, float amp_scale, float dk2) {
  const float kk = static_cast<float>(m) * static_cast<float>(m) * dk2;   // (k/kcut)^2
  float ratio = 1.0f;
  if (a.ps_ratio) {
    // the mode's k bin (FP64, so the bin decision matches a double-precision
    // reference): the largest b with edge_b <= k, clamped to the table
    const double k = (2.0 * M_PI / (static_cast<double>(ns) * a.dpix)) * m;
    const double* e = a.ps_edges_k;
    int b = 0;
    if (k >= e[a.ps_nb]) {
      b = a.ps_nb - 1;
    } else if (k >= e[0]) {
      int lo = 0, hi = a.ps_nb;   // e[lo] <= k < e[hi]
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (e[mid] <= k) lo = mid; else hi = mid;
      }
      b = lo;
    }
    ratio = a.ps_ratio[b];
  }
  return __builtin_amdgcn_sqrtf(amp_scale * __expf(-kk) * ratio);
}
// amp_scale and dk2 above
__device__ __forceinline__ float2 ps_scales(double amp, double kcut, double dpix, int ns) {
  const double dk = 2.0 * M_PI / (ns * dpix) / kcut;
  return make_float2(static_cast<float>(amp / (ns * dpix)), static_cast<float>(dk * dk));
}

// Mode Y_m of the small-scale spectrum (0 < m <= ns/2) from its normal pair z.
__device__ __forceinline__ float2 ps_mode(float amp, int m, int ns, int fixed_amp, float2 z) {
  float2 w = (m == ns / 2) ? make_float2(z.x, 0.0f) : make_float2(z.x * kSqrtHalf, z.y * kSqrtHalf);
  if (fixed_amp) {
    const float r = rsqrtf(w.x * w.x + w.y * w.y);
    w.x *= r;
    w.y *= r;
  }
  return make_float2(amp * w.x, amp * w.y);
}

// delta_S of one skewer by one wavefront into buf (pixel 2n in .x and pixel
// 2n+1 in .y of element pidx(n)); ns = next_pow2(npix) >= 2.  P_s(k) =
// amp exp(-(k/kcut)^2), times the ratio of k's bin when a.ps_ratio is set.
// A supplies the Philox key (seed), the fixed-amplitude switch (ps_fixed_amp) and
// either the amplitudes (ps_tab, laid out as k_prep writes them: with a tabulated
// ratio each mode's bin was an FP64 search; amp, kcut are then not read) or the
// pixel length (dpix) and the optional table (ps_nb, ps_edges_k, ps_ratio).  R8: the radix-8 FFT (fewer LDS passes); otherwise the
// radix-4 one, for callers that cannot spare its registers.
template <class A, class TW, bool R8 = true>
__device__ void small_scale_wave(const A& a, double amp, double kcut, uint64_t qid, int ns, float2* buf, TW tw,
                                 int lane) {
  const int M = ns / 2;
  float2 sc{};
  if constexpr (!A::kPsTab) sc = ps_scales(amp, kcut, a.dpix, ns);
  const int twstep = kTw2048 / ns;  // w^k = exp(2 pi i k / ns)
  // the modes Y_1 .. Y_M into buf (Y_M in slot 0: the DC mode is zero).  Mode
  // m is linear index (qid << 33) + m of stream 1, so the modes 2i and 2i + 1
  // share one Philox call (counter = linear index >> 1, words 0-1 and 2-3).
  for (int i = lane; i <= M / 2; i += 64) {
    const uint64_t ctr = ((qid << 33) + 2 * static_cast<uint64_t>(i)) >> 1;
    const uint4 wd = philox10_x3(make_uint4(static_cast<uint32_t>(ctr), static_cast<uint32_t>(ctr >> 32), 1u, 0u),
                                 static_cast<uint32_t>(a.seed), static_cast<uint32_t>(a.seed >> 32));
    const int m0 = 2 * i, m1 = 2 * i + 1;
    float2 am;
    if constexpr (A::kPsTab) {
      am = *reinterpret_cast<const float2*>(a.ps_tab + ns + m0);   // (one entry past M where m1 = M + 1)
    } else {
      am.x = ps_amplitude(a, m0, ns, sc.x, sc.y);
      am.y = ps_amplitude(a, m1, ns, sc.x, sc.y);
    }
    if (m0 >= 1 && m0 <= M) buf[pidx(m0 == M ? 0 : m0)] = ps_mode(am.x, m0, ns, a.ps_fixed_amp, box_muller(wd.x, wd.y));
    if (m1 <= M) buf[pidx(m1 == M ? 0 : m1)] = ps_mode(am.y, m1, ns, a.ps_fixed_amp, box_muller(wd.z, wd.w));
  }
  wave_sync();
  // Z_k = (Y_k + Y_{k+M}) + i (Y_k - Y_{k+M}) w^k with Y_{k+M} = conj(Y_{M-k});
  // a lane reads both of its slots k and M - k before writing them
  for (int k = lane; k <= M / 2; k += 64) {
    if (k == 0) {
      const float2 yM = buf[pidx(0)];  // real Nyquist mode
      buf[pidx(0)] = make_float2(yM.x, -yM.x);
      continue;
    }
    const float2 yk = buf[pidx(k)];
    const float2 ymk = buf[pidx(M - k)];
    const float2 w = tw[k * twstep];   // w^(M-k) = -conj(w^k), exactly so in the table
    {
      const float2 s = make_float2(yk.x + ymk.x, yk.y - ymk.y);   // Y_k + conj(Y_{M-k})
      const float2 d = make_float2(yk.x - ymk.x, yk.y + ymk.y);   // Y_k - conj(Y_{M-k})
      const float2 t = cmul(d, w);
      buf[pidx(k)] = make_float2(s.x - t.y, s.y + t.x);
    }
    if (M - k != k) {
      const float2 s = make_float2(ymk.x + yk.x, ymk.y - yk.y);
      const float2 d = make_float2(ymk.x - yk.x, ymk.y + yk.y);
      const float2 t = cmul(d, make_float2(-w.x, w.y));
      buf[pidx(M - k)] = make_float2(s.x - t.y, s.y + t.x);
    }
  }
  wave_sync();
  if constexpr (R8) wave_ifft8(buf, M, tw, lane);
  else wave_ifft(buf, M, tw, lane);
}

}  // namespace lya
