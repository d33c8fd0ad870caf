// 1D flux power spectrum (gfx950).
//
// delta_F = F / Fbar - 1 (equation::definition_delta) on the first
// N_P = min(2^floor(log2 n_q), 2048) pixels of every skewer, Fbar taken per distance bin
// from given sums; periodogram P(k_m) = Dv |X_m|^2 / N_P for m = 1..N_P/2 with
// k_m = 2 pi m / (N_P Dv) (Dv one FP64 constant, the pixel at the reference
// redshift); the modes of each skewer are summed per k bin in FP64 in a fixed
// order and written per skewer, then the skewers are summed per bin in a fixed
// order (so the result does not depend on scheduling).
//
// The real DFT of length N_P is one complex FFT of length M = N_P/2 on
// z_n = d(2n) + i d(2n+1); with Z its transform (sign +, whose modulus equals
// the forward one's for real input) the full-length coefficient is
// X_m = (Z_m + conj Z_{M-m})/2 + w^m (Z_m - conj Z_{M-m})/(2i), w = exp(2 pi i/N_P).
#include <algorithm>

#include "lya_internal.h"
#include "lya_linesum.h"
#include "lya_pull.h"
#include "lya_wavefft.h"

namespace lya {

constexpr int kPdWaves = 4;
constexpr int kPdNT = 64 * kPdWaves;
constexpr int kPdTw = kTw2048 * 3 / 4;

// A wave per line.  What it costs is latency, so: three blocks per CU (53 KB of
// LDS; the powers take the transform's place), a pull's line table in one load, a
// line's pixels all in flight at once, k bins from the block's table of first
// modes, and the few distance edges inside a line compared one by one (a search
// per pixel over all edges was five dependent LDS reads).  The arithmetic of each
// power is as in a radix-4 transform of one line.  35M pixels of 50,000 lines:
// 305 us with FP64 bin searches per line and two blocks per CU, 214 us;
// 128 us with the queue on 16 cache lines, 124 us with the table from the launch before
// (read per line from memory instead of the block's copy: 131 us).
__global__ void __launch_bounds__(kPdNT, 3) k_p1d(P1dArgs a) {
  __shared__ float2 sbuf[kPdWaves][kHalfBuf];
  __shared__ float2 stw[tidx(kPdTw)];
  __shared__ float sfm[kMaxZBins];
  __shared__ uint32_t smt2[kLenClasses * mode_row(kMaxKBins) / 2];
  const unsigned short* smt = reinterpret_cast<const unsigned short*>(smt2);
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int nk = a.n_kbins, row = mode_row(nk), lg = bin_split(nk);
  // the first modes, on their way while the other tables come
  static_assert(kLenClasses % 2 == 0 && kLenClasses * mode_row(kMaxKBins) / 2 <= 2 * kPdNT, "two words per thread");
  const uint32_t* modes = reinterpret_cast<const uint32_t*>(a.modes);
  const int words = kLenClasses * row / 2;
  const uint32_t w0 = tid < words ? modes[tid] : 0u, w1 = tid + kPdNT < words ? modes[tid + kPdNT] : 0u;
  load_twiddles<kPdTw>(stw, a.tw2048, tid, kPdNT);
  for (int b = tid; b < a.n_fbins; b += kPdNT) {
    const double c = static_cast<double>(a.fcount[b]);
    sfm[b] = c > 0.0 ? static_cast<float>(a.fsum[b] / c) : 1.0f;
  }
  if (tid < words) smt2[tid] = w0;
  if (tid + kPdNT < words) smt2[tid + kPdNT] = w1;
  __syncthreads();
  const LdsTw tw{stw};
  float2* buf = sbuf[wv];
  float* bf = reinterpret_cast<float*>(buf);
  LinePull<P1dArgs, kPdWaves> pull;
  for (int64_t c = pull.first(lane); c < a.chunks; c = pull.next(lane)) {
    const int64_t q0 = c * a.chunk;
    const int64_t q1 = q0 + a.chunk < a.n_sk ? q0 + a.chunk : a.n_sk;
    // the pull's lines, a lane each (chunk <= 64)
    const int64_t ql = q0 + lane < q1 ? q0 + lane : q0;
    const int npl = a.npix[ql];
    const int64_t offl = a.offset[ql];
    const double chil = a.chi0[ql];
    for (int64_t q = q0; q < q1; ++q) {
      if (q == q1 - 1) pull.ask(lane);
      const int i = static_cast<int>(q - q0);
      const int np = lane_i32(npl, i);
      double* psum = a.part_sum + q * nk;   // the line's partial sums
      const int cls = len_class(np);
      if (cls == 0) {
        for (int b = lane; b < nk; b += 64) psum[b] = 0.0;
        continue;
      }
      const int n_p = 1 << cls, M = n_p / 2;
      const float* f = a.flux + lane_i64(offl, i);
      const double chi0 = lane_f64(chil, i);
      float F[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int j = lane + 64 * k;
        if (j < n_p) F[k] = f[j];
      }
      // distance bins: the lane's edge, and edge 64 (of 64 bins) apart
      const int jb = lane <= a.n_fbins ? first_below(a.chi_edges[lane], chi0, a.dchi, n_p) : 0;
      const int jb64 = a.n_fbins == 64 ? first_below(a.chi_edges[64], chi0, a.dchi, n_p) : 0;
      // edges above the whole line, and those inside it
      const int above = __popcll(__ballot(lane <= a.n_fbins && jb >= n_p)) + (jb64 >= n_p ? 1 : 0);
      const uint64_t inside = __ballot(lane <= a.n_fbins && jb > 0 && jb < n_p);
      const bool inside64 = jb64 > 0 && jb64 < n_p;
      const auto pixel = [&](int j, int slot, float v) {
        // edges with jb > j: pixel j lies in bin cnt - 1 (clamped)
        int cnt = above + (inside64 && jb64 > j ? 1 : 0);
        for (uint64_t m = inside; m; m &= m - 1) cnt += lane_i32(jb, __builtin_ctzll(m)) > j ? 1 : 0;
        int b = cnt - 1;
        b = b < 0 ? 0 : (b > a.n_fbins - 1 ? a.n_fbins - 1 : b);
        bf[slot] = v / sfm[b] - 1.0f;
      };
      const int slot0 = 2 * pidx(lane >> 1) + (lane & 1);   // pixel j at bf[2 pidx(j/2) + j%2]
      for (int j0 = 0;;) {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int j = j0 + lane + 64 * k;
          if (j < n_p) pixel(j, slot0 + 2 * pidx((j0 >> 1) + 32 * k), F[k]);
        }
        j0 += 512;
        if (j0 >= n_p) break;
#pragma unroll
        for (int k = 0; k < 8; ++k) F[k] = f[j0 + lane + 64 * k];   // n_p is a multiple of 512 here
      }
      wave_sync();
      wave_ifft(buf, M, tw, lane);
      const unsigned short* mt = smt + cls * row;
      const float scale = static_cast<float>(a.dv / n_p);
      power_in_place(buf, M, mt[nk + 1], mt[nk + 2], scale, tw, lane);
      wave_sync();
      const int b = lane >> lg;
      const double s = b < nk ? bin_sum(buf, M, mt[b], mt[b + 1], lg, lane) : 0.0;
      if (b < nk && (lane & ((1 << lg) - 1)) == 0) psum[b] = s;
      wave_sync();
    }
  }
}

__global__ void __launch_bounds__(256) k_p1d_sum(LineSumArgs a) { line_sum_block(a, blockIdx.x, 0); }

// ONE: the sums of stage 1 as well (R = 1)
template <bool ONE>
__global__ void __launch_bounds__(256) k_p1d_final(LineSumArgs a, const unsigned short* __restrict__ modes, double* psum,
                                                   int64_t* pcount) {
  __shared__ long long cls[kLenClasses + 1];
  const int b = threadIdx.x, row = mode_row(a.nk);
  if constexpr (ONE) {
    line_sum_block(a, 0, 0);
    __syncthreads();
  }
  line_counts(a, 0, cls);
  if (b < a.nk && psum) psum[b] = line_total(a, 0, b);
  __syncthreads();
  if (b >= a.nk || !pcount) return;
  long long n = 0;
  for (int c = 1; c < kLenClasses; ++c) n += cls[c] * max(0, modes[c * row + b + 1] - modes[c * row + b]);
  pcount[b] = n;
}

hipError_t launch_p1d(const P1dArgs& p, double* psum, int64_t* pcount, hipStream_t st) {
  P1dArgs a = p;
  int64_t blocks = static_cast<int64_t>(device_cus()) * 3;
  // eight pulls per wave or more, so that the waves end together
  a.chunk = static_cast<int>(std::min<int64_t>(a.chunk, std::max<int64_t>(1, a.n_sk / (8 * blocks * kPdWaves))));
  a.chunks = (a.n_sk + a.chunk - 1) / a.chunk;
  if (blocks * kPdWaves > a.chunks) blocks = (a.chunks + kPdWaves - 1) / kPdWaves;
  if (blocks < 1) blocks = 1;
  if (a.n_sk > 0) LYA_TIMED("p1d", st, hipLaunchKernelGGL(k_p1d, dim3(static_cast<unsigned>(blocks)), dim3(kPdNT), 0, st, a));
  LineSumArgs l{};
  l.n = a.n_sk;
  l.nk = a.n_kbins;
  l.R = line_sum_blocks(a.n_sk);
  l.npix = a.npix;
  l.rows = a.part_sum;
  l.part = reinterpret_cast<double*>(a.aux);
  l.hist = reinterpret_cast<long long*>(l.part + static_cast<size_t>(l.R) * (l.nk + 1));
  if (l.R > 1) LYA_TIMED("p1d_sum", st, hipLaunchKernelGGL(k_p1d_sum, dim3(l.R), dim3(256), 0, st, l));
  const auto fin = l.R > 1 ? k_p1d_final<false> : k_p1d_final<true>;
  LYA_TIMED("p1d_final", st, hipLaunchKernelGGL(fin, dim3(1), dim3(256), 0, st, l, a.modes, psum, pcount));
  return hipGetLastError();
}

}  // namespace lya
