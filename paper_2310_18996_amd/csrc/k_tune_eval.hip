// Batched evaluation of the tuning statistics (gfx950): for G parameter draws
// (a, b, c) held constant over every stored pixel (the paper's reuse of saved
// forests, section "Adjusting mock parameters"), the mean flux of all pixels
// and the binned P1D of delta_F = F/Fbar - 1 with velocity units of the draw.
// Optionally each draw also carries a small-scale spectrum P_s, and delta_S is
// drawn again per draw and skewer (the P_s iteration's redraw) and added to
// the stored delta_L before the FGPA.
//
// One pass over the pixels for all G draws: a wavefront owns a skewer, holds
// its first 2048 (dens, eta) pixels in registers and, per draw, forms F, adds
// it to the skewer's sum and transforms the first N_P pixels in its LDS slice.
// For m >= 1 the DFT of F/Fbar - 1 is the DFT of F divided by Fbar (the
// constant only enters m = 0), so the periodogram is taken of F itself and
// divided by Fbar^2 once Fbar, a sum over all skewers, is known:
//   P_b = Dv sum_{q, m in b} |X_m(F_q)|^2 / N_P,q / (Fbar^2 count_b).
// Per-skewer partial sums are written in fixed order and reduced over skewers
// in a fixed tree, so the result does not depend on scheduling.
#include <algorithm>

#include "lya_internal.h"
#include "lya_linesum.h"
#include "lya_pull.h"
#include "lya_wavefft.h"

namespace lya {

constexpr int kTeWaves = 4;
constexpr int kTeNT = 64 * kTeWaves;
constexpr int kTeReg = 32;  // pixels per lane kept in registers (2048 per wave)

// Each draw's table of first modes, and the queue cleared.
__global__ void __launch_bounds__(256) k_te_prep(TuneEvalArgs a) {
  const int part = blockIdx.x, g = blockIdx.y;
  if (g == 0 && part == 0 && threadIdx.x < kPullCounters) a.queue[threadIdx.x * kPullStride] = 0u;
  mode_table(a.modes + g * kLenClasses * mode_row(a.nk), a.k_edges, a.nk, a.dv[g], part, threadIdx.x, 256);
}

// DS: delta_S redrawn per draw (a separate instantiation, so that the plain
// evaluation keeps its register budget).  As in k_p1d: three blocks per CU (the
// powers take the transform's place in LDS), k bins from the draws' tables of
// first modes, a line's bin sums written in one piece.  64 draws on 14M pixels of
// 20,000 lines: 5.20 ms with FP64 bin searches per line and draw, two blocks per CU
// and run-time transform lengths, 2.45 ms; 2.05 ms with the queue on 16 cache lines.
template <bool DS>
__global__ void __launch_bounds__(kTeNT, 3) k_tune_eval(TuneEvalArgs a) {
  __shared__ float2 sbuf[kTeWaves][kHalfBuf];
  __shared__ float2 stw[tidx(kTw2048)];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  load_twiddles(stw, a.tw2048, threadIdx.x, kTeNT);
  __syncthreads();
  const LdsTw tw{stw};
  float2* buf = sbuf[wv];
  float* bf = reinterpret_cast<float*>(buf);
  const int nk = a.nk, row = mode_row(nk), lg = bin_split(nk);
  const int64_t ld = a.n_sk;
  LinePull<TuneEvalArgs, kTeWaves> pull;
  for (int64_t c = pull.first(lane); c < a.chunks; c = pull.next(lane)) {
    const int64_t q0 = c * a.chunk;
    const int64_t q1 = q0 + a.chunk < a.n_sk ? q0 + a.chunk : a.n_sk;
    for (int64_t q = q0; q < q1; ++q) {
      if (q == q1 - 1) pull.ask(lane);
      const int np = a.npix[q];
      const int64_t off = a.offset[q];
      const int cls = len_class(np);
      const int n_p = cls ? 1 << cls : 0;
      const int M = n_p / 2;
      float d[kTeReg], e[kTeReg];
#pragma unroll
      for (int i = 0; i < kTeReg; ++i) {
        const int j = lane + 64 * i;
        d[i] = j < np ? a.dens[off + j] : 0.0f;
        e[i] = j < np ? a.eta[off + j] : 0.0f;
      }
      int ns = 1;
      while (ns < np) ns <<= 1;
      const bool with_ds = DS && ns >= 2;
      for (int g = 0; g < a.G; ++g) {
        const float ca = a.draw[g][0], cb = a.draw[g][1], cc = a.draw[g][2];
        double* ps = a.ps + (static_cast<int64_t>(g) * ld + q) * nk;
        if (with_ds && ns > 2 * kHalfMax) {
          // delta_S exists on lines of at most 2048 pixels: an input error,
          // which makes this draw's mean flux (and so its P1D) NaN
          if (lane == 0) a.fs[g * ld + q] = __builtin_nan("");
          for (int b = lane; b < nk; b += 64) ps[b] = 0.0;
          continue;
        }
        // the bin's modes, read while the line is transformed
        const int* mt = a.modes + (g * kLenClasses + cls) * row;
        const int bin = lane >> lg;
        const int m0 = bin < nk ? mt[bin] : 1, m1 = bin < nk ? mt[bin + 1] : 1;
        const int mlo = mt[nk + 1], mhi = mt[nk + 2];
        // a lane index the compiler cannot hoist addresses by: kept for the whole
        // kernel they would not leave the pixels their registers
        int ln = lane;
        asm volatile("" : "+v"(ln));
        if (with_ds) {
          // delta_S into the LDS line; each lane then reads and overwrites
          // only its own pixels' slots (pixel j at bf[2 pidx(j/2) + j%2])
          small_scale_wave<TuneEvalArgs, LdsTw, false>(a, a.ds_amp[g], a.ds_kcut[g], static_cast<uint64_t>(a.id_base + q), ns, buf, tw, ln);
        }
        const int slot0 = 2 * pidx(ln >> 1) + (ln & 1);   // pixel j at bf[2 pidx(j/2) + j%2]
        double fsum = 0.0;
#pragma unroll
        for (int i = 0; i < kTeReg; ++i) {
          if (64 * i >= np) break;
          const int j = ln + 64 * i;
          if (j < np) {
            const int slot = slot0 + 2 * pidx(32 * i);
            const float delta = with_ds ? d[i] + bf[slot] : d[i];
            const float F = __expf(-ca * __expf(cb * (delta + cc * e[i])));
            fsum += F;
            if (j < n_p) bf[slot] = F;
          }
        }
        for (int j = 64 * kTeReg + lane; j < np; j += 64)  // pixels beyond the register window (no delta_S here)
          fsum += __expf(-ca * __expf(cb * (a.dens[off + j] + cc * a.eta[off + j])));
#pragma unroll
        for (int w = 32; w >= 1; w >>= 1) fsum += __shfl_xor(fsum, w);
        if (lane == 0) a.fs[g * ld + q] = fsum;
        if (M == 0) {
          for (int b = lane; b < nk; b += 64) ps[b] = 0.0;
          continue;
        }
        wave_sync();
        wave_ifft(buf, M, tw, ln);
        power_in_place(buf, M, mlo, mhi, 1.0f, tw, ln);
        wave_sync();
        const double s = bin < nk ? bin_sum(buf, M, m0, m1, lg, lane) : 0.0;
        if (bin < nk && (lane & ((1 << lg) - 1)) == 0) ps[bin] = s * (1.0 / n_p);
        wave_sync();
      }
    }
  }
}

__global__ void __launch_bounds__(256) k_te_sum(LineSumArgs a) { line_sum_block(a, blockIdx.x, blockIdx.y); }

// Statistics per draw: Fbar, then P_b (NaN for an empty bin); FP64 rows and,
// when rows32 is given, FP32 rows (emulator labels).  ONE: the sums of stage 1 as
// well (R = 1).
template <bool ONE>
__global__ void __launch_bounds__(ONE ? 256 : 128) k_te_stats(TuneEvalArgs a, LineSumArgs l, double* rows, float* rows32) {
  __shared__ long long cls[kLenClasses + 1];
  __shared__ double sf;
  const int g = blockIdx.x, b = threadIdx.x, nk = a.nk, row = mode_row(nk);
  if constexpr (ONE) {
    line_sum_block(l, 0, g);
    __syncthreads();
  }
  line_counts(l, g, cls);
  if (b == 127) sf = line_total(l, g, nk);
  __syncthreads();
  if (b > nk) return;
  const long long pix = cls[kLenClasses];
  const double fbar = pix > 0 ? sf / static_cast<double>(pix) : NAN;
  double v = fbar;
  if (b > 0) {
    const int* mt = a.modes + g * kLenClasses * row + b - 1;
    long long n = 0;
    for (int c = 1; c < kLenClasses; ++c) n += cls[c] * max(0, mt[c * row + 1] - mt[c * row]);
    v = n > 0 ? a.dv[g] * line_total(l, g, b - 1) / (fbar * fbar * static_cast<double>(n)) : NAN;
  }
  if (rows) rows[g * (nk + 1) + b] = v;
  if (rows32) rows32[g * (nk + 1) + b] = static_cast<float>(v);
}

size_t tune_eval_aux_bytes(int64_t n_sk, int nk) {
  return sizeof(int) * kTuneEvalMaxG * kLenClasses * ((mode_row(nk) + 1) & ~1) + line_sum_bytes(n_sk, nk, kTuneEvalMaxG);
}

hipError_t launch_tune_eval(const TuneEvalArgs& p, double* rows, float* rows32, hipStream_t st) {
  if (p.G < 1 || p.G > kTuneEvalMaxG || p.nk < 1 || p.nk > kMaxKBins) return hipErrorInvalidValue;
  TuneEvalArgs a = p;
  a.modes = reinterpret_cast<int*>(a.aux);
  LYA_TIMED("tune_eval_prep", st, hipLaunchKernelGGL(k_te_prep, dim3(kModeBlocks, a.G), dim3(256), 0, st, a));
  int64_t blocks = static_cast<int64_t>(device_cus()) * 3;
  // eight pulls per wave or more, so that the waves end together
  a.chunk = static_cast<int>(std::min<int64_t>(a.chunk, std::max<int64_t>(1, a.n_sk / (8 * blocks * kTeWaves))));
  a.chunks = (a.n_sk + a.chunk - 1) / a.chunk;
  if (blocks * kTeWaves > a.chunks) blocks = (a.chunks + kTeWaves - 1) / kTeWaves;
  if (blocks < 1) blocks = 1;
  const dim3 grid(static_cast<unsigned>(blocks));
  if (a.n_sk > 0 && a.with_ds)
    LYA_TIMED("tune_eval_ds", st, hipLaunchKernelGGL(k_tune_eval<true>, grid, dim3(kTeNT), 0, st, a));
  else if (a.n_sk > 0)
    LYA_TIMED("tune_eval", st, hipLaunchKernelGGL(k_tune_eval<false>, grid, dim3(kTeNT), 0, st, a));
  LineSumArgs l{};
  l.n = a.n_sk;
  l.nk = a.nk;
  l.R = line_sum_blocks(a.n_sk);
  l.npix = a.npix;
  l.rows = a.ps;
  l.fs = a.fs;
  l.part = reinterpret_cast<double*>(a.aux + sizeof(int) * kTuneEvalMaxG * kLenClasses * ((mode_row(a.nk) + 1) & ~1));
  l.hist = reinterpret_cast<long long*>(l.part + static_cast<size_t>(a.G) * l.R * (l.nk + 1));
  if (l.R > 1) {
    LYA_TIMED("tune_eval_sum", st, hipLaunchKernelGGL(k_te_sum, dim3(l.R, a.G), dim3(256), 0, st, l));
    LYA_TIMED("tune_eval_stats", st,
              hipLaunchKernelGGL(k_te_stats<false>, dim3(a.G), dim3(128), 0, st, a, l, rows, rows32));
  } else {
    LYA_TIMED("tune_eval_stats", st,
              hipLaunchKernelGGL(k_te_stats<true>, dim3(a.G), dim3(256), 0, st, a, l, rows, rows32));
  }
  return hipGetLastError();
}

}  // namespace lya
