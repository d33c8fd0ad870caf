// Tuning emulator: a 4 -> 256 -> 256 -> 256 -> n_out MLP (GELU hidden layers,
// linear output) mapping FGPA parameters and redshift (a, b, c, z) to the
// statistics the tuning loop matches (mean flux and ln P1D per k bin).
// Training: MSE on standardised inputs and outputs, Adam (Kingma & Ba 2014),
// FP32 master weights; the matrix products run on MFMA in bfloat16 with FP32
// accumulation (v_mfma_f32_16x16x16_bf16), or in plain FP32 for checks.
// Row-vector convention: h = gelu(x W + b), W stored [in][out] row-major.
// GELU is the exact form x Phi(x) = x erfc(-x / sqrt 2) / 2.
#include <math.h>
#include <string.h>

#include <vector>

#include "../../include/lyamock.h"
#include "lya_internal.h"
#include "lya_nm.h"

namespace lya {

constexpr int kIn = 4, kHid = 256, kMaxOut = 64;

struct EmuHeader {
  int32_t n_out;
  int32_t step;    // Adam steps taken
  int32_t log_from;
  int32_t in_log;  // bit i: input i enters as ln x
  float in_lo[4], in_hi[4];
  float in_mul[4], in_add[4];  // scaled input = in_mul (x or ln x) + in_add, in [-1, 1] over the range
  float out_mean[kMaxOut], out_std[kMaxOut], out_mask[kMaxOut];
};

__device__ __forceinline__ float scale_input(const EmuHeader* __restrict__ h, int i, float x) {
  const float v = ((h->in_log >> i) & 1) ? logf(x) : x;
  return fmaf(h->in_mul[i], v, h->in_add[i]);
}
constexpr size_t kHeaderBytes = 2048;
static_assert(sizeof(EmuHeader) <= kHeaderBytes, "header");

__host__ __device__ inline size_t n_params(int n_out) {
  return static_cast<size_t>(kIn) * kHid + kHid + 2 * (static_cast<size_t>(kHid) * kHid + kHid) +
         static_cast<size_t>(kHid) * n_out + n_out;
}

struct Offs {
  size_t W[4], b[4];
};
__host__ __device__ inline Offs param_offsets(int n_out) {
  Offs o;
  size_t p = 0;
  const int fin[4] = {kIn, kHid, kHid, kHid};
  const int fout[4] = {kHid, kHid, kHid, n_out};
  for (int l = 0; l < 4; ++l) {
    o.W[l] = p;
    p += static_cast<size_t>(fin[l]) * fout[l];
    o.b[l] = p;
    p += fout[l];
  }
  return o;
}

__device__ __forceinline__ float gelu(float x) { return 0.5f * x * erfcf(-x * 0.70710678118654752f); }
__device__ __forceinline__ float gelu_grad(float x) {
  return 0.5f * erfcf(-x * 0.70710678118654752f) + x * 0.39894228040143268f * expf(-0.5f * x * x);
}

// ---------------------------------------------------------------- init
__global__ void __launch_bounds__(256) k_emu_init(float* params, float* m, float* v, int n_out, uint64_t seed) {
  const Offs o = param_offsets(n_out);
  const size_t np = n_params(n_out);
  for (size_t i = blockIdx.x * 256ull + threadIdx.x; i < np; i += static_cast<size_t>(gridDim.x) * 256) {
    const int l = i < o.W[1] ? 0 : i < o.W[2] ? 1 : i < o.W[3] ? 2 : 3;
    float val = 0.0f;
    if (i < (l == 0 ? o.b[0] : l == 1 ? o.b[1] : l == 2 ? o.b[2] : o.b[3])) {
      // weight of layer l: He normal, std sqrt(2 / fan_in)
      const float2 z = normal_pair(seed, 3u, static_cast<uint64_t>(i) << 1);
      val = z.x * sqrtf(2.0f / (l == 0 ? kIn : kHid));
    }
    params[i] = val;
    m[i] = 0.0f;
    v[i] = 0.0f;
  }
}

// per output column: mean and std over the labels (ln for columns >= log_from),
// mask 0 if any label is not finite; one block per column, fixed-order FP64 sums
__global__ void __launch_bounds__(256) k_emu_stats(const float* __restrict__ y, int64_t n, int n_out, int log_from,
                                                   EmuHeader* h) {
  __shared__ double s1[256], s2[256];
  __shared__ int sbad[256];
  const int c = blockIdx.x, t = threadIdx.x;
  double a = 0.0, b = 0.0;
  int bad = 0;
  for (int64_t i = t; i < n; i += 256) {
    float v = y[i * n_out + c];
    if (c >= log_from) v = logf(v);
    if (!isfinite(v)) {
      bad = 1;
      continue;
    }
    a += v;
    b += static_cast<double>(v) * v;
  }
  s1[t] = a;
  s2[t] = b;
  sbad[t] = bad;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w) {
      s1[t] += s1[t + w];
      s2[t] += s2[t + w];
      sbad[t] |= sbad[t + w];
    }
    __syncthreads();
  }
  if (t == 0) {
    const double mean = s1[0] / static_cast<double>(n);
    const double var = s2[0] / static_cast<double>(n) - mean * mean;
    h->out_mean[c] = static_cast<float>(mean);
    h->out_std[c] = static_cast<float>(var > 1e-30 ? sqrt(var) : 1.0);
    h->out_mask[c] = sbad[0] ? 0.0f : 1.0f;
  }
}

// training batch of step s: rows (s B + i) mod n, standardised
__global__ void __launch_bounds__(256) k_emu_gather(const float* __restrict__ x, const float* __restrict__ y, int64_t n,
                                                    int64_t s, int B, const EmuHeader* __restrict__ h, float* x0,
                                                    float* tgt) {
  const int n_out = h->n_out;
  for (int k = blockIdx.x * 256 + threadIdx.x; k < B * (kIn + n_out); k += gridDim.x * 256) {
    const int i = k / (kIn + n_out), c = k % (kIn + n_out);
    const int64_t r = (s * B + i) % n;
    if (c < kIn) {
      x0[i * kIn + c] = scale_input(h, c, x[r * kIn + c]);
    } else {
      const int o = c - kIn;
      float v = y[r * n_out + o];
      if (o >= h->log_from) v = logf(v);
      v = (v - h->out_mean[o]) / h->out_std[o];
      tgt[i * n_out + o] = (h->out_mask[o] > 0.0f && isfinite(v)) ? v : 0.0f;
    }
  }
}

// ---------------------------------------------------------------- GEMM
enum { EPI_STORE = 0, EPI_BIAS = 1, EPI_BIAS_GELU = 2, EPI_GELU_GRAD = 3 };

// C = op(A) op(B) with epilogue.  op(A)[m][k] = TA ? A[k lda + m] : A[m lda + k],
// op(B)[k][n] = TB ? B[n ldb + k] : B[k ldb + n].  EPI_BIAS_GELU also writes the
// pre-activation to aux; EPI_GELU_GRAD multiplies by gelu'(aux).
__device__ __forceinline__ float epilogue(int epi, float acc, int m, int n, const float* bias, float* aux, int ldaux,
                                          float& out_aux) {
  (void)out_aux;
  if (epi == EPI_BIAS) return acc + bias[n];
  if (epi == EPI_BIAS_GELU) {
    const float zv = acc + bias[n];
    aux[static_cast<size_t>(m) * ldaux + n] = zv;
    return gelu(zv);
  }
  if (epi == EPI_GELU_GRAD) return acc * gelu_grad(aux[static_cast<size_t>(m) * ldaux + n]);
  return acc;
}

// FP32 reference product: one output per thread
template <bool TA, bool TB>
__global__ void __launch_bounds__(256) k_gemm_f32(int M, int N, int K, const float* __restrict__ A, int lda,
                                                  const float* __restrict__ B, int ldb, float* C, int ldc,
                                                  const float* bias, int epi, float* aux, int ldaux) {
  const int64_t id = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (id >= static_cast<int64_t>(M) * N) return;
  const int m = static_cast<int>(id / N), n = static_cast<int>(id % N);
  float acc = 0.0f;
  for (int k = 0; k < K; ++k) {
    const float a = TA ? A[static_cast<size_t>(k) * lda + m] : A[static_cast<size_t>(m) * lda + k];
    const float b = TB ? B[static_cast<size_t>(n) * ldb + k] : B[static_cast<size_t>(k) * ldb + n];
    acc = fmaf(a, b, acc);
  }
  float dummy;
  C[static_cast<size_t>(m) * ldc + n] = epilogue(epi, acc, m, n, bias, aux, ldaux, dummy);
}

// FP32 product for few outputs and a long inner dimension (the first
// layer's weight gradient): sixteen outputs per block, sixteen threads per
// output each summing every sixteenth k in order, then a fixed tree
template <bool TA, bool TB>
__global__ void __launch_bounds__(256) k_gemm_f32_ks(int M, int N, int K, const float* __restrict__ A, int lda,
                                                     const float* __restrict__ B, int ldb, float* C, int ldc,
                                                     const float* bias, int epi, float* aux, int ldaux) {
  __shared__ float sp[16][17];
  const int oi = threadIdx.x & 15, j = threadIdx.x >> 4;
  const int64_t id = static_cast<int64_t>(blockIdx.x) * 16 + oi;
  const bool valid = id < static_cast<int64_t>(M) * N;
  const int m = valid ? static_cast<int>(id / N) : 0, n = valid ? static_cast<int>(id % N) : 0;
  float acc = 0.0f;
  if (valid)
    for (int k = j; k < K; k += 16) {
      const float a = TA ? A[static_cast<size_t>(k) * lda + m] : A[static_cast<size_t>(m) * lda + k];
      const float b = TB ? B[static_cast<size_t>(n) * ldb + k] : B[static_cast<size_t>(k) * ldb + n];
      acc = fmaf(a, b, acc);
    }
  sp[j][oi] = acc;
  __syncthreads();
  for (int w = 8; w > 0; w >>= 1) {
    if (j < w) sp[j][oi] += sp[j + w][oi];
    __syncthreads();
  }
  if (j == 0 && valid) {
    float dummy;
    C[static_cast<size_t>(m) * ldc + n] = epilogue(epi, sp[0][oi], m, n, bias, aux, ldaux, dummy);
  }
}

template <bool TA, bool TB>
hipError_t gemm(int M, int N, int K, const float* A, int lda, const float* B, int ldb, float* C, int ldc,
                const float* bias, int epi, float* aux, int ldaux, hipStream_t st) {
  const int64_t tot = static_cast<int64_t>(M) * N;
  if (tot <= 65536 && K >= 64) {
    hipLaunchKernelGGL((k_gemm_f32_ks<TA, TB>), dim3(static_cast<unsigned>((tot + 15) / 16)), dim3(256), 0, st, M, N,
                       K, A, lda, B, ldb, C, ldc, bias, epi, aux, ldaux);
  } else {
    hipLaunchKernelGGL((k_gemm_f32<TA, TB>), dim3(static_cast<unsigned>((tot + 255) / 256)), dim3(256), 0, st, M, N,
                       K, A, lda, B, ldb, C, ldc, bias, epi, aux, ldaux);
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------- loss, bias grads, Adam
// dY = 2 (Y - T) mask / (B n_eff), one element per thread; per-block FP64
// partial sums of the squared misfit, then k_emu_loss sums the partials in a
// fixed order (loss = sum / (B n_eff))
__device__ __forceinline__ float emu_neff(const EmuHeader* __restrict__ h) {
  float neff = 0.0f;
  for (int o = 0; o < h->n_out; ++o) neff += h->out_mask[o];
  return neff > 0.0f ? neff : 1.0f;
}

__global__ void __launch_bounds__(256) k_emu_dloss(const float* __restrict__ y, const float* __restrict__ t, int B,
                                                   const EmuHeader* __restrict__ h, float* dy, double* lpart) {
  __shared__ double sl[256];
  const int n_out = h->n_out;
  const float scale = 2.0f / (static_cast<float>(B) * emu_neff(h));
  const int k = blockIdx.x * 256 + threadIdx.x;
  double l = 0.0;
  if (k < B * n_out) {
    const float d = (y[k] - t[k]) * h->out_mask[k % n_out];
    dy[k] = scale * d;
    l = static_cast<double>(d) * d;
  }
  sl[threadIdx.x] = l;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) sl[threadIdx.x] += sl[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) lpart[blockIdx.x] = sl[0];
}

__global__ void __launch_bounds__(256) k_emu_loss(const double* __restrict__ lpart, int nparts, int B,
                                                  const EmuHeader* __restrict__ h, float* loss) {
  __shared__ double sl[256];
  double l = 0.0;
  for (int i = threadIdx.x; i < nparts; i += 256) l += lpart[i];
  sl[threadIdx.x] = l;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) sl[threadIdx.x] += sl[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0 && loss) loss[0] = static_cast<float>(sl[0] / (static_cast<double>(B) * emu_neff(h)));
}

// db[n] = sum over rows of d[m][n]: 64 columns per block, sixteen row groups
// (rows g, g + 16, ...) summed in order, then the groups in a fixed tree
__global__ void __launch_bounds__(1024) k_colsum(const float* __restrict__ d, int M, int N, float* db) {
  __shared__ float sp[16][64];
  const int c = threadIdx.x & 63, g = threadIdx.x >> 6;
  const int n = blockIdx.x * 64 + c;
  float s = 0.0f;
  if (n < N)
    for (int m = g; m < M; m += 16) s += d[static_cast<size_t>(m) * N + n];
  sp[g][c] = s;
  __syncthreads();
  for (int w = 8; w > 0; w >>= 1) {
    if (g < w) sp[g][c] += sp[g + w][c];
    __syncthreads();
  }
  if (g == 0 && n < N) db[n] = sp[0][c];
}

struct AdamArgs {
  float *p, *m, *v;
  float lr, b1, b2, eps, bc1, bc2;
};
__device__ __forceinline__ float adam_update(const AdamArgs& a, size_t i, float gi) {
  const float mi = a.b1 * a.m[i] + (1.0f - a.b1) * gi;
  const float vi = a.b2 * a.v[i] + (1.0f - a.b2) * gi * gi;
  a.m[i] = mi;
  a.v[i] = vi;
  return a.p[i] -= a.lr * (mi / a.bc1) / (sqrtf(vi / a.bc2) + a.eps);
}

__global__ void __launch_bounds__(256) k_adam(AdamArgs a, const float* __restrict__ g, size_t np) {
  for (size_t i = blockIdx.x * 256ull + threadIdx.x; i < np; i += static_cast<size_t>(gridDim.x) * 256)
    adam_update(a, i, g[i]);
}

// ---------------------------------------------------------------- bfloat16 training batch in two launches
// The batch used to take 17 launches (a product, an epilogue or a column sum
// each, 4-16 us apiece, on 16-64 blocks), a training step 180 us at batch 512
// for 0.4 GFLOP; now 32 us, bound by the chain of six dependent layers in
// k_emu_rows.
// No row of the batch needs another until the weight gradients, so
// k_emu_rows takes 4, 8 or 16 rows (row_shape) through the forward pass, the loss and the backward
// pass to the inputs of every layer, and k_emu_grads then forms all weight and
// bias gradients (and, in training, Adam's update of each parameter, which only
// it touches).  The products, their order of summation and their roundings are
// those of a chain of 16-deep MFMA steps per output, so the gradients do not
// depend on how rows and tiles are dealt out.
typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef float v4f32 __attribute__((ext_vector_type(4)));
typedef __bf16 v2bf16 __attribute__((ext_vector_type(2)));
typedef float v2f32 __attribute__((ext_vector_type(2)));

// round to nearest even (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v2f32{a, b}, v2bf16));
}
__device__ __forceinline__ v4i16 bf16x4(float a, float b, float c, float d) {
  return __builtin_bit_cast(v4i16, make_uint2(pack_bf16(a, b), pack_bf16(c, d)));
}

constexpr int kRowPad = 16;            // the batch is padded to whole MFMA steps of rows
constexpr int kRowNT = 512;            // a wave per 32 hidden units
constexpr int kRowLd = kHid + 8;       // LDS row of bfloat16 activations

// The weights of layers 2-4 as bfloat16 MFMA B operands, forward and
// transposed: four values (k = 16 s + 4 (lane / 16) + q) of column lane % 16 of
// tile t at [t][s][lane], so a wave reads an operand as 512 contiguous bytes
// and 64 registers hold the next product's.  Built by k_emu_pack for a call,
// kept up to date by Adam's update within a training call.
constexpr int kPackTile = 16 * 64;                        // uint2 of a 16-step tile
constexpr int kPackHid = 16 * kPackTile;                  // a hidden layer's
constexpr int kPackOut = (kMaxOut / 16) * kPackTile;      // the output layer's
constexpr int kPackTotal = 4 * kPackHid + 2 * kPackOut;
// start of layer l (1-3), forward or transposed (arithmetic: a table indexed by
// l would go to scratch)
__host__ __device__ constexpr int pack_f(int l) { return (l - 1) * 2 * kPackHid; }
__host__ __device__ constexpr int pack_b(int l) { return pack_f(l) + (l < 3 ? kPackHid : kPackOut); }
// place of W[m][n] of layer l in shorts
__device__ __forceinline__ int pack_fwd(int l, int m, int n) {
  return 4 * (pack_f(l) + ((n >> 4) * 16 + (m >> 4)) * 64 + ((m >> 2) & 3) * 16 + (n & 15)) + (m & 3);
}
__device__ __forceinline__ int pack_bwd(int l, int m, int n) {
  return 4 * (pack_b(l) + ((m >> 4) * (l < 3 ? 16 : kMaxOut / 16) + (n >> 4)) * 64 + ((n >> 2) & 3) * 16 + (m & 15)) +
         (n & 3);
}

__global__ void __launch_bounds__(256) k_emu_pack(const float* __restrict__ params, int n_out, uint2* __restrict__ pk) {
  const Offs o = param_offsets(n_out);
  const int i = blockIdx.x * 256 + threadIdx.x;  // kPackTotal is a multiple of 256, and so is every part
  const int l = i < pack_f(2) ? 1 : i < pack_f(3) ? 2 : 3;
  const bool fwd = i < pack_b(l);
  const int e = i - (fwd ? pack_f(l) : pack_b(l)), lane = e & 63, steps = l == 3 && !fwd ? kMaxOut / 16 : 16;
  const int s = (e >> 6) & (steps - 1), t = (e >> 6) / steps, N = l < 3 ? kHid : n_out;
  const float* __restrict__ W = params + (l == 1 ? o.W[1] : l == 2 ? o.W[2] : o.W[3]);
  const int kk = 16 * s + 4 * (lane >> 4), c = 16 * t + (lane & 15);
  float v[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int m = fwd ? kk + q : c, n = fwd ? c : kk + q;
    v[q] = n < N ? W[m * N + n] : 0.0f;
  }
  pk[i] = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
}

struct RowArgs {
  const EmuHeader* h;
  const float* params;
  const uint2* pk;         // packed weights
  int n_out, B, Bp;        // Bp: B rounded up to whole blocks
  const float *x0, *tgt;   // standardised batch, or (null):
  const float *x, *y;      // raw rows (first + i) mod n
  int64_t n, first;
  float* x0s;              // the standardised inputs [B][4] of raw rows
  unsigned short* hT[3];   // hidden activations, bfloat16, [unit][Bp]
  unsigned short* dT[4];   // dZ2, dZ3 (entries 1, 2) and dY (3), bfloat16, [unit][Bp]
  float* d[4];             // dZ1..dZ3, dY, FP32 [B][units]
  double* lpart;           // squared misfit per block
};

// MFMA 16x16x16 operands: lane l supplies A row l % 16 and B column l % 16 at
// k = 4 (l / 16) .. + 3; result element r of lane l is row 4 (l / 16) + r,
// column l % 16.  A block takes 4 R rows of the batch, R = 1, 2 or 4: row
// R g + r is the product's row 4 g + r, r < R, and the products' other rows are
// not used (a row depends on its own A row alone).  Fewer rows a block leave
// matrix work idle but spread the erfc and exp of the activations over more
// CUs, and those cost more: at batch 512 R = 4 (32 blocks) takes 22.9 us,
// R = 1 (128 blocks) 18.8 us; see row_shape for the rule.  Wave w of a block owns the hidden units 32 w .. 32 w + 31
// (two column tiles) of every layer, so pre-activations stay in its registers
// until the backward pass needs them.  The weights of the next product are
// read before the barrier that the current one ends with.
template <int R>
__global__ void __launch_bounds__(kRowNT) k_emu_rows(RowArgs a) {
  constexpr int kRowT = 4 * R;
  __shared__ unsigned short sact[2][kRowT][kRowLd];
  __shared__ float sx[kRowT][kIn], st[kRowT][kMaxOut], smask[kMaxOut];
  __shared__ double sl[4];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6, c = lane & 15, kq = 4 * (lane >> 4), rq = R * (lane >> 4);
  const int ar = R * (c >> 2) + ((c & 3) < R ? c & 3 : R - 1);  // the batch row of this lane's A row
  const int n_out = a.n_out, row0 = blockIdx.x * kRowT;
  const Offs o = param_offsets(n_out);
  const float* __restrict__ P = a.params;
  const int col = 32 * wv + c;   // and col + 16
  uint2 w[2][16];   // B operands of this wave's two tiles
  auto load = [&](size_t at) {
    const uint2* __restrict__ f = a.pk + at + 2 * wv * 16 * 64 + lane;
#pragma unroll
    for (int s = 0; s < 16; ++s)
#pragma unroll
      for (int j = 0; j < 2; ++j) w[j][s] = f[(j * 16 + s) * 64];
  };
  v4f32 acc[2];
  auto product = [&](const unsigned short (*act)[kRowLd]) {
    acc[0] = acc[1] = v4f32{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      const v4i16 af = __builtin_bit_cast(v4i16, *reinterpret_cast<const uint2*>(&act[ar][16 * s + kq]));
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(af, __builtin_bit_cast(v4i16, w[j][s]), acc[j], 0, 0, 0);
    }
  };
  // this lane's R rows of unit u: bfloat16 into LDS (act) and [unit][Bp] (gT)
  auto put = [&](const float* v, int u, unsigned short (*act)[kRowLd], unsigned short* gT) {
    unsigned short b[4];
#pragma unroll
    for (int r = 0; r < R; r += 2) {
      const uint32_t p2 = pack_bf16(v[r], v[r + 1 < R ? r + 1 : r]);
      b[r] = static_cast<unsigned short>(p2);
      b[r + 1] = static_cast<unsigned short>(p2 >> 16);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) act[rq + r][u] = b[r];
    if (gT) {
      unsigned short* g = gT + static_cast<size_t>(u) * a.Bp + row0 + rq;
      if constexpr (R == 4) *reinterpret_cast<uint2*>(g) = make_uint2(b[0] | b[1] << 16, b[2] | b[3] << 16);
      else if constexpr (R == 2) *reinterpret_cast<uint32_t*>(g) = b[0] | b[1] << 16;
      else *g = b[0];
    }
  };
  load(pack_f(1));
  // the rows' inputs and targets (rows past the batch: 0)
  if (t < kRowT * kIn) {
    const int i = t / kIn, k = t % kIn, row = row0 + i;
    float v = 0.0f;
    if (row < a.B) {
      if (a.x0) {
        v = a.x0[row * kIn + k];
      } else {
        v = scale_input(a.h, k, a.x[((a.first + row) % a.n) * kIn + k]);
        a.x0s[row * kIn + k] = v;
      }
    }
    sx[i][k] = v;
  }
  if (t < kMaxOut) smask[t] = a.h->out_mask[t];
#pragma unroll
  for (int e = t; e < kRowT * kMaxOut; e += kRowNT) {
    const int i = e / kMaxOut, k = e % kMaxOut, row = row0 + i;
    float v = 0.0f;
    if (row < a.B && k < n_out) {
      if (a.x0) {
        v = a.tgt[static_cast<size_t>(row) * n_out + k];
      } else {
        v = a.y[((a.first + row) % a.n) * n_out + k];
        if (k >= a.h->log_from) v = logf(v);
        v = (v - a.h->out_mean[k]) / a.h->out_std[k];
        v = (a.h->out_mask[k] > 0.0f && isfinite(v)) ? v : 0.0f;
      }
    }
    st[i][k] = v;
  }
  __syncthreads();
  float z[3][2][R], v[2][R];
#pragma unroll
  for (int j = 0; j < 2; ++j) {  // layer 1 (FP32)
    const int u = col + 16 * j;
    const float b = P[o.b[0] + u];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      float s1 = 0.0f;
#pragma unroll
      for (int k = 0; k < kIn; ++k) s1 = fmaf(sx[rq + r][k], P[o.W[0] + k * kHid + u], s1);
      z[0][j][r] = s1 + b;
      v[j][r] = gelu(z[0][j][r]);
    }
    put(v[j], u, sact[0], a.hT[0]);
  }
  __syncthreads();
#pragma unroll
  for (int l = 1; l < 3; ++l) {
    product(sact[(l - 1) & 1]);
    if (l == 1) load(pack_f(2));
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const float b = P[o.b[l] + col + 16 * j];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        z[l][j][r] = acc[j][r] + b;
        v[j][r] = gelu(z[l][j][r]);
      }
      put(v[j], col + 16 * j, sact[l & 1], a.hT[l]);
    }
    __syncthreads();
  }
  load(pack_b(2));
  // output layer (waves 0-3, 16 columns each) and loss: h3 in sact[0]
  if (wv < 4) {
    const int u = 16 * wv + c;
    v4f32 y = {0.f, 0.f, 0.f, 0.f};
    if (16 * wv < n_out) {
      const uint2* __restrict__ f = a.pk + pack_f(3) + wv * 16 * 64 + lane;
      uint2 wo[16];
#pragma unroll
      for (int s = 0; s < 16; ++s) wo[s] = f[s * 64];
#pragma unroll
      for (int s = 0; s < 16; ++s) {
        const v4i16 af = __builtin_bit_cast(v4i16, *reinterpret_cast<const uint2*>(&sact[0][ar][16 * s + kq]));
        y = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(af, __builtin_bit_cast(v4i16, wo[s]), y, 0, 0, 0);
      }
    }
    float neff = 0.0f;
    for (int k = 0; k < n_out; ++k) neff += smask[k];
    const float scale = 2.0f / (static_cast<float>(a.B) * (neff > 0.0f ? neff : 1.0f));
    const float b = u < n_out ? P[o.b[3] + u] : 0.0f;
    double lsum = 0.0;
    float dy[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int row = row0 + rq + r;
      dy[r] = 0.0f;
      if (u < n_out && row < a.B) {
        const float yv = y[r] + b;
        const float d = (yv - st[rq + r][u]) * smask[u];
        dy[r] = scale * d;
        lsum += static_cast<double>(d) * d;
        a.d[3][static_cast<size_t>(row) * n_out + u] = dy[r];
      }
    }
    // sact[1] still holds h2, which no wave reads any more
    put(dy, u, sact[1], u < n_out ? a.dT[3] : nullptr);
    for (int k = 32; k >= 1; k >>= 1) lsum += __shfl_xor(lsum, k);
    if (lane == 0) sl[wv] = lsum;
  }
  __syncthreads();
  if (t == 0) a.lpart[blockIdx.x] = sl[0] + sl[1] + sl[2] + sl[3];
#pragma unroll
  for (int j = 0; j < 2; ++j) {  // dZ3 = (dY W4^T) gelu'(Z3)
    v4f32 e = {0.f, 0.f, 0.f, 0.f};
    const uint2* __restrict__ f = a.pk + pack_b(3) + (2 * wv + j) * (kMaxOut / 16) * 64 + lane;
#pragma unroll
    for (int s = 0; s < kMaxOut / 16; ++s) {
      if (16 * s >= n_out) break;
      const v4i16 af = __builtin_bit_cast(v4i16, *reinterpret_cast<const uint2*>(&sact[1][ar][16 * s + kq]));
      e = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(af, __builtin_bit_cast(v4i16, f[s * 64]), e, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) v[j][r] = e[r] * gelu_grad(z[2][j][r]);
    put(v[j], col + 16 * j, sact[0], a.dT[2]);
  }
#pragma unroll
  for (int l = 2; l >= 0; --l) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (row0 + rq + r < a.B) a.d[l][static_cast<size_t>(row0 + rq + r) * kHid + col + 16 * j] = v[j][r];
    if (l == 0) break;
    __syncthreads();
    product(sact[l & 1]);
    if (l == 2) load(pack_b(1));
#pragma unroll
    for (int j = 0; j < 2; ++j) {
#pragma unroll
      for (int r = 0; r < R; ++r) v[j][r] = acc[j][r] * gelu_grad(z[l - 1][j][r]);
      if (l == 2) put(v[j], col + 16 * j, sact[1], a.dT[1]);
    }
  }
}

struct GradArgs {
  const EmuHeader* h;
  int n_out, B, Bp, nparts;
  const float* x0;
  const unsigned short* hT[3];
  const unsigned short* dT[4];
  const float* d[4];
  const double* lpart;
  float* grad;   // gradients out, or
  AdamArgs adam; // (ADAM) the parameters updated in place
  unsigned short* pk;  // (ADAM) the packed weights, kept up to date
  float* loss;   // or null
};

// Grid of k_emu_grads: 16x16 tiles of the weight gradients of layers 2, 3, 4 (a
// wave each), then 16 columns a block of the bias gradients (with layer 1's
// weights), then one block for the loss.
struct GradGrid {
  int tiles4, tile_blocks, cols4, blocks;
};
__host__ __device__ inline GradGrid grad_grid(int n_out) {
  GradGrid g;
  g.tiles4 = 16 * ((n_out + 15) / 16);
  g.tile_blocks = (512 + g.tiles4) / 4;
  g.cols4 = (n_out + 15) / 16;
  g.blocks = g.tile_blocks + 3 * (kHid / 16) + g.cols4 + 1;
  return g;
}

template <bool ADAM>
__global__ void __launch_bounds__(256) k_emu_grads(GradArgs a) {
  __shared__ float sp[5][16][17];
  __shared__ double sl[256];
  const int t = threadIdx.x, lane = t & 63, n_out = a.n_out;
  const Offs o = param_offsets(n_out);
  const GradGrid gg = grad_grid(n_out);
  auto give = [&](size_t i, float g) {
    if constexpr (ADAM) return adam_update(a.adam, i, g);
    else return a.grad[i] = g;
  };
  int b = blockIdx.x;
  if (b < gg.tile_blocks) {
    // dW = H^T dZ over the batch, 16 rows per MFMA step in order; both operands
    // lie [unit][row], four consecutive rows per lane
    const int tile = 4 * b + (t >> 6), c = lane & 15, kq = 4 * (lane >> 4);
    const int l = tile < 256 ? 1 : tile < 512 ? 2 : 3, u = tile & 255;
    const int mt = l < 3 ? u >> 4 : u % 16, nt = l < 3 ? u & 15 : u / 16;
    const int N = l < 3 ? kHid : n_out, n = 16 * nt + c;
    // (arrays of the argument indexed by constants: by l they would go to scratch)
    const unsigned short* __restrict__ A =
        (l == 1 ? a.hT[0] : l == 2 ? a.hT[1] : a.hT[2]) + static_cast<size_t>(16 * mt + c) * a.Bp + kq;
    const unsigned short* __restrict__ D =
        (l == 1 ? a.dT[1] : l == 2 ? a.dT[2] : a.dT[3]) + static_cast<size_t>(n < N ? n : 0) * a.Bp + kq;
    const size_t wo = l == 1 ? o.W[1] : l == 2 ? o.W[2] : o.W[3];
    v4f32 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 16
    for (int k = 0; k < a.Bp; k += 16) {
      const uint2 av = *reinterpret_cast<const uint2*>(A + k);
      const uint2 dv = *reinterpret_cast<const uint2*>(D + k);
      acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(v4i16, av), __builtin_bit_cast(v4i16, dv),
                                                      acc, 0, 0, 0);
    }
    if (n < N) {
      float p[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) p[r] = give(wo + static_cast<size_t>(16 * mt + kq + r) * N + n, acc[r]);
      if constexpr (ADAM) {
        const uint2 u = make_uint2(pack_bf16(p[0], p[1]), pack_bf16(p[2], p[3]));
        const int m = 16 * mt + kq;
        *reinterpret_cast<uint2*>(a.pk + pack_fwd(l, m, n)) = u;
        a.pk[pack_bwd(l, m, n)] = static_cast<unsigned short>(u.x);
        a.pk[pack_bwd(l, m + 1, n)] = static_cast<unsigned short>(u.x >> 16);
        a.pk[pack_bwd(l, m + 2, n)] = static_cast<unsigned short>(u.y);
        a.pk[pack_bwd(l, m + 3, n)] = static_cast<unsigned short>(u.y >> 16);
      }
    }
    return;
  }
  b -= gg.tile_blocks;
  const int nb = kHid / 16;
  if (b < 3 * nb + gg.cols4) {
    // column sums: sixteen row groups (rows g, g + 16, ...) in order, then the
    // groups in a fixed tree; layer 1's weights alike (below 64 rows in one chain)
    const int l = b < 3 * nb ? b / nb : 3, N = l < 3 ? kHid : n_out;
    const int c = t & 15, g = t >> 4, n = 16 * (l < 3 ? b % nb : b - 3 * nb) + c;
    const float* __restrict__ d = l == 0 ? a.d[0] : l == 1 ? a.d[1] : l == 2 ? a.d[2] : a.d[3];
    const size_t bo = l == 0 ? o.b[0] : l == 1 ? o.b[1] : l == 2 ? o.b[2] : o.b[3];
    float s[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
    if (n < N) {
      if (l == 0) {
#pragma unroll 8
        for (int m = g; m < a.B; m += 16) {
          const float dv = d[static_cast<size_t>(m) * kHid + n];
          s[4] += dv;
#pragma unroll
          for (int i = 0; i < kIn; ++i) s[i] = fmaf(a.x0[m * kIn + i], dv, s[i]);
        }
        if (a.B < 64 && g < kIn) {
          float acc = 0.0f;
          for (int m = 0; m < a.B; ++m) acc = fmaf(a.x0[m * kIn + g], d[static_cast<size_t>(m) * kHid + n], acc);
          give(o.W[0] + static_cast<size_t>(g) * kHid + n, acc);
        }
      } else {
#pragma unroll 16
        for (int m = g; m < a.B; m += 16) s[4] += d[static_cast<size_t>(m) * N + n];
      }
    }
#pragma unroll
    for (int i = 0; i < 5; ++i) sp[i][g][c] = s[i];
    __syncthreads();
    for (int w = 8; w > 0; w >>= 1) {
      if (g < w)
#pragma unroll
        for (int i = 0; i < 5; ++i) sp[i][g][c] += sp[i][g + w][c];
      __syncthreads();
    }
    if (g == 0 && n < N) {
      give(bo + n, sp[4][0][c]);
      if (l == 0 && a.B >= 64)
#pragma unroll
        for (int i = 0; i < kIn; ++i) give(o.W[0] + static_cast<size_t>(i) * kHid + n, sp[i][0][c]);
    }
    return;
  }
  double l = 0.0;
  for (int i = t; i < a.nparts; i += 256) l += a.lpart[i];
  sl[t] = l;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w) sl[t] += sl[t + w];
    __syncthreads();
  }
  if (t == 0 && a.loss) a.loss[0] = static_cast<float>(sl[0] / (static_cast<double>(a.B) * emu_neff(a.h)));
}

// ---------------------------------------------------------------- small-batch FP32 forward (prediction)
// one block per group of up to 8 samples: each thread owns one hidden unit;
// outputs are un-standardised (exp for columns >= log_from)
__global__ void __launch_bounds__(256) k_emu_predict(const EmuHeader* __restrict__ h, const float* __restrict__ params,
                                                     const float* __restrict__ x, int64_t n, float* y) {
  __shared__ float hs[2][8][kHid];
  const int n_out = h->n_out;
  const Offs o = param_offsets(n_out);
  const int t = threadIdx.x;
  const int64_t s0 = static_cast<int64_t>(blockIdx.x) * 8;
  const int ns = n - s0 < 8 ? static_cast<int>(n - s0) : 8;
  float acc[8];
  // layer 1
  for (int s = 0; s < ns; ++s) {
    float a = params[o.b[0] + t];
    for (int i = 0; i < kIn; ++i) {
      const float u = scale_input(h, i, x[(s0 + s) * kIn + i]);
      a = fmaf(u, params[o.W[0] + i * kHid + t], a);
    }
    hs[0][s][t] = gelu(a);
  }
  __syncthreads();
  int cur = 0;
  for (int l = 1; l < 3; ++l) {
    for (int s = 0; s < ns; ++s) acc[s] = params[o.b[l] + t];
    for (int k = 0; k < kHid; ++k) {
      const float w = params[o.W[l] + static_cast<size_t>(k) * kHid + t];
      for (int s = 0; s < ns; ++s) acc[s] = fmaf(hs[cur][s][k], w, acc[s]);
    }
    for (int s = 0; s < ns; ++s) hs[cur ^ 1][s][t] = gelu(acc[s]);
    __syncthreads();
    cur ^= 1;
  }
  if (t < n_out) {
    for (int s = 0; s < ns; ++s) acc[s] = params[o.b[3] + t];
    for (int k = 0; k < kHid; ++k) {
      const float w = params[o.W[3] + static_cast<size_t>(k) * n_out + t];
      for (int s = 0; s < ns; ++s) acc[s] = fmaf(hs[cur][s][k], w, acc[s]);
    }
    for (int s = 0; s < ns; ++s) {
      float v = acc[s] * h->out_std[t] + h->out_mean[t];
      if (t >= h->log_from) v = expf(v);
      y[(s0 + s) * n_out + t] = v;
    }
  }
}

// ---------------------------------------------------------------- host side
struct TrainBufs {
  float *x0, *tgt, *z[3], *hh[3], *y, *dy, *dz[3], *grad, *loss;
  double* lpart;  // per-block loss partials
  size_t total;
};

static size_t al(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

static TrainBufs carve_train(char* w, int B, int n_out) {
  TrainBufs t{};
  size_t o = 0;
  auto take = [&](size_t nfloat) {
    float* p = w ? reinterpret_cast<float*>(w + o) : nullptr;
    o += al(nfloat * sizeof(float));
    return p;
  };
  t.x0 = take(static_cast<size_t>(B) * kIn);
  t.tgt = take(static_cast<size_t>(B) * n_out);
  for (int l = 0; l < 3; ++l) {
    t.z[l] = take(static_cast<size_t>(B) * kHid);
    t.hh[l] = take(static_cast<size_t>(B) * kHid);
    t.dz[l] = take(static_cast<size_t>(B) * kHid);
  }
  t.y = take(static_cast<size_t>(B) * n_out);
  t.dy = take(static_cast<size_t>(B) * n_out);
  t.grad = take(n_params(n_out));
  t.loss = take(1);
  t.lpart = reinterpret_cast<double*>(take(2 * ((static_cast<size_t>(B) * n_out + 255) / 256)));
  t.total = o;
  return t;
}

// Buffers of the bfloat16 path in the same workspace.
struct Bf16Bufs {
  float *x0s, *d[4];
  unsigned short *hT[3], *dT[4];
  double* lpart;
  uint2* pk;
  int Bp;
  size_t total;
};

static Bf16Bufs carve_bf16(char* w, int B, int n_out) {
  Bf16Bufs t{};
  t.Bp = (B + kRowPad - 1) / kRowPad * kRowPad;
  size_t o = 0;
  auto take = [&](size_t bytes) {
    char* p = w ? w + o : nullptr;
    o += al(bytes);
    return p;
  };
  t.lpart = reinterpret_cast<double*>(take(sizeof(double) * (t.Bp / 4)));
  t.pk = reinterpret_cast<uint2*>(take(sizeof(uint2) * kPackTotal));
  t.x0s = reinterpret_cast<float*>(take(sizeof(float) * kIn * B));
  for (int l = 0; l < 4; ++l) {
    const size_t units = l < 3 ? kHid : n_out;
    t.d[l] = reinterpret_cast<float*>(take(sizeof(float) * units * B));
    if (l > 0) t.dT[l] = reinterpret_cast<unsigned short*>(take(sizeof(unsigned short) * units * t.Bp));
    if (l < 3) t.hT[l] = reinterpret_cast<unsigned short*>(take(sizeof(unsigned short) * units * t.Bp));
  }
  t.total = o;
  return t;
}

// Rows per block of k_emu_rows (4 R): as few as leave no more blocks than CUs
// (a training step with R = 1, 2, 4: batch 1024 42, 44, 47 us; 2048 67, 61, 64
// us; 4096 122, 110, 95 us).
static int row_shape(int B) {
  const int blocks = (B + 3) / 4, cus = device_cus();
  return blocks <= cus ? 1 : blocks <= 2 * cus ? 2 : 4;
}

static size_t train_bytes(int B, int n_out) {
  const size_t a = carve_train(nullptr, B, n_out).total, b = carve_bf16(nullptr, B, n_out).total;
  return a > b ? a : b;
}

// FP32 forward and backward of one batch (x0, tgt already standardised); gradients
// into t.grad, loss into t.loss.
static hipError_t emu_fwd_bwd(const EmuHeader* h_dev, const float* params, int n_out, int B,
                              const TrainBufs& t, hipStream_t st) {
  const Offs o = param_offsets(n_out);
  hipError_t e;
  // forward
  if ((e = gemm<false, false>(B, kHid, kIn, t.x0, kIn, params + o.W[0], kHid, t.hh[0], kHid, params + o.b[0],
                              EPI_BIAS_GELU, t.z[0], kHid, st)) != hipSuccess) return e;
  for (int l = 1; l < 3; ++l)
    if ((e = gemm<false, false>(B, kHid, kHid, t.hh[l - 1], kHid, params + o.W[l], kHid, t.hh[l], kHid,
                                params + o.b[l], EPI_BIAS_GELU, t.z[l], kHid, st)) != hipSuccess) return e;
  if ((e = gemm<false, false>(B, n_out, kHid, t.hh[2], kHid, params + o.W[3], n_out, t.y, n_out,
                              params + o.b[3], EPI_BIAS, nullptr, 0, st)) != hipSuccess) return e;
  {
    const int nparts = (B * n_out + 255) / 256;
    hipLaunchKernelGGL(k_emu_dloss, dim3(nparts), dim3(256), 0, st, t.y, t.tgt, B, h_dev, t.dy, t.lpart);
    hipLaunchKernelGGL(k_emu_loss, dim3(1), dim3(256), 0, st, t.lpart, nparts, B, h_dev, t.loss);
  }
  // backward: output layer
  if ((e = gemm<true, false>(kHid, n_out, B, t.hh[2], kHid, t.dy, n_out, t.grad + o.W[3], n_out, nullptr,
                             EPI_STORE, nullptr, 0, st)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_colsum, dim3((n_out + 63) / 64), dim3(1024), 0, st, t.dy, B, n_out, t.grad + o.b[3]);
  // dZ3 = (dY W4^T) * gelu'(Z3)
  if ((e = gemm<false, true>(B, kHid, n_out, t.dy, n_out, params + o.W[3], n_out, t.dz[2], kHid, nullptr,
                             EPI_GELU_GRAD, t.z[2], kHid, st)) != hipSuccess) return e;
  for (int l = 2; l >= 1; --l) {
    if ((e = gemm<true, false>(kHid, kHid, B, t.hh[l - 1], kHid, t.dz[l], kHid, t.grad + o.W[l], kHid, nullptr,
                               EPI_STORE, nullptr, 0, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_colsum, dim3(kHid / 64), dim3(1024), 0, st, t.dz[l], B, kHid, t.grad + o.b[l]);
    if ((e = gemm<false, true>(B, kHid, kHid, t.dz[l], kHid, params + o.W[l], kHid, t.dz[l - 1], kHid, nullptr,
                               EPI_GELU_GRAD, t.z[l - 1], kHid, st)) != hipSuccess) return e;
  }
  if ((e = gemm<true, false>(kIn, kHid, B, t.x0, kIn, t.dz[0], kHid, t.grad + o.W[0], kHid, nullptr,
                             EPI_STORE, nullptr, 0, st)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_colsum, dim3(kHid / 64), dim3(1024), 0, st, t.dz[0], B, kHid, t.grad + o.b[0]);
  return hipGetLastError();
}

// The packed weights of the bfloat16 path, from the parameters.
static hipError_t emu_pack(const float* params, int n_out, int B, char* w, hipStream_t st) {
  hipLaunchKernelGGL(k_emu_pack, dim3(kPackTotal / 256), dim3(256), 0, st, params, n_out,
                     carve_bf16(w, B, n_out).pk);
  return hipGetLastError();
}

// The same in bfloat16 MFMA products (k_emu_rows, k_emu_grads): the batch is
// (x0, tgt), or with x0 null the raw rows (first + i) mod n of (x, y).  Adam's
// update of the parameters where adam is given, else gradients into grad.
static hipError_t emu_batch_bf16(const EmuHeader* h_dev, const float* params, int n_out, int B, char* w,
                                 const float* x0, const float* tgt, const float* x, const float* y, int64_t n,
                                 int64_t first, float* grad, const AdamArgs* adam, float* loss, hipStream_t st) {
  const Bf16Bufs t = carve_bf16(w, B, n_out);
  RowArgs r{};
  r.h = h_dev;
  r.params = params;
  r.pk = t.pk;
  r.n_out = n_out;
  r.B = B;
  r.Bp = t.Bp;
  r.x0 = x0;
  r.tgt = tgt;
  r.x = x;
  r.y = y;
  r.n = n;
  r.first = first;
  r.x0s = t.x0s;
  r.lpart = t.lpart;
  GradArgs g{};
  g.h = h_dev;
  g.n_out = n_out;
  g.B = B;
  g.Bp = t.Bp;
  const int R = row_shape(B);
  const dim3 rows(t.Bp / (4 * R));
  g.nparts = t.Bp / (4 * R);
  g.x0 = x0 ? x0 : t.x0s;
  g.lpart = t.lpart;
  g.grad = grad;
  g.pk = reinterpret_cast<unsigned short*>(t.pk);
  if (adam) g.adam = *adam;
  g.loss = loss;
  for (int l = 0; l < 4; ++l) {
    if (l < 3) g.hT[l] = r.hT[l] = t.hT[l];
    g.dT[l] = r.dT[l] = t.dT[l];
    g.d[l] = r.d[l] = t.d[l];
  }
  if (R == 1)
    hipLaunchKernelGGL(k_emu_rows<1>, rows, dim3(kRowNT), 0, st, r);
  else if (R == 2)
    hipLaunchKernelGGL(k_emu_rows<2>, rows, dim3(kRowNT), 0, st, r);
  else
    hipLaunchKernelGGL(k_emu_rows<4>, rows, dim3(kRowNT), 0, st, r);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 grid(grad_grid(n_out).blocks);
  if (adam)
    hipLaunchKernelGGL(k_emu_grads<true>, grid, dim3(256), 0, st, g);
  else
    hipLaunchKernelGGL(k_emu_grads<false>, grid, dim3(256), 0, st, g);
  return hipGetLastError();
}

size_t emulator_bytes(int n_out) { return kHeaderBytes + 3 * al(n_params(n_out) * sizeof(float)); }
static float* emu_params(void* emu) { return reinterpret_cast<float*>(static_cast<char*>(emu) + kHeaderBytes); }
static const float* emu_params(const void* emu) {
  return reinterpret_cast<const float*>(static_cast<const char*>(emu) + kHeaderBytes);
}

size_t emulator_eval_bytes() { return 1024; }

// ---------------------------------------------------------------- device-side tuning search
constexpr int kSearchNT = 1024;
constexpr int kLmS = 3;  // samples per batched forward pass: a point and two difference steps

struct SearchArgs {
  const EmuHeader* h;
  const float* params;
  double fbar_t, c, z, x0[2], xk[2], step, xatol, fatol, sigma;
  int nk, max_evals;
  // small-scale power mode (ps = 1): th = (ln amp, ln kcut) of P_s, emulator
  // inputs (a, b, amp, kcut) with sigma_g^2 = sig0 + sigma_s^2(amp, kcut; dpix),
  // (ln a, ln s) = lin[0..1] + lin[2..3] (ln sigma_g - lin[4]) and b = s / sigma_g
  int ps;
  double sig0, dpix, lin[5];
  double pk_t[kMaxOut];
  double off[kMaxOut];       // model offset per statistic (Fbar first)
  double jac[kMaxOut][2];    // model slope per statistic in (ln a, ln b) about xk
  double* out;               // x[2], best objective, evaluations, raw prediction [1 + nk] at x
};

// Forward passes of ns <= kLmS inputs by a block of kSearchNT threads sharing
// every weight load (hidden layers: float4 loads of four units, sixteen
// threads per unit group; output layer: sixteen threads per column); raw
// outputs (exp for columns >= log_from) into outv[s].
__device__ void forward_batch(const EmuHeader* __restrict__ h, const float* __restrict__ params, const Offs& o,
                              const float (*xin)[4], int ns, float (*hs)[kLmS][kHid], float* part,
                              float (*outv)[kMaxOut]) {
  const int t = threadIdx.x, n_out = h->n_out;
  if (t < kHid) {
    const float b0 = params[o.b[0] + t];
    for (int s = 0; s < ns; ++s) {
      float a = b0;
#pragma unroll
      for (int i = 0; i < kIn; ++i) a = fmaf(scale_input(h, i, xin[s][i]), params[o.W[0] + i * kHid + t], a);
      hs[0][s][t] = gelu(a);
    }
  }
  __syncthreads();
  int cur = 0;
  // hidden layers: thread = four consecutive units (one float4 weight load per
  // k) x a sixteenth of the inner sum; the sixteen partial sums are added in
  // a fixed order
  const int ug = t & 63, kg = t >> 6;
  for (int l = 1; l < 3; ++l) {
    float acc[kLmS][4] = {};
    const float4* W = reinterpret_cast<const float4*>(params + o.W[l]) + ug;
#pragma unroll 8
    for (int k = 16 * kg; k < 16 * kg + 16; ++k) {
      const float4 w = W[static_cast<size_t>(k) * (kHid / 4)];
#pragma unroll
      for (int s = 0; s < kLmS; ++s) {
        if (s < ns) {
          const float hv = hs[cur][s][k];
          acc[s][0] = fmaf(hv, w.x, acc[s][0]);
          acc[s][1] = fmaf(hv, w.y, acc[s][1]);
          acc[s][2] = fmaf(hv, w.z, acc[s][2]);
          acc[s][3] = fmaf(hv, w.w, acc[s][3]);
        }
      }
    }
#pragma unroll
    for (int s = 0; s < kLmS; ++s)
#pragma unroll
      for (int j = 0; j < 4; ++j) part[(kg * kLmS + s) * kHid + 4 * ug + j] = acc[s][j];
    __syncthreads();
    if (t < kHid) {
      const float bl = params[o.b[l] + t];
      for (int s = 0; s < ns; ++s) {
        float v = 0.0f;
        for (int i = 0; i < 16; ++i) v += part[(i * kLmS + s) * kHid + t];
        hs[cur ^ 1][s][t] = gelu(bl + v);
      }
    }
    __syncthreads();
    cur ^= 1;
  }
  const int oc = t & 63, r = t >> 6;  // column, sixteenth of the sum
  float acc[kLmS] = {0.0f, 0.0f, 0.0f};
  if (oc < n_out) {
    const float* W = params + o.W[3] + oc;
#pragma unroll
    for (int k = 16 * r; k < 16 * r + 16; ++k) {
      const float w = W[static_cast<size_t>(k) * n_out];
#pragma unroll
      for (int s = 0; s < kLmS; ++s)
        if (s < ns) acc[s] = fmaf(hs[cur][s][k], w, acc[s]);
    }
  }
#pragma unroll
  for (int s = 0; s < kLmS; ++s) part[(r * kLmS + s) * 64 + oc] = acc[s];
  __syncthreads();
  if (t < n_out) {
    for (int s = 0; s < ns; ++s) {
      float v = 0.0f;
      for (int i = 0; i < 16; ++i) v += part[(i * kLmS + s) * 64 + t];
      v = (params[o.b[3] + t] + v) * h->out_std[t] + h->out_mean[t];
      if (t >= h->log_from) v = expf(v);
      outv[s][t] = v;
    }
  }
  __syncthreads();
}

// Levenberg-Marquardt over th = (ln a, ln b) on the residuals of the model
//   stat(th) = emulator(th) + off + jac (th - xk),
//   r_0 = (stat_0 - Fbar_t)/(s Fbar_t), r_{1+b} = (stat_{1+b} - P_t,b)/(s P_t,b)
// (0 where the target or the value is not finite; chi^2 = sum r^2), entirely
// on the device in one block.  In the small-scale power mode th = (ln amp,
// ln kcut) of P_s instead, a and b follow from th (SearchArgs), and only the
// P1D residuals count (Fbar is fixed by a and b sigma_g).  Each iteration runs one batched forward pass at
// the trial point and its two forward-difference steps (h = 1e-3), so the
// Jacobian of an accepted point comes with it.  Wave 0 forms the residuals
// (one statistic per lane) and the 2x2 normal equations (fixed-order shuffle
// sums); lane 0 steps the search and broadcasts through LDS.  Trial points
// outside the emulator's (a, b) input range are rejected like uphill steps.
// Stops when an accepted step is below xatol in both coordinates, when the
// damping exceeds 1e10, or after max_evals forward samples.
__global__ void __launch_bounds__(kSearchNT) k_emu_search(SearchArgs a) {
  __shared__ float hs[2][kLmS][kHid];
  __shared__ float part[16 * kLmS * kHid];
  __shared__ float outv[kLmS][kMaxOut];
  __shared__ double strial[2];
  __shared__ int sstate;  // 0 evaluate strial, 1 done
  const Offs o = param_offsets(a.h->n_out);
  const int nk = a.nk, t = threadIdx.x;
  // the emulator's input ranges in logarithms; a non-positive lower limit
  // leaves that side open
  auto lnlim = [](float v) { return v > 0.0f ? log(static_cast<double>(v)) : -HUGE_VAL; };
  double lo[4], hi[4];
  for (int i = 0; i < 4; ++i) {
    lo[i] = lnlim(a.h->in_lo[i]);
    hi[i] = log(static_cast<double>(a.h->in_hi[i]));
  }
  constexpr double kH = 1e-3;
  // emulator inputs at th: (a, b, c, z), or (a, b, amp, kcut) in the
  // small-scale power mode, with (ln a, ln b) returned for the range check
  auto inputs = [&](double p0, double p1, float* x, double* lab) {
    if (!a.ps) {
      x[0] = static_cast<float>(exp(p0));
      x[1] = static_cast<float>(exp(p1));
      x[2] = static_cast<float>(a.c);
      x[3] = static_cast<float>(a.z);
      lab[0] = p0;
      lab[1] = p1;
      return;
    }
    const double amp = exp(p0), kc = exp(p1);
    const double ss2 = amp * kc * erf(M_PI / (a.dpix * kc)) / (2.0 * sqrt(M_PI));
    const double lsg = 0.5 * log(a.sig0 + ss2);
    lab[0] = a.lin[0] + a.lin[2] * (lsg - a.lin[4]);
    lab[1] = a.lin[1] + a.lin[3] * (lsg - a.lin[4]) - lsg;
    x[0] = static_cast<float>(exp(lab[0]));
    x[1] = static_cast<float>(exp(lab[1]));
    x[2] = static_cast<float>(amp);
    x[3] = static_cast<float>(kc);
  };
  // lane-0 state
  double th[2] = {a.x0[0], a.x0[1]}, chi2 = HUGE_VAL, lam = 1e-3, A00 = 0, A01 = 0, A11 = 0, g0 = 0, g1 = 0;
  bool have = false;
  int nev = 0;
  if (t == 0) {
    strial[0] = th[0];
    strial[1] = th[1];
    sstate = 0;
  }
  __syncthreads();
  const int max_iter = a.max_evals / kLmS + 1;
  for (int it = 0; it < max_iter + 1; ++it) {
    const double p0 = strial[0], p1 = strial[1];
    const int state = sstate;
    float xin[kLmS][4];
    double lab[2], lab1[2];
    inputs(p0, p1, xin[0], lab);
    inputs(p0 + kH, p1, xin[1], lab1);
    inputs(p0, p1 + kH, xin[2], lab1);
    forward_batch(a.h, a.params, o, xin, state ? 1 : kLmS, hs, part, outv);
    if (state) break;  // the last pass: the raw prediction at the optimum
    if (t < 64) {
      double r = 0.0, j0 = 0.0, j1 = 0.0;
      const int i = t;
      if (i <= nk && !(a.ps && i == 0)) {
        const double tgt = i == 0 ? a.fbar_t : a.pk_t[i - 1];
        const double inv = 1.0 / (a.sigma * tgt);
        const double d0 = p0 - a.xk[0], d1 = p1 - a.xk[1];
        const double lin = a.off[i] + a.jac[i][0] * d0 + a.jac[i][1] * d1;
        const double m = static_cast<double>(outv[0][i]) + lin;
        const double ma = static_cast<double>(outv[1][i]) + lin + a.jac[i][0] * kH;
        const double mb = static_cast<double>(outv[2][i]) + lin + a.jac[i][1] * kH;
        if (isfinite(tgt) && isfinite(m) && isfinite(ma) && isfinite(mb)) {
          r = (m - tgt) * inv;
          j0 = (ma - m) * inv / kH;
          j1 = (mb - m) * inv / kH;
        }
      }
      double c2 = r * r, s00 = j0 * j0, s01 = j0 * j1, s11 = j1 * j1, q0 = j0 * r, q1 = j1 * r;
#pragma unroll
      for (int w = 32; w >= 1; w >>= 1) {
        c2 += __shfl_xor(c2, w);
        s00 += __shfl_xor(s00, w);
        s01 += __shfl_xor(s01, w);
        s11 += __shfl_xor(s11, w);
        q0 += __shfl_xor(q0, w);
        q1 += __shfl_xor(q1, w);
      }
      if (t == 0) {
        nev += kLmS;
        bool inside = lab[0] >= lo[0] && lab[0] <= hi[0] && lab[1] >= lo[1] && lab[1] <= hi[1];
        if (a.ps) inside = inside && p0 >= lo[2] && p0 <= hi[2] && p1 >= lo[3] && p1 <= hi[3];
        bool done = false;
        if (inside && c2 < chi2) {  // accept the point (and its Jacobian)
          const double step = have ? fmax(fabs(p0 - th[0]), fabs(p1 - th[1])) : HUGE_VAL;
          th[0] = p0;
          th[1] = p1;
          chi2 = c2;
          A00 = s00;
          A01 = s01;
          A11 = s11;
          g0 = q0;
          g1 = q1;
          lam = fmax(lam / 3.0, 1e-12);
          have = true;
          if (step <= a.xatol) done = true;
        } else {
          lam *= 4.0;
          if (lam > 1e10) done = true;
        }
        if (!have) done = true;  // the start itself is unusable
        if (nev + kLmS > a.max_evals) done = true;
        double n0 = th[0], n1 = th[1];
        if (!done) {  // (A + lam diag A) delta = -g
          const double m00 = A00 * (1.0 + lam) + 1e-300, m11 = A11 * (1.0 + lam) + 1e-300, m01 = A01;
          const double det = m00 * m11 - m01 * m01;
          if (!(det > 0.0) || !isfinite(det)) {
            done = true;
          } else {
            n0 = th[0] + (-g0 * m11 + g1 * m01) / det;
            n1 = th[1] + (-g1 * m00 + g0 * m01) / det;
          }
        }
        strial[0] = done ? th[0] : n0;
        strial[1] = done ? th[1] : n1;
        sstate = done ? 1 : 0;
      }
    }
    __syncthreads();
  }
  if (t == 0) {
    a.out[0] = th[0];
    a.out[1] = th[1];
    a.out[2] = chi2;
    a.out[3] = static_cast<double>(nev);
  }
  if (t <= nk) a.out[4 + t] = static_cast<double>(outv[0][t]);
}

hipError_t emulator_search(const void* emu, const EmuSearchSpec& sp, double x[2], double* fbest, int* nev,
                           double* pred, char* scratch, hipStream_t st) {
  if (!emu || sp.nk < 0 || sp.nk + 1 > kMaxOut) return hipErrorInvalidValue;
  SearchArgs a{};
  a.h = static_cast<const EmuHeader*>(emu);
  a.params = emu_params(emu);
  a.fbar_t = sp.fbar_t;
  a.c = sp.c;
  a.z = sp.z;
  a.x0[0] = x[0];
  a.x0[1] = x[1];
  a.xk[0] = sp.xk[0];
  a.xk[1] = sp.xk[1];
  a.step = sp.step;
  a.xatol = sp.xatol;
  a.fatol = sp.fatol;
  a.sigma = sp.sigma;
  a.nk = sp.nk;
  a.max_evals = sp.max_evals;
  a.ps = sp.ps;
  a.sig0 = sp.sig0;
  a.dpix = sp.dpix;
  for (int i = 0; i < 5; ++i) a.lin[i] = sp.lin[i];
  for (int i = 0; i <= sp.nk; ++i) {
    if (i < sp.nk) a.pk_t[i] = sp.pk_t[i];
    a.off[i] = sp.off[i];
    a.jac[i][0] = sp.jac[2 * i];
    a.jac[i][1] = sp.jac[2 * i + 1];
  }
  a.out = reinterpret_cast<double*>(scratch);
  hipLaunchKernelGGL(k_emu_search, dim3(1), dim3(kSearchNT), 0, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  double hout[4 + kMaxOut];
  if ((e = hipMemcpyAsync(hout, a.out, sizeof(double) * (5 + sp.nk), hipMemcpyDeviceToHost, st)) != hipSuccess)
    return e;
  if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
  x[0] = hout[0];
  x[1] = hout[1];
  *fbest = hout[2];
  *nev = static_cast<int>(hout[3]);
  for (int i = 0; i <= sp.nk; ++i) pred[i] = hout[4 + i];
  return hipSuccess;
}

}  // namespace lya

// ---------------------------------------------------------------- C-ABI
namespace {
thread_local char g_emu_err[256] = "";
int efail(int code, const char* msg) {
  snprintf(g_emu_err, sizeof(g_emu_err), "%s", msg);
  return code;
}
}  // namespace

extern "C" {

const char* lya_emulator_last_error(void) { return g_emu_err; }

size_t lya_emulator_bytes(int32_t n_out) {
  if (n_out < 1 || n_out > lya::kMaxOut) return 0;
  return lya::emulator_bytes(n_out);
}

size_t lya_emulator_param_offset(void) { return lya::kHeaderBytes; }
size_t lya_emulator_param_count(int32_t n_out) {
  return (n_out < 1 || n_out > lya::kMaxOut) ? 0 : lya::n_params(n_out);
}

int lya_emulator_init(void* emu, int32_t n_out, int32_t log_from, uint64_t seed, const double in_lo[4],
                      const double in_hi[4], int32_t log_inputs, void* stream) {
  if (!emu || n_out < 1 || n_out > lya::kMaxOut || !in_lo || !in_hi || log_from < 0 || log_inputs < 0 ||
      log_inputs > 15)
    return efail(LYA_EINVAL, "invalid emulator arguments");
  for (int i = 0; i < 4; ++i) {
    if (!(in_hi[i] > in_lo[i])) return efail(LYA_EINVAL, "input ranges must be increasing");
    if (((log_inputs >> i) & 1) && !(in_lo[i] > 0.0)) return efail(LYA_EINVAL, "log-scaled inputs need lo > 0");
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
  lya::EmuHeader h{};
  h.n_out = n_out;
  h.log_from = log_from;
  h.in_log = log_inputs;
  for (int i = 0; i < 4; ++i) {
    h.in_lo[i] = static_cast<float>(in_lo[i]);
    h.in_hi[i] = static_cast<float>(in_hi[i]);
    const bool lg = (log_inputs >> i) & 1;
    const double lo = lg ? log(in_lo[i]) : in_lo[i], hi = lg ? log(in_hi[i]) : in_hi[i];
    h.in_mul[i] = static_cast<float>(2.0 / (hi - lo));
    h.in_add[i] = static_cast<float>(-(hi + lo) / (hi - lo));
  }
  for (int o = 0; o < lya::kMaxOut; ++o) {
    h.out_mean[o] = 0.0f;
    h.out_std[o] = 1.0f;
    h.out_mask[o] = o < n_out ? 1.0f : 0.0f;
  }
  hipError_t e = hipMemcpyAsync(emu, &h, sizeof(h), hipMemcpyHostToDevice, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) return efail(LYA_EHIP, hipGetErrorString(e));
  const size_t np = lya::n_params(n_out);
  float* p = lya::emu_params(emu);
  const size_t stride = lya::al(np * sizeof(float)) / sizeof(float);
  hipLaunchKernelGGL(lya::k_emu_init, dim3(256), dim3(256), 0, st, p, p + stride, p + 2 * stride, n_out, seed);
  e = hipGetLastError();
  if (e != hipSuccess) return efail(LYA_EHIP, hipGetErrorString(e));
  return LYA_OK;
}

size_t lya_emulator_train_workspace_size(int32_t batch, int32_t n_out) {
  if (batch < 1 || n_out < 1 || n_out > lya::kMaxOut) return 0;
  return lya::train_bytes(batch, n_out);
}

int lya_emulator_set_scaling(void* emu, const float* y, int64_t n, void* stream) {
  if (!emu || !y || n < 1) return efail(LYA_EINVAL, "invalid scaling arguments");
  hipStream_t st = static_cast<hipStream_t>(stream);
  lya::EmuHeader h;
  hipError_t e = hipMemcpyAsync(&h, emu, sizeof(h), hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) return efail(LYA_EHIP, hipGetErrorString(e));
  hipLaunchKernelGGL(lya::k_emu_stats, dim3(h.n_out), dim3(256), 0, st, y, n, h.n_out, h.log_from,
                     static_cast<lya::EmuHeader*>(emu));
  e = hipGetLastError();
  return e == hipSuccess ? LYA_OK : efail(LYA_EHIP, hipGetErrorString(e));
}

int lya_emulator_loss_grad(const void* emu, const float* x0, const float* t, int32_t batch, int32_t use_bf16,
                           float* grad, float* loss, void* work, size_t work_bytes, void* stream) {
  if (!emu || !x0 || !t || batch < 1 || !grad) return efail(LYA_EINVAL, "invalid gradient arguments");
  hipStream_t st = static_cast<hipStream_t>(stream);
  lya::EmuHeader h;
  hipError_t e = hipMemcpyAsync(&h, emu, sizeof(h), hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) return efail(LYA_EHIP, hipGetErrorString(e));
  lya::TrainBufs tb = lya::carve_train(static_cast<char*>(work), batch, h.n_out);
  if (!work || work_bytes < lya::train_bytes(batch, h.n_out))
    return efail(LYA_EWORKSPACE, "workspace too small for the emulator batch");
  if (use_bf16) {
    e = lya::emu_pack(lya::emu_params(emu), h.n_out, batch, static_cast<char*>(work), st);
    if (e == hipSuccess)
      e = lya::emu_batch_bf16(static_cast<const lya::EmuHeader*>(emu), lya::emu_params(emu), h.n_out, batch,
                              static_cast<char*>(work), x0, t, nullptr, nullptr, 0, 0, grad, nullptr, loss, st);
    return e == hipSuccess ? LYA_OK : efail(LYA_EHIP, hipGetErrorString(e));
  }
  const size_t np = lya::n_params(h.n_out);
  e = hipMemcpyAsync(tb.x0, x0, sizeof(float) * batch * lya::kIn, hipMemcpyDeviceToDevice, st);
  if (e == hipSuccess) e = hipMemcpyAsync(tb.tgt, t, sizeof(float) * batch * h.n_out, hipMemcpyDeviceToDevice, st);
  if (e == hipSuccess)
    e = lya::emu_fwd_bwd(static_cast<const lya::EmuHeader*>(emu), lya::emu_params(emu), h.n_out, batch, tb, st);
  if (e == hipSuccess) e = hipMemcpyAsync(grad, tb.grad, sizeof(float) * np, hipMemcpyDeviceToDevice, st);
  if (e == hipSuccess && loss) e = hipMemcpyAsync(loss, tb.loss, sizeof(float), hipMemcpyDeviceToDevice, st);
  return e == hipSuccess ? LYA_OK : efail(LYA_EHIP, hipGetErrorString(e));
}

int lya_emulator_train(void* emu, const float* x, const float* y, int64_t n, int32_t steps, int32_t batch,
                       double lr, int32_t use_bf16, float* loss_hist, void* work, size_t work_bytes, void* stream) {
  if (!emu || !x || !y || n < 1 || steps < 0 || batch < 1 || !(lr > 0.0))
    return efail(LYA_EINVAL, "invalid training arguments");
  hipStream_t st = static_cast<hipStream_t>(stream);
  lya::EmuHeader h;
  hipError_t e = hipMemcpyAsync(&h, emu, sizeof(h), hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) return efail(LYA_EHIP, hipGetErrorString(e));
  lya::TrainBufs tb = lya::carve_train(static_cast<char*>(work), batch, h.n_out);
  if (!work || work_bytes < lya::train_bytes(batch, h.n_out))
    return efail(LYA_EWORKSPACE, "workspace too small for the emulator batch");
  const size_t np = lya::n_params(h.n_out);
  float* p = lya::emu_params(emu);
  const size_t stride = lya::al(np * sizeof(float)) / sizeof(float);
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  int step = h.step;
  if (use_bf16 && steps > 0) {
    e = lya::emu_pack(p, h.n_out, batch, static_cast<char*>(work), st);
    if (e != hipSuccess) return efail(LYA_EHIP, hipGetErrorString(e));
  }
  for (int s = 0; s < steps; ++s) {
    const float bc1 = 1.0f - powf(b1, static_cast<float>(step + 1));
    const float bc2 = 1.0f - powf(b2, static_cast<float>(step + 1));
    const lya::AdamArgs adam{p, p + stride, p + 2 * stride, static_cast<float>(lr), b1, b2, eps, bc1, bc2};
    const lya::EmuHeader* hd = static_cast<const lya::EmuHeader*>(emu);
    if (use_bf16) {
      e = lya::emu_batch_bf16(hd, p, h.n_out, batch, static_cast<char*>(work), nullptr, nullptr, x, y, n,
                              static_cast<int64_t>(step) * batch, nullptr, &adam, loss_hist ? loss_hist + s : nullptr,
                              st);
      if (e != hipSuccess) return efail(LYA_EHIP, hipGetErrorString(e));
    } else {
      hipLaunchKernelGGL(lya::k_emu_gather, dim3(64), dim3(256), 0, st, x, y, n, static_cast<int64_t>(step), batch, hd,
                         tb.x0, tb.tgt);
      e = lya::emu_fwd_bwd(hd, p, h.n_out, batch, tb, st);
      if (e != hipSuccess) return efail(LYA_EHIP, hipGetErrorString(e));
      hipLaunchKernelGGL(lya::k_adam, dim3(512), dim3(256), 0, st, adam, tb.grad, np);
      if (loss_hist) {
        e = hipMemcpyAsync(loss_hist + s, tb.loss, sizeof(float), hipMemcpyDeviceToDevice, st);
        if (e != hipSuccess) return efail(LYA_EHIP, hipGetErrorString(e));
      }
    }
    ++step;
  }
  e = hipMemcpyAsync(reinterpret_cast<char*>(emu) + offsetof(lya::EmuHeader, step), &step, sizeof(step),
                     hipMemcpyHostToDevice, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e == hipSuccess) e = hipGetLastError();
  return e == hipSuccess ? LYA_OK : efail(LYA_EHIP, hipGetErrorString(e));
}

int lya_emulator_predict(const void* emu, const float* x, int64_t n, float* y, void* stream) {
  if (!emu || !x || !y || n < 0) return efail(LYA_EINVAL, "invalid prediction arguments");
  if (n == 0) return LYA_OK;
  hipStream_t st = static_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(lya::k_emu_predict, dim3(static_cast<unsigned>((n + 7) / 8)), dim3(256), 0, st,
                     static_cast<const lya::EmuHeader*>(emu), lya::emu_params(emu), x, n, y);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? LYA_OK : efail(LYA_EHIP, hipGetErrorString(e));
}

}  // extern "C"
