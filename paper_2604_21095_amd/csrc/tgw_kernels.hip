// gfx950 kernels of the phenotype-panel linear association scan.
//
//  gram_*_kernel      FP64 orthonormal basis Q of [1 | C] by Cholesky twice
//                     (Methods 2.2: Q spans the covariate space and has
//                     orthonormal columns)
//  qr_*_kernel        the same by Householder QR, for ill-conditioned covariates
//  prep_*_kernel      Eq. 1 + column standardization, once per panel, FP64;
//                     writes the contraction operand (FP32 or hi + lo);
//                     prep_kernel alone for cohorts of under 4,096 samples
//  table_kernel       -log10 p nodes for |t| in [0, 40] at the panel's df
//  stats_kernel       exact integer per-marker counts -> mean, ||g_c||^2,
//                     re-centring constant and the 2-bit decode table
//  gemm_wide_kernel,  the contraction of Eq. 2 on the matrix cores with the
//  gemm_kernel        fused epilogue (r, t of Eq. 3, beta, SE, -log10 p);
//                     small tiles and Q^T g are in tgw_small.hip
//  redo_kernel        FP64 path of covariate-collinear markers
//  finalize_kernel    ||g_res||^2 = ||g_c||^2 - sum_k (q_k^T g)^2
//  tail_kernel        FP64 -log10 p for |t| > 40
#include "tgw_device.h"

namespace tgw {

// ---------------------------------------------------------------------------
// FP64 Student-t tail: ln of the two-sided p-value
//   p = I_x(df/2, 1/2), x = df / (df + t^2)
// I_x(a, b) = x^a (1 - x)^b / (a B(a, b)) * F, F the continued fraction of
// the incomplete beta function (Abramowitz & Stegun 26.5.8), evaluated with
// the modified Lentz method; valid for x < (a + 1) / (a + b + 2), otherwise
// I_x(a, b) = 1 - I_{1-x}(b, a).
// ---------------------------------------------------------------------------
__device__ double beta_cf(double x, double a, double b) {
  const double tiny = 1e-300, eps = 4e-16;
  double f = tiny, c = tiny, d = 0.0;
  for (int j = 0; j < 20000; ++j) {
    double num;
    if (j == 0) {
      num = 1.0;
    } else {
      const double m = (double)(j >> 1);
      if (j & 1)
        num = -(a + m) * (a + b + m) * x / ((a + 2.0 * m) * (a + 2.0 * m + 1.0));
      else
        num = m * (b - m) * x / ((a + 2.0 * m - 1.0) * (a + 2.0 * m));
    }
    d = 1.0 + num * d;
    if (fabs(d) < tiny) d = tiny;
    c = 1.0 + num / c;
    if (fabs(c) < tiny) c = tiny;
    d = 1.0 / d;
    const double del = c * d;
    f *= del;
    if (j > 0 && fabs(del - 1.0) < eps) break;
  }
  return f;
}

// ln Gamma at a = df / 2, b = 1/2 and a + b
struct TGamma {
  double a, b, ab;
};
__device__ inline TGamma t_gamma(double df) {
  return TGamma{lgamma(0.5 * df), lgamma(0.5), lgamma(0.5 * df + 0.5)};
}

__device__ double ln_betai_cf(double x, double a, double b, const TGamma& g) {
  const double lbeta = g.a + g.b - g.ab;
  return a * log(x) + b * log1p(-x) - log(a) - lbeta + log(beta_cf(x, a, b));
}

__device__ double ln_p_two_sided(double t, double df, const TGamma& g) {
  t = fabs(t);
  if (isinf(t)) return -INFINITY;
  if (t == 0.0) return 0.0;
  const double a = 0.5 * df, b = 0.5;
  const double t2 = t * t;
  const double x = df / (df + t2);
  const double omx = t2 / (df + t2);
  if (x < (a + 1.0) / (a + b + 2.0)) return ln_betai_cf(x, a, b, g);
  return log1p(-exp(ln_betai_cf(omx, b, a, g)));
}
__device__ double ln_p_two_sided(double t, double df) { return ln_p_two_sided(t, df, t_gamma(df)); }

__device__ double ln_pdf_t(double t, double df, const TGamma& g) {
  return g.ab - g.a - 0.5 * log(df * M_PI) - 0.5 * (df + 1.0) * log1p(t * t / df);
}

// the cubic Hermite interpolant of -log10 p on interval k (nodes k and k + 1,
// values and slopes), written as its power-series coefficients in the local
// variable s in [0, 1] so that the epilogue evaluates it with three FMAs.  A
// thread evaluates one node in FP64 (the time of the kernel is one thread's
// continued fraction and ln Gamma calls, whose values three lanes share out);
// neighbours exchange theirs, so a wave of 64 nodes gives 63 intervals.
constexpr int kTabWave = 63;
__global__ __launch_bounds__(64) void table_kernel(float4* table, double df) {
  const int lane = threadIdx.x;
  const double lg = lgamma(lane == 0 ? 0.5 * df : lane == 1 ? 0.5 : 0.5 * df + 0.5);
  const TGamma g{__shfl(lg, 0), __shfl(lg, 1), __shfl(lg, 2)};
  const int k = blockIdx.x * kTabWave + lane;
  const double t = (double)(k < kTabNodes ? k : kTabNodes - 1) / kTabPerUnit;
  const double lnp = ln_p_two_sided(t, df, g);
  const double f0 = -lnp / M_LN10;
  const double d0 = 2.0 * exp(ln_pdf_t(t, df, g) - lnp) / M_LN10 / kTabPerUnit;  // slope per unit of s
  const double f1 = __shfl_down(f0, 1), d1 = __shfl_down(d0, 1);
  if (lane == kTabWave || k >= kTabIntervals) return;
  table[k] = make_float4((float)f0, (float)d0, (float)(3.0 * (f1 - f0) - 2.0 * d0 - d1),
                         (float)(2.0 * (f0 - f1) + d0 + d1));
}

// ---------------------------------------------------------------------------
// covariate QR: Householder reflections on the (q x n_pad) column-major work
// copy X of [1 | C].  Each step is three launches: row-parallel partial dot
// products (kQrGrid workgroups, one contiguous row range each), one small
// workgroup that sums the partials in workgroup order and forms the
// reflection's coefficients, and a row-parallel update; so every pass over
// the samples is spread over the GPU.  On exit X holds the Householder
// vectors and Q (q x n_pad) the orthonormal basis.  Fixed grid and fixed
// summation order: the result is the same in every run.
// ---------------------------------------------------------------------------
constexpr int kQrThreads = 256;
constexpr int kQrCB = 4;  // columns reduced together

__global__ __launch_bounds__(kQrThreads) void qr_load_kernel(const double* __restrict__ C, int64_t ldc, int64_t n,
                                                             int64_t n_pad, int q, double* __restrict__ X,
                                                             int32_t* flags) {
  const int64_t total = n_pad * q;
  int bad = 0;
  for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int k = (int)(idx / n_pad);
    const int64_t i = idx - (int64_t)k * n_pad;
    double v = 0.0;  // pad rows are zero
    if (i < n) {
      v = (k == 0) ? 1.0 : C[(int64_t)(k - 1) * ldc + i];
      if (!isfinite(v)) bad = 1;
    }
    X[idx] = v;
  }
  if (bad) flags[0] = 1;
}

// part[b][k] = sum over workgroup b's rows i >= i0 of v[i] * W[k][i], for
// k0 <= k < q (zero for a workgroup with no such rows)
__global__ __launch_bounds__(kQrThreads) void qr_dots_kernel(const double* __restrict__ v,
                                                             const double* __restrict__ W, int64_t n,
                                                             int64_t n_pad, int q, int k0, int64_t i0,
                                                             double* __restrict__ part) {
  __shared__ double sh[(kQrThreads / 64) * kQrCB];
  const int64_t per = (n + gridDim.x - 1) / gridDim.x;
  int64_t rb = (int64_t)blockIdx.x * per;
  const int64_t re = rb + per < n ? rb + per : n;
  rb = rb > i0 ? rb : i0;
  for (int c0 = k0; c0 < q; c0 += kQrCB) {
    double d[kQrCB];
#pragma unroll
    for (int t = 0; t < kQrCB; ++t) d[t] = 0.0;
    for (int64_t i = rb + threadIdx.x; i < re; i += kQrThreads) {
      const double vi = v[i];
#pragma unroll
      for (int t = 0; t < kQrCB; ++t) {
        const int64_t col = c0 + t < q ? c0 + t : q - 1;  // clamped: a valid address, value unused
        d[t] += vi * W[col * n_pad + i];
      }
    }
    block_sum_vec<kQrThreads, kQrCB>(d, sh);
    if (threadIdx.x == 0) {
#pragma unroll
      for (int t = 0; t < kQrCB; ++t)
        if (c0 + t < q) part[(int64_t)blockIdx.x * kSlots + c0 + t] = d[t];
    }
  }
}

// step j's sums dv[k] (k >= j) from the partials, then the coefficients.
// forward: dv[j] = squares of x_j below row j, dv[k > j] = x_j . x_k below
// row j; the reflection maps x_j to alpha e_j (rdiag[j] = alpha), v_j = x_j
// with v_j[j] = x_j[j] - alpha, and fv[k] = 2 (v_j . x_k) / (v_j . v_j).
// backward (forming Q): dv[k] = v_j . Q_k from row j on, fv[k] = 2 dv[k] / vtv[j].
// (one workgroup of kQrThreads; the partials are staged in LDS with
// coalesced loads, then lane k sums column k's in workgroup order)
__global__ __launch_bounds__(kQrThreads) void qr_coef_kernel(double* X, int64_t n_pad, int q, int j, int forward,
                                                             const double* __restrict__ part, double* rdiag,
                                                             double* fv, double* vtv) {
  __shared__ double ps[kQrGrid * kSlots];
  __shared__ double dv[kSlots], row[kSlots];
  const int k = threadIdx.x;
  const bool mine = k >= j && k < q;
  if (forward && mine) row[k] = X[(int64_t)k * n_pad + j];
  for (int idx = threadIdx.x; idx < kQrGrid * kSlots; idx += kQrThreads) ps[idx] = part[idx];
  __syncthreads();
  if (mine) {
    double s = 0.0;
#pragma unroll 16
    for (int b = 0; b < kQrGrid; ++b) s += ps[b * kSlots + k];
    dv[k] = s;
  }
  __syncthreads();
  if (!mine) return;
  if (forward) {
    const double xjj = row[j];
    const double below = dv[j];
    const double nrm = sqrt(xjj * xjj + below);
    const double alpha = xjj > 0.0 ? -nrm : nrm;
    const double v0 = xjj - alpha;
    const double t = below + v0 * v0;
    if (k == j) {
      X[(int64_t)j * n_pad + j] = v0;
      rdiag[j] = alpha;
      vtv[j] = t;
    } else {
      fv[k] = t > 0.0 ? 2.0 * (dv[k] + v0 * row[k]) / t : 0.0;
    }
  } else {
    const double t = vtv[j];
    fv[k] = t > 0.0 ? 2.0 * dv[k] / t : 0.0;
  }
}

// W[k][i] -= fv[k] * v[i] for rows i0 <= i < n and k0 <= k < q
__global__ __launch_bounds__(kQrThreads) void qr_reflect_kernel(const double* v, double* W, int64_t n, int64_t n_pad,
                                                                int q, int k0, int64_t i0,
                                                                const double* __restrict__ fv) {
  __shared__ double f_s[kSlots];
  if (threadIdx.x < kSlots) f_s[threadIdx.x] = (int)threadIdx.x >= k0 && (int)threadIdx.x < q ? fv[threadIdx.x] : 0.0;
  __syncthreads();
  for (int64_t i = i0 + blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const double vi = v[i];
    for (int k = k0; k < q; ++k) W[(int64_t)k * n_pad + i] -= f_s[k] * vi;
  }
}

// Q = [I_q; 0] before the reflections are applied from the last
__global__ void qr_qinit_kernel(double* Q, int64_t n_pad, int q) {
  const int64_t total = n_pad * q;
  for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int k = (int)(idx / n_pad);
    Q[idx] = (idx - (int64_t)k * n_pad == k) ? 1.0 : 0.0;
  }
}

// rank check: every |R_jj| above 1e-10 max |R_ii|
__global__ void qr_rank_kernel(const double* rdiag, int q, int32_t* flags) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  double mx = 0.0;
  for (int j = 0; j < q; ++j) mx = fmax(mx, fabs(rdiag[j]));
  int rd = 0;
  for (int j = 0; j < q; ++j)
    if (!(fabs(rdiag[j]) > 1e-10 * mx)) rd = 1;
  flags[1] = rd;
}


// operand blocks of the covariate columns used for Q^T g: slot k <- Q[:, k]
// for 1 <= k < q, slot 0 and slots >= q are zero.  FP32: one 32-column
// block.  The split forms take packed blocks (hl), one per 16 slots (one
// block when q <= 16, else two): slot k goes to block k / 16, its hi part in
// column k % 16 and its lo part in column k % 16 + 16 of the hi half, the lo
// half zero, so that one matrix-core pass forms both products.
// the Q^T g operands of samples 16 b .. 16 b + 15 of chunk ch and slots 16 t + l16
// (q[i]: sample 4 i + l4 of slot 16 t + l16): slot k >= 1 <- Q[:, k], slot 0 and
// slots >= q are zero
__device__ __forceinline__ void cov_operand_store(float* wop_fp32, char* const (&wop_hl)[2], int n_slots, int n_chunks,
                                                  int ch, int b, int t, int l16, int l4, f64x4 q) {
  const int k = 16 * t + l16;
  double v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = k >= 1 && k < n_slots ? q[i] : 0.0;
  // packed block t: hi part in column l16, lo part in column l16 + 16 (of its
  // first half; the second half is never read), dword l4 of step j = 2 (b & 1)
  // + (i & 1) holding samples i and i + 2
  if (t < hl_blocks(n_slots)) {
    const int64_t at =
        ((int64_t)t * n_chunks + ch) * kBlockBytes + 2 * (b & 1) * 1024 + (b >> 1) * 512 + l16 * 16 + 4 * l4;
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      uint32_t hb[4], lb[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) split_parts(f == 0 ? kSplit : kSplit16, v[i], &hb[i], &lb[i]);
      char* p = wop_hl[f] + at;
      gstore(p, hb[0] | (hb[2] << 16));
      gstore(p + 1024, hb[1] | (hb[3] << 16));
      gstore(p + 256, lb[0] | (lb[2] << 16));
      gstore(p + 1024 + 256, lb[1] | (lb[3] << 16));
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
    wop_fp32[(int64_t)ch * 2048 + (4 * (b & 1) + i) * 256 + (32 * (b >> 1) + k) * 4 + l4] = (float)v[i];
}

struct CovOperandArgs {
  const double* Q;
  int64_t n_pad;
  int q;
  float* wop_fp32;
  char* wop_hl[2];  // BF16 split, FP16 split
};
// the operands of a Q that is in memory: one workgroup per chunk, a wave per 16 samples
__global__ __launch_bounds__(256) void cov_operand_kernel(CovOperandArgs a) {
  const int lane = threadIdx.x & 63, l16 = lane & 15, l4 = lane >> 4;
  const int ch = blockIdx.x, b = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int k = 16 * t + l16;
    f64x4 v = {0.0, 0.0, 0.0, 0.0};
    if (k < a.q) {
      const double* q = a.Q + (int64_t)k * a.n_pad + (int64_t)ch * kChunk + 16 * b + l4;
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = q[4 * i];
    }
    cov_operand_store(a.wop_fp32, a.wop_hl, a.q, (int)(a.n_pad / kChunk), ch, b, t, l16, l4, v);
  }
}

// Q of the intercept alone: -1 / sqrt(n), the sign as of the Householder QR
__global__ __launch_bounds__(256) void intercept_kernel(double* Q, int64_t n, int64_t n_pad) {
  const double v = -1.0 / sqrt((double)n);
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n_pad; i += (int64_t)gridDim.x * blockDim.x)
    Q[i] = i < n ? v : 0.0;
}

// ---------------------------------------------------------------------------
// covariate QR by Cholesky, twice (Yamamoto, Nakatsukasa, Yanagisawa & Fukaya,
// "Roundoff error analysis of the CholeskyQR2 algorithm", ETNA 44, 2015): the
// Gram matrix of X = [1 | C] with unit columns gives R and Q1 = X R^-1, whose
// own Gram matrix, the unit matrix to cond(X)^2 rounding errors, corrects it
// to Q orthonormal to rounding.  Five launches instead of six per column.
// (The intercept alone needs no factorization: intercept_kernel.)
// Taken when every pivot of the first factorization is above kGramPivot
// (condition below about 1e4: Q is then as accurate as the Householder QR's);
// otherwise flags[2] is set, the caller runs the Householder QR above, and
// that one also decides on rank deficiency.
// The Householder QR's column signs are kept: R_jj = -sign(pivot) |R_jj|, the
// pivots being those of Householder reflections on Q itself, which need only
// its first q rows (for orthonormal columns a_j the reflection's products are
// v^T v = 2 (1 + |a_jj|) and v^T a_k = -s a_jk).
// The Gram matrices and products run on the FP64 matrix cores, W waves over
// the sample chunks; the waves' 16 x 16 tiles are added in order.  The last
// kernel also writes the Q^T g operands.
// N = 23,000, K = 10: 0.39 ms in 67 launches -> 0.10 ms; bound by the latency
// of five dependent launches.
// ---------------------------------------------------------------------------
constexpr double kGramPivot = 1e-8;  // squares: 1e-4 of a column's norm
constexpr int kGramTiles = 3;        // (0,0), (0,1), (1,1) of 16 slots each
struct GramArgs {
  const double* C;
  int64_t ldc, n, n_pad;
  int q, waves;
  double* part;   // [waves][kGramTiles][256]
  double* coef;   // first and second q x q factors (kSlots x kSlots each), then R's diagonal
  double* Q1;
  double* Q;
  int32_t* flags;
  float* wop_fp32;
  char* wop_hl[2];  // BF16 split, FP16 split
};
__device__ __forceinline__ double gram_x(const GramArgs& a, int k, int64_t i) {
  if (k == 0 || k >= a.q) return k == 0 && i < a.n ? 1.0 : 0.0;
  const double v = a.C[(int64_t)(k - 1) * a.ldc + (i < a.n ? i : 0)];
  return i < a.n ? v : 0.0;
}
// the tiles a wave's Gram products leave: element (row 4 i + l4, column l16)
template <int NT>
__device__ __forceinline__ void gram_store(const GramArgs& a, int w, int l16, int l4, const f64x4 (&g)[kGramTiles]) {
#pragma unroll
  for (int t = 0; t < (NT == 1 ? 1 : kGramTiles); ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) a.part[((int64_t)w * kGramTiles + t) * 256 + (4 * i + l4) * 16 + l16] = g[t][i];
}

// PASS 0: Gram of X; 1: Q1 = X M1 and its Gram; 2: Q = Q1 M2 and the operands
template <int PASS, int NT>
__global__ __launch_bounds__(64) void gram_kernel(GramArgs a) {
  const int lane = threadIdx.x, l16 = lane & 15, l4 = lane >> 4;
  const int w = blockIdx.x;
  const int nch = (int)(a.n_pad / kChunk);
  const int ch_lo = (int)((int64_t)nch * w / gridDim.x), ch_hi = (int)((int64_t)nch * (w + 1) / gridDim.x);
  if (PASS > 0 && a.flags[2]) return;
  constexpr int KK = 4 * NT;
  double m[NT][KK];  // this pass's factor: element (4 kk + l4, 16 t + l16)
  if constexpr (PASS > 0) {
    const double* c = a.coef + (PASS - 1) * kSlots * kSlots;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) m[t][kk] = c[(4 * kk + l4) * kSlots + 16 * t + l16];
  }
  f64x4 g[kGramTiles];
#pragma unroll
  for (int t = 0; t < kGramTiles; ++t) g[t] = f64x4{0.0, 0.0, 0.0, 0.0};
  int bad = 0;
  for (int ch = ch_lo; ch < ch_hi; ++ch) {
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int64_t s0 = (int64_t)ch * kChunk + 16 * b;
      f64x4 d[NT];
      if constexpr (PASS == 0) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            d[t][i] = gram_x(a, 16 * t + l16, s0 + 4 * i + l4);
            if (!isfinite(d[t][i])) bad = 1;
          }
      } else {
        double x[KK];
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
          const int k = 4 * kk + l4;
          x[kk] = PASS == 1 ? gram_x(a, k, s0 + l16) : k < a.q ? a.Q1[(int64_t)k * a.n_pad + s0 + l16] : 0.0;
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          d[t] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
          for (int kk = 0; kk < KK; ++kk) d[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[kk], m[t][kk], d[t], 0, 0, 0);
          const int k = 16 * t + l16;
          double* out = PASS == 1 ? a.Q1 : a.Q;
          if (k < a.q) {
#pragma unroll
            for (int i = 0; i < 4; ++i) out[(int64_t)k * a.n_pad + s0 + 4 * i + l4] = d[t][i];
          }
          if constexpr (PASS == 2) cov_operand_store(a.wop_fp32, a.wop_hl, a.q, nch, ch, b, t, l16, l4, d[t]);
        }
        if constexpr (PASS == 2 && NT == 1)  // the FP32 block's other 16 columns
          cov_operand_store(a.wop_fp32, a.wop_hl, a.q, nch, ch, b, 1, l16, l4, f64x4{0.0, 0.0, 0.0, 0.0});
      }
      if constexpr (PASS < 2) {  // a product's accumulator layout is both operands' layout
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          g[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(d[0][i], d[0][i], g[0], 0, 0, 0);
          if constexpr (NT == 2) {
            g[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(d[0][i], d[1][i], g[1], 0, 0, 0);
            g[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(d[1][i], d[1][i], g[2], 0, 0, 0);
          }
        }
      }
    }
  }
  if constexpr (PASS < 2) gram_store<NT>(a, w, l16, l4, g);
  if (bad) a.flags[0] = 1;
}

// One workgroup: the Gram matrix from the waves' tiles, its Cholesky factor R
// and the next pass's factor R^-1 (SECOND: with the column signs; also the
// rank check of the Householder QR on R's diagonal).
template <bool SECOND>
__global__ __launch_bounds__(1024) void gram_factor_kernel(GramArgs a) {
  __shared__ double sum[4][256];
  __shared__ double G[kSlots][kSlots + 1], R[kSlots][kSlots + 1], inv[kSlots][kSlots + 1], T[kSlots][kSlots + 1];
  __shared__ double dsc[kSlots], sgn[kSlots];
  __shared__ int ill;
  const int tid = threadIdx.x, q = a.q;
  if (SECOND && a.flags[2]) return;  // uniform
  if (tid == 0) ill = 0;
  for (int t = 0; t < (q <= 16 ? 1 : kGramTiles); ++t) {
    const int r = tid >> 8, e = tid & 255;
    double v = 0.0;
#pragma unroll 8
    for (int w = a.waves * r / 4; w < a.waves * (r + 1) / 4; ++w) v += a.part[((int64_t)w * kGramTiles + t) * 256 + e];
    sum[r][e] = v;
    __syncthreads();
    if (r == 0) {
      v = ((sum[0][e] + sum[1][e]) + sum[2][e]) + sum[3][e];
      const int row = (e >> 4) + (t == 2 ? 16 : 0), col = (e & 15) + (t >= 1 ? 16 : 0);
      G[row][col] = v;
      if (t == 1) G[col][row] = v;
    }
    __syncthreads();
  }
  const int i = tid >> 5, k = tid & 31;  // one thread per element
  if (tid < kSlots) {
    const double d = tid < q ? G[tid][tid] : 1.0;
    if (!SECOND && !(d > 0.0 && isfinite(d))) ill = 1;
    dsc[tid] = SECOND || !(d > 0.0) ? 1.0 : 1.0 / sqrt(d);
  }
  __syncthreads();
  const bool in = i < q && k < q;
  double gv = in ? G[i][k] * dsc[i] * dsc[k] : 0.0;
  for (int j = 0; j < q; ++j) {  // right-looking: thread (i, k) keeps its element
    if (i == j) G[j][k] = gv;
    __syncthreads();
    const double piv = G[j][j];
    if (tid == 0 && !(piv > (SECOND ? 0.5 : kGramPivot))) ill = 1;
    const double rj = sqrt(piv > 0.0 ? piv : 1.0);
    if (i == j) R[j][k] = k >= j && k < q ? gv / rj : 0.0;
    if (i > j && k > j && in) gv -= G[j][i] / rj * (G[j][k] / rj);
    __syncthreads();
  }
  if (ill) {
    if (tid == 0) a.flags[2] = 1;
    return;
  }
  if (tid < kSlots) {  // column tid of R^-1, from its diagonal up
    for (int r = kSlots - 1; r >= 0; --r) {
      double v = 0.0;
      if (tid < q && r <= tid) {
        v = r == tid ? 1.0 : 0.0;
        for (int x = r + 1; x <= tid; ++x) v -= R[r][x] * inv[x][tid];
        v /= R[r][r];
      }
      inv[r][tid] = v;
    }
  }
  __syncthreads();
  double* coef = a.coef + (SECOND ? kSlots * kSlots : 0);
  double* rdiag = a.coef + 2 * kSlots * kSlots;
  if (!SECOND) {
    coef[i * kSlots + k] = dsc[i] * inv[i][k];
    if (tid < q) rdiag[tid] = R[tid][tid] / dsc[tid];
    return;
  }
  // first q rows of Q = Q1 R^-1, then the signs
  double t = 0.0;
  if (in)
    for (int x = 0; x <= k; ++x) t += a.Q1[(int64_t)x * a.n_pad + i] * inv[x][k];
  T[i][k] = t;
  __syncthreads();
  for (int j = 0; j < q; ++j) {
    const double p = T[j][j];
    const double s = p > 0.0 ? -1.0 : 1.0;
    if (tid == 0) sgn[j] = s;
    const double u = in && i > j && k > j ? T[i][j] * s * T[j][k] / (1.0 + fabs(p)) : 0.0;
    __syncthreads();
    if (in && i > j && k > j) T[i][k] += u;
    __syncthreads();
  }
  coef[i * kSlots + k] = k < q ? inv[i][k] * sgn[k] : 0.0;
  if (tid == 0) {  // every |R_jj| above 1e-10 max |R_ii|
    double mx = 0.0;
    for (int j = 0; j < q; ++j) mx = fmax(mx, fabs(rdiag[j] * R[j][j]));
    int rd = 0;
    for (int j = 0; j < q; ++j)
      if (!(fabs(rdiag[j] * R[j][j]) > 1e-10 * mx)) rd = 1;
    a.flags[1] = rd;
  }
}

// ---------------------------------------------------------------------------
// phenotype preparation (Eq. 1 + standardization): one workgroup per CPW
// columns, so that each element of Q read from L2 serves CPW columns; QS >= q
// slots of the projections are kept per column.  Every column's arithmetic
// and summation order is that of a workgroup running it alone.
// ---------------------------------------------------------------------------
constexpr int kPrepThreads = 256;

template <int QS, int CPW>
__global__ __launch_bounds__(kPrepThreads) void prep_kernel(const void* __restrict__ Y, int y_fp64, int64_t ldy,
                                                            int64_t n, int64_t n_pad, int64_t P,
                                                            const double* __restrict__ Q, int q, int prec,
                                                            void* yop, float* scale, float* invny, float* cw,
                                                            uint8_t* lscale, int32_t* flags) {
  static_assert(QS <= kSlots, "projection slots");
  constexpr int NV = CPW * (QS + 2);
  __shared__ double sh[(kPrepThreads / 64) * NV];
  __shared__ double qty_s[CPW][QS];
  const int tid = threadIdx.x;
  const int n_chunks = (int)(n_pad / kChunk);
  const int64_t p0 = (int64_t)blockIdx.x * CPW;
  // columns past P repeat the last one; nothing of theirs is stored
  int64_t pc[CPW];
#pragma unroll
  for (int c = 0; c < CPW; ++c) pc[c] = p0 + c < P ? p0 + c : P - 1;
  auto yval = [&](int c, int64_t i) -> double {
    return y_fp64 ? ((const double*)Y)[pc[c] * ldy + i] : (double)((const float*)Y)[pc[c] * ldy + i];
  };
  // slots k >= q hold zero: every slot is loaded (past q, column q - 1
  // again) and multiplied without a branch, which adds exact zeros only, so
  // the loads of a sample issue together
  auto load_q = [&](int64_t i, double* qv) {
#pragma unroll
    for (int k = 0; k < QS; ++k) {
      const double v = Q[(int64_t)(k < q ? k : q - 1) * n_pad + i];
      qv[k] = k < q ? v : 0.0;
    }
  };

  // pass 1: means (and finiteness)
  double mean[CPW];
#pragma unroll
  for (int c = 0; c < CPW; ++c) mean[c] = 0.0;
  int bad = 0;
  for (int64_t i = tid; i < n; i += kPrepThreads) {
#pragma unroll
    for (int c = 0; c < CPW; ++c) {
      const double v = yval(c, i);
      if (!isfinite(v)) bad = 1;
      mean[c] += v;
    }
  }
  bad = __syncthreads_or(bad);
  if (bad) {
    if (tid == 0) atomicOr(flags, 1);
    return;
  }
  block_sum_vec<kPrepThreads, CPW>(mean, sh);
#pragma unroll
  for (int c = 0; c < CPW; ++c) mean[c] /= (double)n;

  // pass 2: Q^T y_c and ||y_c||^2 (slot QS)
  double acc[CPW][QS + 2];
#pragma unroll
  for (int c = 0; c < CPW; ++c)
#pragma unroll
    for (int k = 0; k < QS + 2; ++k) acc[c][k] = 0.0;
  for (int64_t i = tid; i < n; i += kPrepThreads) {
    double qv[QS];
    load_q(i, qv);
#pragma unroll
    for (int c = 0; c < CPW; ++c) {
      const double yc = yval(c, i) - mean[c];
      acc[c][QS] += yc * yc;
#pragma unroll
      for (int k = 0; k < QS; ++k) acc[c][k] += qv[k] * yc;
    }
  }
  block_sum_vec<kPrepThreads, NV>(&acc[0][0], sh);
  double yc2[CPW];
#pragma unroll
  for (int c = 0; c < CPW; ++c) {
    yc2[c] = acc[c][QS];
#pragma unroll
    for (int k = 0; k < QS; ++k)
      if (tid == k) qty_s[c][k] = acc[c][k];
  }
  __syncthreads();

  // y_res of column c at sample i, given Q's column i
  auto yres = [&](int c, int64_t i, const double* qv) {
    double v = yval(c, i) - mean[c];
#pragma unroll
    for (int k = 0; k < QS; ++k) v -= qv[k] * qty_s[c][k];
    return v;
  };

  // pass 3: ||y_res||^2
  double r2[CPW];
#pragma unroll
  for (int c = 0; c < CPW; ++c) r2[c] = 0.0;
  for (int64_t i = tid; i < n; i += kPrepThreads) {
    double qv[QS];
    load_q(i, qv);
#pragma unroll
    for (int c = 0; c < CPW; ++c) {
      const double v = yres(c, i, qv);
      r2[c] += v * v;
    }
  }
  block_sum_vec<kPrepThreads, CPW>(r2, sh);
  double sp[CPW], inv[CPW];
  bool valid[CPW];
#pragma unroll
  for (int c = 0; c < CPW; ++c) {
    sp[c] = sqrt(r2[c]);
    valid[c] = sp[c] > 1e-12 * sqrt(yc2[c]);
    inv[c] = valid[c] ? 1.0 / sp[c] : 0.0;
  }

  // pass 3b (FP8 lo form): each column's largest lo term sets its scale
  int lsh[CPW];
#pragma unroll
  for (int c = 0; c < CPW; ++c) lsh[c] = 0;
  if (prec == kSplit8) {
    double mx[CPW];
#pragma unroll
    for (int c = 0; c < CPW; ++c) mx[c] = 0.0;
    for (int64_t i = tid; i < n; i += kPrepThreads) {
      double qv[QS];
      load_q(i, qv);
#pragma unroll
      for (int c = 0; c < CPW; ++c) {
        const double vs = yres(c, i, qv) * inv[c] * (double)kF16Scale;
        mx[c] = fmax(mx[c], fabs(vs - (double)f16_to_float(f16_bits_rn((float)vs))));
      }
    }
#pragma unroll
    for (int c = 0; c < CPW; ++c) {
      lsh[c] = lo_shift(block_max<kPrepThreads>(mx[c], sh));
      if (tid == 0 && p0 + c < P) lscale[p0 + c] = (uint8_t)(127 - lsh[c]);
    }
  }

  // pass 4: y~ = y_res / s_p into the operand; accumulate what the stored
  // (rounded) operand actually holds: Q^T y_op, sum (slot QS), norm^2 (QS + 1),
  // and (FP16 + FP8 form) the sum of the FP8 lo terms alone
#pragma unroll
  for (int c = 0; c < CPW; ++c)
#pragma unroll
    for (int k = 0; k < QS + 2; ++k) acc[c][k] = 0.0;
  double lsum[CPW];
#pragma unroll
  for (int c = 0; c < CPW; ++c) lsum[c] = 0.0;
  for (int64_t i = tid; i < n; i += kPrepThreads) {
    double qv[QS];
    load_q(i, qv);
#pragma unroll
    for (int c = 0; c < CPW; ++c) {
      if (p0 + c >= P) continue;
      double st, lo;
      store_operand(yop, prec, p0 + c, i, n_chunks, yres(c, i, qv) * inv[c], &st, lsh[c], &lo);
      lsum[c] += lo;
      acc[c][QS] += st;
      acc[c][QS + 1] += st * st;
#pragma unroll
      for (int k = 0; k < QS; ++k) acc[c][k] += qv[k] * st;
    }
  }
  block_sum_vec<kPrepThreads, NV>(&acc[0][0], sh);
  // FP16 + FP8 form with q <= 31: the last correction slot takes minus the
  // column's sum of lo terms (a plan whose markers centre their FP8 pass on
  // c8 = rint(c) puts c - c8 against it)
  const bool lo_slot = prec == kSplit8 && q <= kLoSlot;
  if (lo_slot) block_sum_vec<kPrepThreads, CPW>(lsum, sh);
#pragma unroll
  for (int c = 0; c < CPW; ++c) {
    const int64_t p = p0 + c;
    if (p >= P) break;
    if (tid == 0) {
      double proj = 0.0;
#pragma unroll
      for (int k = 0; k < QS; ++k)
        if (k < q) proj += acc[c][k] * acc[c][k];
      const double ny2 = acc[c][QS + 1] - proj;
      scale[p] = (float)sp[c];
      invny[p] = (valid[c] && ny2 > 0.0) ? (float)(1.0 / sqrt(ny2)) : __builtin_nanf("");
    }
    if (tid < kSlots) {
      float v = tid == 0 ? (float)(-acc[c][QS]) : 0.0f;
#pragma unroll
      for (int k = 1; k < QS; ++k)
        if (tid == k && k < q) v = (float)(-acc[c][k]);
      if (lo_slot && tid == kLoSlot) v = (float)(-lsum[c]);
      cw[p * kSlots + tid] = v;
    }
  }
}

// ---------------------------------------------------------------------------
// phenotype preparation over sample segments (cohorts of kPrepSplitMin
// samples and more): the same quantities as prep_kernel, with the projections
// on the FP64 matrix cores and the samples of 16 columns cut into S segments,
// one wave each, so that a panel of any width fills the GPU and each element
// of Q read serves 16 columns.  Each pass leaves its sums per segment
// (part[slot][segment][column]) and prep_sum_kernel adds them in segment
// order:
//   A: sums of v = y - y_0, v^2 and Q^T v (y_0: the column's first sample,
//      so that offsets cancel; Q^T of a constant is that constant times
//      n Q_0 in slot 0, Q_0 being constant, and 0 in the others)
//   B: ||y_res||^2 explicitly, only for columns where ||y_c||^2 - ||Q^T y_c||^2
//      is below 1e-4 of the sum of v^2 it is a difference from (there still
//      good to 1e-12): columns that the covariates nearly explain, or whose
//      first sample is far off the others
//   C: FP16 + FP8 form: the largest |lo| term
//   D: the operand, and the sums of what it holds
// N = 23,000, K = 10, FP16 + FP8 form: P = 2,048 (FP64 input) 1,010 -> 510 us,
// P = 300 (K = 13) 530 -> 135 us, P = 1 333 -> 65 us; N = 500,001, P = 8: 15.2
// -> 0.4 ms (prep_kernel before).  Bound by latency at few columns, by the
// reads of Y (three passes of 377 MB, 3 TB/s) and FP64 issue in pass D at many.
// ---------------------------------------------------------------------------
struct PrepArgs {
  const void* Y;
  int64_t ldy, n, n_pad, P;
  const double* Q;
  int q, y_fp64;
  int n_tiles, segs;      // 16-column tiles, sample segments
  int slots;              // 16 per slot tile of the covariate basis (kPrepMore more follow)
  void* yop;
  double* part;           // [slots][segs][16 n_tiles]
  double* sums;           // [slots][16 n_tiles]: A's, then D's in the second half
  double* r2;             // [16 n_tiles]: B
  double* maxlo;          // [16 n_tiles]: C
  uint8_t* lscale;
  float* scale;
  float* invny;
  float* cw;
  int32_t* flags;
};
// slots of the sums after those of Q^T v
constexpr int kPrepV = 0;   // sum of v (D: sum of the operand)
constexpr int kPrepVV = 1;  // sum of v^2 (D: its square)
constexpr int kPrepL = 2;   // D: sum of the lo terms
constexpr int kPrepMore = 3;
__host__ __device__ constexpr int prep_slot_tiles(int q) { return q <= 16 ? 1 : 2; }

// y at samples s0 + 4 i (s0 = first + l4) of this lane's column; zero past n
template <bool F64>
__device__ __forceinline__ f64x4 prep_y(const void* col, int64_t s0, int64_t n, bool whole) {
  f64x4 v;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t s = s0 + 4 * i;
    const bool ok = whole || s < n;
    const int64_t sc = ok ? s : 0;
    double x;
    if constexpr (F64)
      x = gload<double>((const double*)col + sc);
    else
      x = (double)gload<float>((const float*)col + sc);
    v[i] = ok ? x : 0.0;
  }
  return v;
}

// this wave's tile, segment and column
struct PrepWave {
  int tile, seg, l16, l4, ch_lo, ch_hi;
  int64_t col;        // clamped to the panel
  bool on;
};
__device__ __forceinline__ PrepWave prep_wave(const PrepArgs& a) {
  PrepWave w;
  const int lane = threadIdx.x & 63;
  const int64_t id = (int64_t)blockIdx.x * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  w.on = id < (int64_t)a.n_tiles * a.segs;
  w.tile = (int)(id % a.n_tiles);
  w.seg = (int)(id / a.n_tiles);
  w.l16 = lane & 15;
  w.l4 = lane >> 4;
  const int64_t nch = a.n_pad / kChunk;
  w.ch_lo = (int)(nch * w.seg / a.segs);
  w.ch_hi = (int)(nch * (w.seg + 1) / a.segs);
  const int64_t c = (int64_t)w.tile * 16 + w.l16;
  w.col = c < a.P ? c : a.P - 1;
  return w;
}
__device__ __forceinline__ int64_t prep_at(const PrepArgs& a, int slot, int seg, int64_t c) {
  return ((int64_t)slot * a.segs + seg) * (16 * (int64_t)a.n_tiles) + c;
}
// a lane's sum over its 16-sample blocks, added over the four lanes of a column
__device__ __forceinline__ double prep_col_sum(double v) {
  v += __shfl_xor(v, 16);
  v += __shfl_xor(v, 32);
  return v;
}

template <int NT, bool F64>
__global__ __launch_bounds__(256, 4) void prep_project_kernel(PrepArgs a) {
  const PrepWave w = prep_wave(a);
  if (!w.on) return;
  const char* col = (const char*)a.Y + w.col * a.ldy * (F64 ? 8 : 4);
  const double y0 = F64 ? *(const double*)col : (double)*(const float*)col;
  f64x4 acc[NT];
  int64_t oq[NT];
#pragma unroll
  for (int x = 0; x < NT; ++x) {
    acc[x] = f64x4{0.0, 0.0, 0.0, 0.0};
    oq[x] = (min(16 * x + w.l16, a.q - 1) * a.n_pad + w.l4) * 8;
  }
  double sv = 0.0, svv = 0.0;
  int bad = 0;
  for (int ch = w.ch_lo; ch < w.ch_hi; ++ch) {
    const bool whole = (int64_t)(ch + 1) * kChunk <= a.n;
    const char* qc = (const char*)(a.Q + (int64_t)ch * kChunk);
    // the chunk's loads are issued together
    f64x4 y[4], qv[4][NT];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      y[b] = prep_y<F64>(col, (int64_t)ch * kChunk + 16 * b + w.l4, a.n, whole);
#pragma unroll
      for (int x = 0; x < NT; ++x)
#pragma unroll
        for (int i = 0; i < 4; ++i) qv[b][x][i] = gload<double>(qc + 128 * b + 32 * i + oq[x]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int64_t s0 = (int64_t)ch * kChunk + 16 * b + w.l4;
      f64x4 v = y[b];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (!isfinite(v[i])) bad = 1;
        v[i] = whole || s0 + 4 * i < a.n ? v[i] - y0 : 0.0;
        sv += v[i];
        svv += v[i] * v[i];
      }
#pragma unroll
      for (int x = 0; x < NT; ++x)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          acc[x] = __builtin_amdgcn_mfma_f64_16x16x4f64(qv[b][x][i], v[i], acc[x], 0, 0, 0);
    }
  }
  if (bad) atomicOr(a.flags, 1);
  const int64_t c = (int64_t)w.tile * 16 + w.l16;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) a.part[prep_at(a, 16 * t + 4 * i + w.l4, w.seg, c)] = acc[t][i];
  sv = prep_col_sum(sv);
  svv = prep_col_sum(svv);
  if (w.l4 == 0) {
    a.part[prep_at(a, 16 * NT + kPrepV, w.seg, c)] = sv;
    a.part[prep_at(a, 16 * NT + kPrepVV, w.seg, c)] = svv;
  }
}

// sums over the segments, in order: 16 columns x 16 runs of segments per
// workgroup, each run in order and then the runs in order (MAX: the largest)
template <bool MAX>
__global__ __launch_bounds__(256) void prep_sum_kernel(const double* __restrict__ part, double* __restrict__ out,
                                                       int segs, int64_t ncol) {
  __shared__ double sh[16][17];
  const int c = threadIdx.x & 15, r = threadIdx.x >> 4;
  const int64_t col = (int64_t)blockIdx.x * 16 + c;
  const double* p = part + (int64_t)blockIdx.y * segs * ncol + col;
  const int lo = segs * r / 16, hi = segs * (r + 1) / 16;
  double v = 0.0;
#pragma unroll 8
  for (int s = lo; s < hi; ++s) v = MAX ? fmax(v, p[s * ncol]) : v + p[s * ncol];
  sh[r][c] = v;
  __syncthreads();
  if (r == 0) {
    v = sh[0][c];
#pragma unroll
    for (int x = 1; x < 16; ++x) v = MAX ? fmax(v, sh[x][c]) : v + sh[x][c];
    out[(int64_t)blockIdx.y * ncol + col] = v;
  }
}

// x as a float rounded to odd (truncated, the last bit set where anything was
// cut off): rounding that to nearest even at any width two or more bits
// narrower gives what rounding x itself gives
__device__ __forceinline__ float float_to_odd(double x) {
  const float f = (float)x;
  uint32_t u = __float_as_uint(f);
  if (fabs((double)f) > fabs(x)) --u;
  if ((double)f != x) u |= 1u;
  return __uint_as_float(u);
}

// what a column's sums of pass A say
struct PrepColumn {
  double mean, yc2, r2;
  bool direct;  // ||y_res||^2 from the difference of squares
};
__device__ __forceinline__ double prep_qty(const PrepArgs& a, int k, int64_t c, double delta) {
  const double v = a.sums[min(k, a.q - 1) * (16 * (int64_t)a.n_tiles) + c];
  return k == 0 ? v - delta * ((double)a.n * a.Q[0]) : k < a.q ? v : 0.0;
}
__device__ __forceinline__ PrepColumn prep_column(const PrepArgs& a, int64_t c, double y0, double* delta) {
  const int64_t nc = 16 * (int64_t)a.n_tiles;
  PrepColumn p;
  const double d = a.sums[(a.slots + kPrepV) * nc + c] / (double)a.n;
  p.mean = y0 + d;
  *delta = d;
  const double v2 = a.sums[(a.slots + kPrepVV) * nc + c];
  p.yc2 = fmax(v2 - (double)a.n * d * d, 0.0);
  double s = p.yc2;
#pragma unroll 8
  for (int k = 0; k < a.q; ++k) {
    const double t = prep_qty(a, k, c, d);
    s -= t * t;
  }
  p.r2 = s;
  p.direct = s > 1e-4 * v2;
  return p;
}

// PASS 0: B, 1: C, 2: D; NT: 16-slot tiles of the covariate basis
template <int PASS, int PREC, int NT, bool F64>
__global__ __launch_bounds__(256, PASS == 2 ? 3 : 4) void prep_residual_kernel(PrepArgs a) {
  const PrepWave w = prep_wave(a);
  if (!w.on) return;
  const char* colp = (const char*)a.Y + w.col * a.ldy * (F64 ? 8 : 4);
  const double y0 = F64 ? *(const double*)colp : (double)*(const float*)colp;
  const int64_t c = (int64_t)w.tile * 16 + w.l16;
  double delta;
  const PrepColumn pc = prep_column(a, c, y0, &delta);
  if (PASS == 0 && __builtin_amdgcn_ballot_w64(!pc.direct) == 0) return;  // uniform: no column of the tile needs it
  const double r2 = PASS == 0 || pc.direct ? pc.r2 : a.r2[c];
  const double sp = sqrt(r2);
  const bool valid = sp > 1e-12 * sqrt(pc.yc2);
  const double inv = valid ? 1.0 / sp : 0.0;
  const double inv16 = inv * (double)kF16Scale;  // a power of two times inv: v inv16 rounds as (v inv) 2^12
  const int lsh = PASS == 2 && PREC == kSplit8 ? lo_shift(a.maxlo[c]) : 0;
  const double lo_up = ldexp(1.0, lsh), lo_down = ldexp(1.0, -lsh);
  constexpr int KK = 4 * NT;
  double nq[KK];
  int64_t oq[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    nq[kk] = -prep_qty(a, 4 * kk + w.l4, c, delta);
    oq[kk] = (min(4 * kk + w.l4, a.q - 1) * a.n_pad + w.l16) * 8;
  }
  constexpr int BB = block_bytes(PREC);
  const bool colok = c < a.P;
  // this lane's dwords of the column block's chunk (see operand_block)
  char* opc = PASS == 2 ? (char*)a.yop + (c >> 5) * (a.n_pad / kChunk) * (int64_t)BB + (c & 31) * 16 + 4 * w.l4 : nullptr;
  f64x4 acc[NT];
  int64_t oa[NT];
#pragma unroll
  for (int x = 0; x < NT; ++x) {
    acc[x] = f64x4{0.0, 0.0, 0.0, 0.0};
    oa[x] = (min(16 * x + w.l16, a.q - 1) * a.n_pad + w.l4) * 8;
  }
  double s1 = 0.0, s2 = 0.0, sl = 0.0, mx = 0.0;
  for (int ch = w.ch_lo; ch < w.ch_hi; ++ch) {
    const bool whole = (int64_t)(ch + 1) * kChunk <= a.n;
    const char* qc = (const char*)(a.Q + (int64_t)ch * kChunk);
    // the chunk's loads are issued together
    f64x4 y[4];
    double qv[4][KK];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      y[b] = prep_y<F64>(colp, (int64_t)ch * kChunk + 16 * b + w.l4, a.n, whole);
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) qv[b][kk] = gload<double>(qc + 128 * b + oq[kk]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int64_t s0 = (int64_t)ch * kChunk + 16 * b + w.l4;
      f64x4 v = y[b];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = whole || s0 + 4 * i < a.n ? v[i] - pc.mean : 0.0;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk)
        v = __builtin_amdgcn_mfma_f64_16x16x4f64(qv[b][kk], nq[kk], v, 0, 0, 0);
      if constexpr (PASS == 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) s1 += v[i] * v[i];
      } else if constexpr (PASS == 1) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const double vs = v[i] * inv16;
          mx = fmax(mx, fabs(vs - (double)f16_to_float(f16_bits_rn((float)vs))));
        }
      } else {
        f64x4 st;
        char* p = opc + (int64_t)ch * BB + (b >> 1) * 512;
        if constexpr (PREC == kFP32) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float f = (float)(v[i] * inv);
            if (colok) gstore(p + (4 * (b & 1) + i) * 1024, f);
            st[i] = (double)f;
          }
        } else {
          uint32_t hb[4], lb[4];
          if constexpr (PREC == kSplit8) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const double vs = v[i] * inv16;
              hb[i] = f16_bits_rn((float)vs);
              st[i] = (double)f16_to_float(hb[i]);
              lb[i] = __float_as_uint(float_to_odd((vs - st[i]) * lo_up));
            }
            int lo = __builtin_amdgcn_cvt_pk_fp8_f32(__uint_as_float(lb[0]), __uint_as_float(lb[1]), 0, false);
            lo = __builtin_amdgcn_cvt_pk_fp8_f32(__uint_as_float(lb[2]), __uint_as_float(lb[3]), lo, true);
            const float lf[4] = {__builtin_amdgcn_cvt_f32_fp8(lo, 0), __builtin_amdgcn_cvt_f32_fp8(lo, 1),
                                 __builtin_amdgcn_cvt_f32_fp8(lo, 2), __builtin_amdgcn_cvt_f32_fp8(lo, 3)};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const double lv = (double)lf[i] * lo_down;
              sl += lv;
              st[i] += lv;
            }
            if (colok) gstore(p + 4096 + (b & 1) * 1024, lo);
          } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              split_parts(PREC, v[i] * inv, &hb[i], &lb[i]);
              st[i] = PREC == kSplit16 ? (double)f16_to_float(hb[i]) + (double)f16_to_float(lb[i])
                                       : (double)bf16_to_float(hb[i]) + (double)bf16_to_float(lb[i]);
            }
            if (colok) {
              gstore(p + 4096 + 2 * (b & 1) * 1024, lb[0] | (lb[2] << 16));
              gstore(p + 4096 + 2 * (b & 1) * 1024 + 1024, lb[1] | (lb[3] << 16));
            }
          }
          if (colok) {
            gstore(p + 2 * (b & 1) * 1024, hb[0] | (hb[2] << 16));
            gstore(p + 2 * (b & 1) * 1024 + 1024, hb[1] | (hb[3] << 16));
          }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          s1 += st[i];
          s2 += st[i] * st[i];
        }
#pragma unroll
        for (int x = 0; x < NT; ++x)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            acc[x] = __builtin_amdgcn_mfma_f64_16x16x4f64(gload<double>(qc + 128 * b + 32 * i + oa[x]), st[i], acc[x], 0, 0,
                                                         0);
      }
    }
  }
  if constexpr (PASS == 0) {
    s1 = prep_col_sum(s1);
    if (w.l4 == 0) a.part[prep_at(a, 0, w.seg, c)] = s1;
  } else if constexpr (PASS == 1) {
    mx = fmax(mx, __shfl_xor(mx, 16));
    mx = fmax(mx, __shfl_xor(mx, 32));
    if (w.l4 == 0) a.part[prep_at(a, 0, w.seg, c)] = mx;
  } else {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) a.part[prep_at(a, 16 * t + 4 * i + w.l4, w.seg, c)] = acc[t][i];
    s1 = prep_col_sum(s1);
    s2 = prep_col_sum(s2);
    sl = prep_col_sum(sl);
    if (w.l4 == 0) {
      a.part[prep_at(a, 16 * NT + kPrepV, w.seg, c)] = s1;
      a.part[prep_at(a, 16 * NT + kPrepVV, w.seg, c)] = s2;
      a.part[prep_at(a, 16 * NT + kPrepL, w.seg, c)] = sl;
    }
  }
}

// per-column constants from the sums of passes A and D (one wave per column)
__global__ __launch_bounds__(256) void prep_finish_kernel(PrepArgs a, int prec) {
  const int64_t p = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (p >= a.P) return;
  const int64_t nc = 16 * (int64_t)a.n_tiles;
  const char* colp = (const char*)a.Y + p * a.ldy * (a.y_fp64 ? 8 : 4);
  double delta;
  const PrepColumn pc = prep_column(a, p, a.y_fp64 ? *(const double*)colp : (double)*(const float*)colp, &delta);
  const double sp = sqrt(pc.direct ? pc.r2 : a.r2[p]);
  const bool valid = sp > 1e-12 * sqrt(pc.yc2);
  const double* d = a.sums + (a.slots + kPrepMore) * nc + p;  // pass D's
  if (lane == 0) {
    double proj = 0.0;
    for (int k = 0; k < a.q; ++k) proj += d[k * nc] * d[k * nc];
    const double ny2 = d[(a.slots + kPrepVV) * nc] - proj;
    a.scale[p] = (float)sp;
    a.invny[p] = (valid && ny2 > 0.0) ? (float)(1.0 / sqrt(ny2)) : __builtin_nanf("");
    if (prec == kSplit8) a.lscale[p] = (uint8_t)(127 - lo_shift(a.maxlo[p]));
  }
  if (lane < kSlots) {
    float v = 0.0f;
    if (lane == 0) v = (float)(-d[(a.slots + kPrepV) * nc]);
    if (lane >= 1 && lane < a.q) v = (float)(-d[lane * nc]);
    // FP16 + FP8 form with q <= 31: the last slot takes minus the column's sum of lo terms (see prep_kernel)
    if (lane == kLoSlot && prec == kSplit8 && a.q <= kLoSlot) v = (float)(-d[(a.slots + kPrepL) * nc]);
    a.cw[p * kSlots + lane] = v;
  }
}
// test hook: raw operand columns (no centring / scaling)
__global__ __launch_bounds__(kPrepThreads) void set_lscale_kernel(const float* __restrict__ V, int64_t ldv,
                                                                  int64_t n, uint8_t* lscale) {
  __shared__ double sh[kPrepThreads / 64];
  const int64_t p = blockIdx.x;
  double mx = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += kPrepThreads) {
    const double vs = (double)V[p * ldv + i] * (double)kF16Scale;
    mx = fmax(mx, fabs(vs - (double)f16_to_float(f16_bits_rn((float)vs))));
  }
  mx = block_max<kPrepThreads>(mx, sh);
  if (threadIdx.x == 0) lscale[p] = (uint8_t)(127 - lo_shift(mx));
}

__global__ void set_operand_kernel(const float* __restrict__ V, int64_t ldv, int64_t n, int64_t n_pad,
                                   int64_t P, int prec, void* yop, const uint8_t* lscale) {
  const int n_chunks = (int)(n_pad / kChunk);
  const int64_t total = n_pad * P;
  for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int64_t p = idx / n_pad;
    const int64_t i = idx % n_pad;
    const double v = i < n ? (double)V[p * ldv + i] : 0.0;
    double st;
    store_operand(yop, prec, p, i, n_chunks, v, &st, prec == kSplit8 ? 127 - (int)lscale[p] : 0);
  }
}

// Decode table of a marker of 8-bit dosages (q = 0..254, 255 missing),
// operand value q - c with an integer c = rint(mu), missing -> mu - c:
//   x = FP16 pair of -(1024 + c)    (1024 + q is built exactly by byte insertion)
//   y = FP16 pair of mu - c
//   z = FP32 bits of c, w = FP32 bits of mu - c   (the FP32 form)
__device__ void stats_dosage8(const StatsArgs& a, int64_t m, int lane) {
  const uint32_t* row = (const uint32_t*)(a.geno + (a.m0 + m) * a.row_bytes);
  const int64_t nd = (a.n + 3) / 4;
  uint32_t nmiss = 0;
  uint64_t S1 = 0, S2 = 0;
  for (int64_t d = lane; d < nd; d += 64) {
    const uint32_t w = row[d];
    const int64_t nv = a.n - 4 * d;
    const uint32_t vm = nv >= 4 ? 0xffffffffu : ((1u << (8 * nv)) - 1u);
    const uint32_t miss = ff_bytes(w) & vm;
    const uint32_t obs = w & ~miss & vm;
    nmiss += __popc(miss) >> 3;
    S1 += __builtin_amdgcn_udot4(obs, 0x01010101u, 0u, false);
    S2 += __builtin_amdgcn_udot4(obs, obs, 0u, false);
  }
  uint64_t M = nmiss;
  for (int o = 32; o > 0; o >>= 1) {
    M += __shfl_xor(M, o);
    S1 += __shfl_xor(S1, o);
    S2 += __shfl_xor(S2, o);
  }
  if (lane != 0) return;
  const int64_t n_obs = a.n - (int64_t)M;
  const int64_t sg = (int64_t)S1, sg2 = (int64_t)S2;
  const __int128 num128 = (__int128)n_obs * sg2 - (__int128)sg * sg;  // n_obs * sum (q - mu)^2
  const bool ok = n_obs > 0 && num128 != 0;
  MarkerStat st;
  st.flags = ok ? 0 : 1;
  const double mu = n_obs > 0 ? (double)sg / (double)n_obs : 0.0;
  const double c = ok ? rint(mu) : 0.0;
  st.mu = mu;
  st.shift = c;
  st.gscale = 1.0f;
  st.dlo = 0.0f;
  st.gc2 = n_obs > 0 ? (double)num128 / (double)n_obs : 0.0;
  st.dmu = (float)(mu - c);
  const uint32_t nc = f16_bits_rn((float)(-1024.0 - c));
  const uint32_t dm = f16_bits_rn((float)(mu - c));
  a.mlut[m] = make_uint4(nc | (nc << 16), dm | (dm << 16), __float_as_uint((float)c), __float_as_uint((float)(mu - c)));
  a.mstat[m] = st;
}

// ---------------------------------------------------------------------------
// per-marker statistics (one wave per marker)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void stats_kernel(StatsArgs a) {
  if (blockIdx.x == 0 && a.redo_count)  // the FP64 list of this block starts empty
    for (int j = threadIdx.x; j < a.n_panels; j += blockDim.x) a.redo_count[j] = 0u;
  const int lane = threadIdx.x & 63;
  const int64_t m = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (m >= a.nm) return;
  if (a.code == 2) {
    stats_dosage8(a, m, lane);
    return;
  }
  // 16 bytes (64 samples) per lane and load; rows are 16-byte aligned and
  // hold at least ceil(n / 64) such pieces
  const uint4* row = (const uint4*)(a.geno + (a.m0 + m) * a.row_bytes);
  const int64_t n16 = (a.n + 63) / 64;
  // three popcounts per word: codes with the low bit set (pl), with the high
  // bit set (ph), with both (pb); codes past n are masked to 00, which counts
  // in none of them.  The tallies follow from these per coding below.
  int pl = 0, ph = 0, pb = 0;
  for (int64_t d4 = lane; d4 < n16; d4 += 64) {
    const uint4 w4 = row[d4];
    const uint32_t ws[4] = {w4.x, w4.y, w4.z, w4.w};
    const bool full = 64 * (d4 + 1) <= a.n;  // all 64 samples of this piece are real
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint32_t w = ws[q];
      if (!full) {
        const int64_t nv = a.n - 16 * (4 * d4 + q);  // samples in this word
        w &= nv >= 16 ? 0xffffffffu : (nv <= 0 ? 0u : ((1u << (2 * nv)) - 1u));
      }
      const uint32_t lo = w & 0x55555555u;
      const uint32_t hi = (w >> 1) & 0x55555555u;
      pl += __popc(lo);
      ph += __popc(hi);
      pb += __popc(lo & hi);
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    pl += __shfl_xor(pl, o);
    ph += __shfl_xor(ph, o);
    pb += __shfl_xor(pb, o);
  }
  int nmiss, c1, c2;
  if (a.code == 0) {  // dosage: 0, 1, 2, 3 = missing (low bit only: 1; high bit only: 2)
    nmiss = pb;
    c1 = pl - pb;
    c2 = ph - pb;
  } else {  // PLINK .bed: 00 -> 0, 01 -> missing, 10 -> 1, 11 -> 2
    c2 = pb;
    nmiss = pl - pb;
    c1 = ph - pb;
  }
  const int64_t n_obs = a.n - nmiss;
  const int64_t sg = c1 + 2 * (int64_t)c2;
  const int64_t sg2 = c1 + 4 * (int64_t)c2;
  const int64_t num = n_obs * sg2 - sg * sg;  // n_obs * sum (g - mu)^2
  const bool ok = n_obs > 0 && num != 0;
  const double mu = n_obs > 0 ? (double)sg / (double)n_obs : 0.0;
  // operand value of a call g: gs (g - c); of a missing call: gs (mu - c)
  // rounded to the operand type.  FP16 forms: gs = 1, c on the 1/512 grid
  // (g - c exact in 11 bits, missing value to 2^-21).  FP32: gs = 1, c on
  // the 1/64 grid.  BF16 (8 significant bits): gs = K / 128 and c = U / K
  // with integers K >= 1 and U = rint(K mu) such that the calls' values
  // (-U, K - U, 2K - U) / 128 have magnitude <= 2, hence are exact; of those
  // K, the one whose missing value (K mu - U) / 128 rounds to BF16 with the
  // smallest error per genotype unit (ties: the larger K).  The error is
  // about 2^-9 |mu - U / K|: at most about 2^-18 (mu within 1/512 of a
  // simple fraction such as 1/2 or 1), typically below 2^-24, against up
  // to 2^-16 for the nearest multiple of 1/64.  The 256 candidates are
  // spread over the wave's lanes.
  // A marker without missing calls carries no missing value: every form
  // takes gs = 1 and the integer c = rint(mu), so that its operand holds
  // small integers, whose few changing bits cost the matrix cores less
  // power than fractional values (the contraction's clock is power-bound).
  const bool whole = ok && nmiss == 0;
  double c = 0.0, gs = 1.0, vmiss = mu, vg[3] = {0.0, 1.0, 2.0};  // degenerate: not re-centred
  if (whole) {
    c = rint(mu);
    vmiss = mu - c;
    for (int g = 0; g < 3; ++g) vg[g] = (double)g - c;
  } else if (ok && a.prec == kSplit) {
    double best = INFINITY;
    int bk = 0;
    for (int K = 256 - lane; K >= 1; K -= 64) {
      const double km = (double)K * mu;
      const double U = rint(km);
      if (U > 256.0 || 2.0 * K - U > 256.0) continue;
      const double v = (km - U) * (1.0 / 128.0);
      const double err = fabs((double)bf16_to_float(bf16_bits_rne((float)v)) - v) / (double)K;
      if (err < best) {  // K descends: ties keep the larger K
        best = err;
        bk = K;
      }
    }
    for (int o = 32; o > 0; o >>= 1) {
      const double ob = __shfl_xor(best, o);
      const int ok2 = __shfl_xor(bk, o);
      if (ob < best || (ob == best && ok2 > bk)) {
        best = ob;
        bk = ok2;
      }
    }
    const double Kd = (double)bk, U = rint(Kd * mu);
    gs = Kd / 128.0;
    c = U / Kd;
    vmiss = (Kd * mu - U) * (1.0 / 128.0);
    for (int g = 0; g < 3; ++g) vg[g] = ((double)g * Kd - U) * (1.0 / 128.0);
  } else if (ok) {
    const double grid = f16_scaled(a.prec) ? 512.0 : 64.0;
    c = rint(grid * mu) / grid;
    vmiss = mu - c;
    for (int g = 0; g < 3; ++g) vg[g] = (double)g - c;
  }
  if (lane != 0) return;
  MarkerStat st;
  st.flags = ok ? 0 : 1;
  st.mu = mu;
  st.shift = c;
  st.gscale = (float)gs;
  // the FP8 lo pass of the FP16 + FP8 form may centre on the integer c8 =
  // rint(c): its calls' values g - c8 are then exact in e4m3 and, being
  // small integers, cheaper in matrix-core power; a missing call's mu - c8
  // rounds to e4m3, an error that the lo term of y~ (about 2^-12 of y~)
  // keeps below about 2^-17 of a genotype unit.  The shift (c - c8) times
  // the column's sum of lo terms leaves through the last correction slot.
  const double c8 = (a.prec == kSplit8 && a.lo_int) ? rint(c) : c;
  st.dlo = (float)(c - c8);  // a multiple of 1/512 in [-1/2, 1/2]: exact
  st.gc2 = n_obs > 0 ? (double)num / (double)n_obs : 0.0;
  st.dmu = (float)vmiss;
  // operand value of each 2-bit code, in the coding scheme's code order
  double val[4];
  if (a.code == 0) {
    val[0] = vg[0]; val[1] = vg[1]; val[2] = vg[2]; val[3] = vmiss;
  } else {
    val[0] = vg[0]; val[1] = vmiss; val[2] = vg[1]; val[3] = vg[2];
  }
  uint4 lut;
  if (a.prec != kFP32) {
    uint32_t lo8 = 0, hi8 = 0, f8 = 0;
    for (int k = 0; k < 4; ++k) {
      const uint32_t b = a.prec == kSplit ? bf16_bits_rne((float)val[k]) : f16_bits_rn((float)val[k]);
      lo8 |= (b & 0xffu) << (8 * k);
      hi8 |= (b >> 8) << (8 * k);
      f8 |= e4m3_bits_rne(val[k] + (c - c8)) << (8 * k);  // g - c8, or mu - c8, rounded to e4m3
    }
    lut = make_uint4(lo8, hi8, f8, 0u);
  } else {
    lut = make_uint4(__float_as_uint((float)val[0]), __float_as_uint((float)val[1]),
                     __float_as_uint((float)val[2]), __float_as_uint((float)val[3]));
  }
  a.mlut[m] = lut;
  a.mstat[m] = st;
}

__global__ void debug_stats_kernel(const MarkerStat* ms, int64_t nm, double* shift, double* mean, double* scale) {
  const int64_t m = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (m >= nm) return;
  if (shift) shift[m] = ms[m].shift;
  if (mean) mean[m] = ms[m].mu;
  if (scale) scale[m] = (double)ms[m].gscale;
}

// ---------------------------------------------------------------------------
// ||g_res||^2 per (marker, panel) from Q^T g; slot 0 <- mu - c
// ---------------------------------------------------------------------------
__global__ void finalize_kernel(const MarkerStat* __restrict__ ms, float* __restrict__ wws,
                                float2* __restrict__ invh, int64_t nm, int n_panels, float wscale, int lo_slot,
                                RedoDev redo) {
  const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (idx >= nm * n_panels) return;
  const int64_t m = idx / n_panels;
  invh[idx] = finalize_row(ms[m], wws + idx * kSlots, wscale, lo_slot, redo, (int)(idx - m * n_panels), (int32_t)m);
}

// ---------------------------------------------------------------------------
// per-call output table, tail list
// ---------------------------------------------------------------------------
__global__ void bind_kernel(BindArgs a) {
  const int i = threadIdx.x;
  if (i < a.count) a.dst[a.first + i] = a.outs[i];
}

__global__ void tail_reset_kernel(TailDev t) {
  if (threadIdx.x == 0 && blockIdx.x == 0) t.count[0] = 0ull;
}

__global__ void tail_kernel(TailDev t, const PanelDev* __restrict__ panels, const OutDev* __restrict__ outs,
                            HitDev hits, int64_t m_begin) {
  const unsigned long long cnt = t.count[0];
  const int64_t n = cnt < (unsigned long long)t.capacity ? (int64_t)cnt : t.capacity;
  for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < n;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const TailEntry e = t.entries[idx];
    const double df = (double)panels[e.panel].df;
    const double r = (double)e.r;
    const double tt = r * sqrt(df / ((1.0 - r) * (1.0 + r)));
    const double lnp = ln_p_two_sided(tt, df);
    const float nl = (float)(-lnp / M_LN10);
    const OutDev o = outs[e.panel];
    if (o.nl) o.nl[e.row * o.ld + e.col] = nl;
    if (o.best) atomicMax(o.best + e.col, best_pack(nl, m_begin + e.row));  // replaces the lower bound
    if (hits.entries && nl >= hits.threshold) append_hit(hits, m_begin + e.row, e.panel, e.col, nl, e.r);
  }
}

// ---------------------------------------------------------------------------
// FP64 path of covariate-collinear markers (the ones finalize_row lists):
// each listed marker is mean-imputed and residualized explicitly against its
// panel's FP64 Q, g_res = g_imp - Q (Q^T g_imp), then contracted in FP64 with
// the stored panel operand, so that r = g_res^T y_op / (||g_res|| ||(I -
// QQ^T) y_op||) carries no cancellation; t, beta, SE as in the main epilogue
// (Eq. 3), -log10 p in FP64 for every test, and the reduced outputs.  A
// marker with ||g_res||^2 <= kCollinearTol ||g_c||^2 gives NaN rows.  One
// work item: up to kRedoGroup listed markers of one panel x kRedoCols of its
// columns, walked by a persistent grid; the work list comes from the
// per-panel counts, so a block without listed markers costs one short launch.
//
// All three products of an item run on the FP64 matrix cores
// (v_mfma_f64_16x16x4_f64, 68 cycles, the FP64 rate of the vector FMA without
// its operand traffic): Q^T g (16 slots x 16 markers), the residual g - Q w of
// 16 samples x 16 markers, whose accumulator layout is the next product's
// operand as it stands, and g_res^T y (16 markers x 64 columns).  The
// 64-sample chunks are cut into kRedoWaves contiguous ranges, one per wave,
// and the waves' sums are added in wave order, so that a marker's result
// depends on neither the list nor the grid.  A lane reads two or three dwords
// of the panel operand per four values.  600 listed markers x 300 phenotypes
// at N = 23,000, K = 13: 15.7 ms with one column per thread and scalar
// operand reads, 0.64 ms here.
// ---------------------------------------------------------------------------
constexpr int kRedoWaves = 16;
constexpr int kRedoThreads = 64 * kRedoWaves;
static_assert(kRedoGroup == 16 && kRedoCols == 64 && kRedoThreads == kRedoGroup * kRedoCols, "redo shape");

// a listed marker's genotype row: 2-bit codes (map: the calls of codes 0..3,
// two bits each; miss: the missing code) or 8-bit dosages
struct RedoRow {
  const uint8_t* row;
  double mu;
  uint32_t map, miss;
};
// samples 16 b + 4 i + l4, i = 0..3 (RUN: 16 b + 4 l4 + i), of the chunk at
// row r.row in genotype units (8-bit dosages: q); missing calls take mu,
// samples past the first ns of the chunk are zero
template <bool G8, bool RUN>
__device__ __forceinline__ f64x4 geno_block(const RedoRow& r, int b, int l4, int ns) {
  f64x4 g;
  uint32_t v[4];
  if constexpr (G8) {
    if constexpr (RUN) {
      const uint32_t w = gload<uint32_t>(r.row + 16 * b + 4 * l4);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = (w >> (8 * i)) & 0xffu;
    } else {
      const u32x4 w = gload<u32x4>(r.row + 16 * b);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = (w[i] >> (8 * l4)) & 0xffu;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) g[i] = v[i] == 255u ? r.mu : (double)v[i];
  } else {
    const uint32_t w = gload<uint32_t>(r.row + 4 * b) >> (RUN ? 8 * l4 : 2 * l4);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[i] = (w >> (RUN ? 2 * i : 8 * i)) & 3u;
      g[i] = v[i] == r.miss ? r.mu : (double)((r.map >> (2 * v[i])) & 3u);
    }
  }
  if (ns < kChunk) {  // uniform: the last chunk of a ragged cohort
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (16 * b + (RUN ? 4 * l4 + i : 4 * i + l4) >= ns) g[i] = 0.0;
  }
  return g;
}

// the operand values of samples 16 b + 4 i + l4 of one column, in the units
// the main kernel contracts (2^12 y~ for the FP16 forms), i.e. what
// prep_kernel accumulated into the column's norm and projections.  blk: the
// column block's chunk; lane: 16 (column within the block) + 4 l4.
template <int PREC>
__device__ __forceinline__ f64x4 operand_block(const char* blk, int b, uint32_t lane, double lo_unit) {
  f64x4 y;
  const char* p = blk + (b >> 1) * 512;
  if constexpr (PREC == kFP32) {
#pragma unroll
    for (int i = 0; i < 4; ++i) y[i] = (double)gload<float>(p + (4 * (b & 1) + i) * 1024 + lane);
  } else {
    // dword l4 of step j = 2 (b & 1) + (i & 1): samples i (low half) and i + 2
    const uint32_t h0 = gload<uint32_t>(p + 2 * (b & 1) * 1024 + lane);
    const uint32_t h1 = gload<uint32_t>(p + 2 * (b & 1) * 1024 + 1024 + lane);
    const uint32_t hv[4] = {h0 & 0xffffu, h1 & 0xffffu, h0 >> 16, h1 >> 16};
    if constexpr (PREC == kSplit8) {  // byte i of dword l4
      const int lo = (int)gload<uint32_t>(p + 4096 + (b & 1) * 1024 + lane);
      const float lv[4] = {__builtin_amdgcn_cvt_f32_fp8(lo, 0), __builtin_amdgcn_cvt_f32_fp8(lo, 1),
                           __builtin_amdgcn_cvt_f32_fp8(lo, 2), __builtin_amdgcn_cvt_f32_fp8(lo, 3)};
#pragma unroll
      for (int i = 0; i < 4; ++i) y[i] = fma((double)lv[i], lo_unit, (double)f16_to_float(hv[i]));
    } else {
      const uint32_t l0 = gload<uint32_t>(p + 4096 + 2 * (b & 1) * 1024 + lane);
      const uint32_t l1 = gload<uint32_t>(p + 4096 + 2 * (b & 1) * 1024 + 1024 + lane);
      const uint32_t lv[4] = {l0 & 0xffffu, l1 & 0xffffu, l0 >> 16, l1 >> 16};
#pragma unroll
      for (int i = 0; i < 4; ++i)
        y[i] = PREC == kSplit16 ? (double)f16_to_float(hv[i]) + (double)f16_to_float(lv[i])
                                : (double)bf16_to_float(hv[i]) + (double)bf16_to_float(lv[i]);
    }
  }
  return y;
}

// FAR: a slot's column of Q can lie 4 GiB and more behind the first one.
// Addresses of 64 bits cost registers that the kernel does not have (it spills
// four to six more): 902 against 862 us for an analysis with one lead marker at
// N = 34,613, 1,993 markers x 27 phenotypes.
template <int PREC, bool G8, bool FAR>
__global__ __launch_bounds__(kRedoThreads) void redo_kernel(RedoArgs a) {
  using Offset = std::conditional_t<FAR, int64_t, uint32_t>;
  __shared__ double part[kRedoWaves][kRedoGroup * kRedoCols];  // the waves' sums: slots, then tests
  __shared__ double w_s[kSlots][kRedoGroup];
  __shared__ double h2_s[kRedoWaves][kRedoGroup];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, l4 = lane >> 4;
  constexpr int CB = G8 ? 64 : 16;  // bytes of a row's chunk
  const int ch_lo = (int)((int64_t)a.n_chunks * wave / kRedoWaves);
  const int ch_hi = (int)((int64_t)a.n_chunks * (wave + 1) / kRedoWaves);
  int64_t total = 0;
  for (int j = 0; j < a.n_panels; ++j)
    total += (int64_t)((a.redo.count[j] + kRedoGroup - 1) / kRedoGroup) * a.max_chunks;
  for (int64_t w = blockIdx.x; w < total; w += gridDim.x) {
    int64_t rem = w;
    int j = 0;
    uint32_t cnt = 0;
    for (; j < a.n_panels; ++j) {
      cnt = a.redo.count[j];
      const int64_t items = (int64_t)((cnt + kRedoGroup - 1) / kRedoGroup) * a.max_chunks;
      if (rem < items) break;
      rem -= items;
    }
    const int gi = (int)(rem / a.max_chunks);
    const int cc = (int)(rem - (int64_t)gi * a.max_chunks);
    const PanelDev pd = a.panels[j];
    if ((int64_t)cc * kRedoCols >= pd.n_pheno) continue;  // uniform over the workgroup
    const int ng = min(kRedoGroup, (int)cnt - gi * kRedoGroup);
    const int32_t* ent = a.redo.entries + j * a.redo.stride + (int64_t)gi * kRedoGroup;
    const int q = pd.q;
    // this lane's marker (past the group's end the last one again; its results are not stored)
    const int64_t mk = ent[l16 < ng ? l16 : ng - 1];
    RedoRow rr;
    rr.mu = a.mstat[mk].mu;
    rr.map = a.code == 1 ? 0x90u : 0x24u;  // .bed order: 0, missing, 1, 2; dosage order: 0, 1, 2, missing
    rr.miss = a.code == 1 ? 1u : 3u;
    const uint8_t* row0 = a.geno + (a.m0 + mk) * a.row_bytes;

    // w = Q^T g_imp: slots x markers
    {
      f64x4 acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
      // step i contracts samples 16 b + 4 l4 + i: a lane reads 32 bytes of its slot's column at once
      const Offset o0 = (Offset)((min(l16, q - 1) * a.n_pad + 4 * l4) * 8);
      const Offset o1 = (Offset)((min(l16 + 16, q - 1) * a.n_pad + 4 * l4) * 8);
      for (int ch = ch_lo; ch < ch_hi; ++ch) {
        const int ns = (int)min((int64_t)kChunk, a.n - (int64_t)ch * kChunk);
        const char* qc = (const char*)(pd.Q + (int64_t)ch * kChunk);
        rr.row = row0 + (int64_t)ch * CB;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const f64x4 g = geno_block<G8, true>(rr, b, l4, ns);
          const f64x4 qa = gload<f64x4>(qc + 128 * b + o0);
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[i], g[i], acc[0], 0, 0, 0);
          if (q > 16) {
            const f64x4 qb = gload<f64x4>(qc + 128 * b + o1);
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(qb[i], g[i], acc[1], 0, 0, 0);
          }
        }
      }
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) part[wave][(16 * t + 4 * i + l4) * kRedoGroup + l16] = acc[t][i];
    }
    __syncthreads();
    if (tid < kSlots * kRedoGroup) {
      const int k = tid >> 4;
      double v = 0.0;
#pragma unroll
      for (int x = 0; x < kRedoWaves; ++x) v += part[x][tid];
      w_s[k][tid & 15] = k < q ? v : 0.0;
    }
    __syncthreads();
    f64x4 S[4];
    double h2 = 0.0;
    {
      double nw[kSlots / 4];
#pragma unroll
      for (int kk = 0; kk < kSlots / 4; ++kk) nw[kk] = -w_s[4 * kk + l4][l16];
      Offset oq[kSlots / 4];
#pragma unroll
      for (int kk = 0; kk < kSlots / 4; ++kk) oq[kk] = (Offset)((min(4 * kk + l4, q - 1) * a.n_pad + l16) * 8);
      // the item's two 32-column blocks (columns past the panel's padded end
      // read the first block again; their results are not stored)
      constexpr int BB = block_bytes(PREC);
      const int64_t cb0 = (int64_t)cc * 2, cb1 = cb0 * 32 + 32 < pd.n_pheno ? cb0 + 1 : cb0;
      const char* yb[2] = {(const char*)pd.yop + cb0 * a.n_chunks * BB, (const char*)pd.yop + cb1 * a.n_chunks * BB};
      double unit[4];
#pragma unroll
      for (int ct = 0; ct < 4; ++ct) {
        S[ct] = f64x4{0.0, 0.0, 0.0, 0.0};
        unit[ct] = PREC == kSplit8
                       ? ldexp(1.0, (int)pd.lscale[(ct < 2 ? cb0 : cb1) * 32 + 16 * (ct & 1) + l16] - 127)
                       : 1.0;
      }
      const uint32_t ylane = l16 * 16 + 4 * l4;
      for (int ch = ch_lo; ch < ch_hi; ++ch) {
        const int ns = (int)min((int64_t)kChunk, a.n - (int64_t)ch * kChunk);
        const char* qc = (const char*)(pd.Q + (int64_t)ch * kChunk);
        const char* yc[2] = {yb[0] + (int64_t)ch * BB, yb[1] + (int64_t)ch * BB};
        rr.row = row0 + (int64_t)ch * CB;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          f64x4 res = geno_block<G8, false>(rr, b, l4, ns);
#pragma unroll
          for (int kk = 0; kk < kSlots / 4; ++kk)
            if (4 * kk < q)
              res = __builtin_amdgcn_mfma_f64_16x16x4f64(gload<double>(qc + 128 * b + oq[kk]), nw[kk], res, 0, 0, 0);
#pragma unroll
          for (int ct = 0; ct < 4; ++ct) {
            const f64x4 y = operand_block<PREC>(yc[ct >> 1], b, 256 * (ct & 1) + ylane, unit[ct]);
#pragma unroll
            for (int i = 0; i < 4; ++i) S[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(res[i], y[i], S[ct], 0, 0, 0);
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) h2 += res[i] * res[i];
        }
      }
    }
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
      for (int i = 0; i < 4; ++i) part[wave][(4 * i + l4) * kRedoCols + 16 * ct + l16] = S[ct][i];
    h2 += __shfl_xor(h2, 16);
    h2 += __shfl_xor(h2, 32);
    if (l4 == 0) h2_s[wave][l16] = h2;
    __syncthreads();
#pragma unroll
    for (int x = 0; x < kRedoGroup * kRedoCols / kRedoThreads; ++x) {
      const int idx = tid + x * kRedoThreads;
      const int e = idx / kRedoCols;
      const int64_t p = (int64_t)cc * kRedoCols + idx % kRedoCols;
      if (e >= ng || p >= pd.n_pheno) continue;
      double s = 0.0, n2 = 0.0;
#pragma unroll
      for (int x = 0; x < kRedoWaves; ++x) {
        s += part[x][idx];
        n2 += h2_s[x][e];
      }
      const double invny = (double)pd.invny[p];
      const double sp = (double)pd.scale[p] * (double)a.gunit;
      const double df = (double)pd.df;
      const OutDev od = a.outs[j];
      const int64_t m = ent[e];
      const int64_t orow = a.out_row0 + m;
      const bool ok = n2 > kCollinearTol * a.mstat[m].gc2 && invny == invny;
      double r = __builtin_nan(""), t = r, beta = r, se = r, nl = r;
      if (ok) {
        const double ih = 1.0 / sqrt(n2);
        r = s * invny * ih;
        r = r > 1.0 ? 1.0 : (r < -1.0 ? -1.0 : r);
        const double omr2 = (1.0 - r) * (1.0 + r);
        t = omr2 > 0.0 ? r * sqrt(df / omr2) : (r > 0.0 ? INFINITY : -INFINITY);
        beta = r * sp * ih;
        se = sp * ih * sqrt(omr2 / df);
        nl = -ln_p_two_sided(t, df) / M_LN10;
      }
      const int64_t o = orow * od.ld + p;
      if (od.r) od.r[o] = (float)r;
      if (od.beta) od.beta[o] = (float)beta;
      if (od.se) od.se[o] = (float)se;
      if (od.t) od.t[o] = (float)t;
      if (od.nl) od.nl[o] = (float)nl;
      if (ok && od.best) atomicMax(od.best + p, best_pack((float)nl, a.m_begin + orow));
      if (ok && od.topk) topk_insert(od.topk + p * od.topk_k, od.topk_k, topk_pack((float)fabs(t), a.m_begin + orow));
      if (ok && a.hits.entries && (float)nl >= a.hits.threshold)
        append_hit(a.hits, a.m_begin + orow, j, p, (float)nl, (float)r);
    }
    __syncthreads();  // the sums are rewritten by the next work item
  }
}

// ---------------------------------------------------------------------------
// the contraction (Eq. 2) with the fused epilogue
//
// Workgroup tile: TM = NW * WMF * 32 markers x TP = WN * 32 columns; every
// wave owns WMF 32-row fragments across all WN column blocks.  K loop over
// 64-sample chunks: the column tile's operand chunk is double-buffered in
// LDS; each wave reads its markers' packed codes straight from global memory
// and decodes them in registers with v_perm_b32 and the per-marker table.
// Persistent: the grid is resident and walks the (marker tile, column tile)
// list; the list is cut into 8 contiguous ranges, one per XCD (workgroups
// are dispatched round-robin to XCDs), so that the workgroups of an XCD
// share column tiles in their L2.
// ---------------------------------------------------------------------------
//
// G8: the rows hold 8-bit dosages, one byte per sample; each lane half reads
// its 32 bytes of the chunk and builds FP16 q - c by inserting the byte under
// the exponent of 1024 and subtracting 1024 + c (exact for integers below
// 2048), or FP32 q - c; a missing byte takes the marker's mu - c.
template <int PREC, int NW, int WMF, int WN, int MODE, bool G8 = false>
__global__ __launch_bounds__(NW * 64) void gemm_kernel(GemmArgs a) {
  static_assert(!G8 || PREC == kFP32 || PREC == kSplit16, "8-bit dosages run the FP32 and FP16 split forms here");
  constexpr int NT = NW * 64;
  constexpr int TM = NW * WMF * 32;
  constexpr int TILE_BYTES = WN * kBlockBytes;
  constexpr int RPB = kBlockBytes / 16 / NT;  // 16-byte pieces per thread per block
  static_assert(kBlockBytes % (16 * NT) == 0, "block copy must divide evenly");
  constexpr int STAGE_BYTES = MODE == kTest ? NW * WMF * 32 * 32 * 4 : 0;
  constexpr int LDS_BYTES = 2 * TILE_BYTES > STAGE_BYTES ? 2 * TILE_BYTES : STAGE_BYTES;
  __shared__ __attribute__((aligned(16))) char smem[LDS_BYTES];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int h = lane >> 5;
  const int r32 = lane & 31;

  const int G = gridDim.x;
  const int b = blockIdx.x;
  const int xcd = b & 7;
  const int slot = b >> 3;
  const int nslots = G >> 3;
  const int64_t W = (int64_t)a.n_mtiles * a.n_ctiles;
  const int64_t wlo = W * xcd / 8;
  const int64_t whi = W * (xcd + 1) / 8;

  for (int64_t w = wlo + slot; w < whi; w += nslots) {
    int mtile, ctile;
    grouped_tile(w, a.n_mtiles, a.n_ctiles, mtile, ctile);

    // operand blocks of this column tile; blocks past the end alias the
    // first one (their columns are never written)
    const char* bop[WN];
#pragma unroll
    for (int fn = 0; fn < WN; ++fn) {
      const int cb = ctile * WN + fn;
      bop[fn] = a.cblocks[cb < a.n_cblocks ? cb : ctile * WN].op;
    }
    const int64_t rowbase = (int64_t)mtile * TM + wave * (WMF * 32);
    const uint8_t* ap[WMF];
    uint4 lut[WMF];
#pragma unroll
    for (int fm = 0; fm < WMF; ++fm) {
      int64_t mr = rowbase + fm * 32 + r32;
      mr = mr < a.nm ? mr : a.nm - 1;
      ap[fm] = a.geno + (a.m0 + mr) * a.row_bytes + (G8 ? 32 : 8) * h;
      lut[fm] = gload<uint4>(a.mlut + mr);
    }

    f32x16 acc[WMF][WN];
#pragma unroll
    for (int fm = 0; fm < WMF; ++fm)
#pragma unroll
      for (int fn = 0; fn < WN; ++fn)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[fm][fn][i] = 0.0f;

    u32x4 breg[WN][RPB];
    // this lane's genotype bytes of the chunk: 8 (2-bit codes) or 32 (dosages).
    // The 32-column shapes do little work per
    // chunk, so it keeps a ring of AD chunks of its rows in flight to cover
    // the memory latency (the chunk loop is unrolled by AD so that the ring
    // is indexed statically); the others keep one chunk ahead.
    constexpr int AD = WN == 1 ? (G8 ? 2 : 4) : 1;
    struct ARow {
      u32x4 q[G8 ? 2 : 1];
    };
    auto load_b = [&](int ch) {
#pragma unroll
      for (int fn = 0; fn < WN; ++fn)
#pragma unroll
        for (int q = 0; q < RPB; ++q)
          breg[fn][q] = gload<u32x4>(bop[fn] + (int64_t)ch * kBlockBytes + (q * NT + tid) * 16);
    };
    auto store_b = [&](int buf) {
#pragma unroll
      for (int fn = 0; fn < WN; ++fn)
#pragma unroll
        for (int q = 0; q < RPB; ++q) *(u32x4*)(smem + buf * TILE_BYTES + fn * kBlockBytes + (q * NT + tid) * 16) = breg[fn][q];
    };
    auto load_a = [&](int ch, ARow* dst) {
#pragma unroll
      for (int fm = 0; fm < WMF; ++fm) {
        if constexpr (G8) {
          dst[fm].q[0] = gload<u32x4>(ap[fm] + (int64_t)ch * 64);
          dst[fm].q[1] = gload<u32x4>(ap[fm] + (int64_t)ch * 64 + 16);
        } else {
          const uint2 v = gload<uint2>(ap[fm] + (int64_t)ch * 16);
          dst[fm].q[0][0] = v.x;
          dst[fm].q[0][1] = v.y;
        }
      }
    };
    // dword k (4 samples) of this lane's dosage bytes
    auto dword8 = [&](const ARow& r, int k) -> uint32_t { return k < 4 ? r.q[0][k] : r.q[G8 ? 1 : 0][k & 3]; };

    // one chunk's decode and matrix-core steps on the staged operand tile cur
    auto compute = [&](const int cur, const ARow* areg, const int half) __attribute__((always_inline)) {
      const char* tile = smem + cur * TILE_BYTES + half * (kBlockBytes / 2);
      if constexpr (PREC != kFP32) {
        u32x4 bh[WN], bl[WN];
#pragma unroll
        for (int fn = 0; fn < WN; ++fn) {
          bh[fn] = *(const u32x4*)(tile + fn * kBlockBytes + (lane * 8) * 2);
          bl[fn] = *(const u32x4*)(tile + fn * kBlockBytes + (2048 + lane * 8) * 2);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          u32x4 A[WMF];
#pragma unroll
          for (int fm = 0; fm < WMF; ++fm) {
            if constexpr (G8) {
              // slots (2d, 2d+1) of step j take samples 16 (j >> 1) + 4 (j & 1) + d
              // and that + 8 of this lane half: byte d of dwords k0 and k0 + 2
              const int k0 = 4 * (j >> 1) + (j & 1);
              const uint32_t D0 = dword8(areg[fm], k0), D1 = dword8(areg[fm], k0 + 2);
              const uint32_t M0 = ff_bytes(D0), M1 = ff_bytes(D1);
#pragma unroll
              for (int d = 0; d < 4; ++d) {
                const uint32_t x = __builtin_amdgcn_perm(D1, D0, 0x0c000c00u | ((4u + d) << 16) | d) | 0x64006400u;
                const uint32_t v = __builtin_bit_cast(uint32_t, __builtin_bit_cast(f16x2, x) +
                                                                    __builtin_bit_cast(f16x2, lut[fm].x));
                const uint32_t mk = __builtin_amdgcn_perm(M1, M0, d | (d << 8) | ((4u + d) << 16) | ((4u + d) << 24));
                A[fm][d] = (mk & lut[fm].y) | (~mk & v);
              }
            } else {
              const uint32_t src = (j < 2) ? areg[fm].q[0][0] : areg[fm].q[0][1];
#pragma unroll
              for (int d = 0; d < 4; ++d) {
                const int t = 4 * (j & 1) + d;
                const uint32_t R = (src >> (2 * t)) & 0x00030003u;
                const uint32_t sel = R * 0x101u + 0x04000400u;
                A[fm][d] = __builtin_amdgcn_perm(lut[fm].y, lut[fm].x, sel);
              }
            }
          }
          u32x4 nh[WN], nl[WN];
          if (j < 3) {
#pragma unroll
            for (int fn = 0; fn < WN; ++fn) {
              nh[fn] = *(const u32x4*)(tile + fn * kBlockBytes + ((j + 1) * 512 + lane * 8) * 2);
              nl[fn] = *(const u32x4*)(tile + fn * kBlockBytes + (2048 + (j + 1) * 512 + lane * 8) * 2);
            }
          }
#pragma unroll
          for (int fn = 0; fn < WN; ++fn)
#pragma unroll
            for (int fm = 0; fm < WMF; ++fm) acc[fm][fn] = mfma16<PREC>(A[fm], bh[fn], acc[fm][fn]);
#pragma unroll
          for (int fn = 0; fn < WN; ++fn)
#pragma unroll
            for (int fm = 0; fm < WMF; ++fm) acc[fm][fn] = mfma16<PREC>(A[fm], bl[fn], acc[fm][fn]);
          if (j < 3) {
#pragma unroll
            for (int fn = 0; fn < WN; ++fn) {
              bh[fn] = nh[fn];
              bl[fn] = nl[fn];
            }
          }
        }
      } else {
        uint64_t bits[WMF];
#pragma unroll
        for (int fm = 0; fm < WMF; ++fm) bits[fm] = (uint64_t)areg[fm].q[0][0] | ((uint64_t)areg[fm].q[0][1] << 32);
#pragma unroll
        for (int j4 = 0; j4 < 8; ++j4) {
          float4 bv[WN];
#pragma unroll
          for (int fn = 0; fn < WN; ++fn)
            bv[fn] = *(const float4*)(tile + fn * kBlockBytes + (j4 * 256 + lane * 4) * 4);
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) {
            const int j = j4 * 4 + jj;
            float av[WMF];
#pragma unroll
            for (int fm = 0; fm < WMF; ++fm) {
              if constexpr (G8) {  // sample 32 h + j: byte j of this lane half's 32
                const uint32_t q = (dword8(areg[fm], j >> 2) >> (8 * (j & 3))) & 0xffu;
                av[fm] = q == 0xffu ? __uint_as_float(lut[fm].w) : (float)q - __uint_as_float(lut[fm].z);
              } else {
                const uint32_t c = (uint32_t)(bits[fm] >> (2 * j)) & 3u;
                const uint32_t lo = (c & 1u) ? lut[fm].y : lut[fm].x;
                const uint32_t hi = (c & 1u) ? lut[fm].w : lut[fm].z;
                av[fm] = __uint_as_float((c & 2u) ? hi : lo);
              }
            }
#pragma unroll
            for (int fn = 0; fn < WN; ++fn) {
              const float bb = jj == 0 ? bv[fn].x : jj == 1 ? bv[fn].y : jj == 2 ? bv[fn].z : bv[fn].w;
#pragma unroll
              for (int fm = 0; fm < WMF; ++fm)
                acc[fm][fn] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[fm], bb, acc[fm][fn], 0, 0, 0);
            }
          }
        }
      }
    };

    const int nch = a.n_chunks;
    if constexpr (AD == 1) {
      ARow areg[WMF], anext[WMF];
      load_b(0);
      load_a(0, areg);
      store_b(0);
      __syncthreads();
      for (int ch = 0; ch < nch; ++ch) {
        const int cur = ch & 1;
        const bool more = ch + 1 < nch;
        if (more) {
          load_b(ch + 1);
          load_a(ch + 1, anext);
        }
        compute(cur, areg, 0);
        if (more) store_b(cur ^ 1);
        __syncthreads();
#pragma unroll
        for (int fm = 0; fm < WMF; ++fm) areg[fm] = anext[fm];
      }
    } else {
      // ring[u] holds the rows of chunk ch0 + u and bring[v] the operand
      // block of the chunk after it that is v mod AD (ch0 a multiple of AD,
      // so chunk ch sits in LDS buffer ch & 1).  Each is refilled once used,
      // with the chunk AD later (the last chunk again past the end: a valid
      // address whose bytes are not used).  A chunk's operand block is
      // requested AD chunks before it is copied to LDS, after that chunk's
      // rows: waiting for it waits only for requests AD chunks old, so AD
      // chunks of rows stay in flight (the wait counter is in order).
      ARow ring[AD][WMF];
      u32x4 bring[AD][WN][RPB];
      auto load_b_to = [&](int ch, u32x4 (*dst)[RPB]) {
#pragma unroll
        for (int fn = 0; fn < WN; ++fn)
#pragma unroll
          for (int q = 0; q < RPB; ++q)
              dst[fn][q] = gload<u32x4>(bop[fn] + (int64_t)ch * kBlockBytes + (q * NT + tid) * 16);
      };
      auto store_b_from = [&](int buf, u32x4 (*src)[RPB]) {
#pragma unroll
        for (int fn = 0; fn < WN; ++fn)
#pragma unroll
          for (int q = 0; q < RPB; ++q)
              *(u32x4*)(smem + buf * TILE_BYTES + fn * kBlockBytes + (q * NT + tid) * 16) = src[fn][q];
      };
      auto clamp = [&](int ch) { return ch < nch ? ch : nch - 1; };
      load_b_to(0, bring[0]);
      store_b_from(0, bring[0]);
#pragma unroll
      for (int u = 0; u < AD; ++u) {
        load_a(clamp(u), ring[u]);
        load_b_to(clamp(u + 1), bring[(u + 1) % AD]);
      }
      __syncthreads();
      // whole rounds of AD chunks, with no branch inside a round (a branch
      // per chunk left the compiler waiting for every request in flight)
      const int nfull = nch / AD * AD;
      for (int ch0 = 0; ch0 < nfull; ch0 += AD) {
#pragma unroll
        for (int u = 0; u < AD; ++u) {
          const int ch = ch0 + u;
          compute(u & 1, ring[u], 0);
          load_a(clamp(ch + AD), ring[u]);
          store_b_from((u & 1) ^ 1, bring[(u + 1) % AD]);  // chunk ch + 1 (a repeat of the last past the end)
          load_b_to(clamp(ch + 1 + AD), bring[(u + 1) % AD]);
          __syncthreads();
        }
      }
      // the last nch - nfull < AD chunks (chunk nfull + u in ring[u], its
      // successor's operand block in bring[(u + 1) % AD])
#pragma unroll
      for (int u = 0; u < AD - 1; ++u) {
        const int ch = nfull + u;
        if (ch < nch) {
          compute(u & 1, ring[u], 0);
          if (ch + 1 < nch) store_b_from((u & 1) ^ 1, bring[(u + 1) % AD]);
          __syncthreads();
        }
      }
    }

    // ---------------------------------------------------------------- epilogue
    if constexpr (MODE == kRaw) {
#pragma unroll
      for (int fn = 0; fn < WN; ++fn) {
        const int cb = ctile * WN + fn;
        if (cb >= a.n_cblocks) continue;
        const ColBlock blk = a.cblocks[cb];
        if (r32 >= blk.ncol) continue;
#pragma unroll
        for (int fm = 0; fm < WMF; ++fm)
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int64_t mr = rowbase + fm * 32 + 8 * (i >> 2) + 4 * h + (i & 3);
            if (mr < a.nm) gstore(a.raw_out + mr * a.raw_ld + blk.col0 + r32, acc[fm][fn][i]);
          }
      }
    } else {
      // correction: acc += sum_slot w[m][slot] * cw[p][slot]
      //   = -(mu - c) sum_i y_op,i - sum_{k>=1} (q_k^T g)(q_k^T y_op)
      // i.e. the intercept and covariate components of the projection
      // (I - QQ^T) applied to the stored operand.  Small term: one BF16
      // matrix-core pass over 32 slots.
#pragma unroll
      for (int fn = 0; fn < WN; ++fn) {
        const int cb = ctile * WN + fn;
        const ColBlock blk = a.cblocks[cb < a.n_cblocks ? cb : ctile * WN];
        const float* cwp = a.panels[blk.panel].cw + (int64_t)(blk.col0 + r32) * kSlots + 8 * h;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          const float4 c0 = gload<float4>(cwp + 16 * ks);
          const float4 c1 = gload<float4>(cwp + 16 * ks + 4);
          u32x4 bo;
          bo[0] = pack_bf16x2(c0.x, c0.y);
          bo[1] = pack_bf16x2(c0.z, c0.w);
          bo[2] = pack_bf16x2(c1.x, c1.y);
          bo[3] = pack_bf16x2(c1.z, c1.w);
          const bf16x8 B = __builtin_bit_cast(bf16x8, bo);
#pragma unroll
          for (int fm = 0; fm < WMF; ++fm) {
            int64_t mr = rowbase + fm * 32 + r32;
            mr = mr < a.nm ? mr : a.nm - 1;
            const float* wp = a.wws + (mr * a.n_panels + blk.panel) * kSlots + 16 * ks + 8 * h;
            const float4 w0 = gload<float4>(wp);
            const float4 w1 = gload<float4>(wp + 4);
            u32x4 ao;
            ao[0] = pack_bf16x2(w0.x, w0.y);
            ao[1] = pack_bf16x2(w0.z, w0.w);
            ao[2] = pack_bf16x2(w1.x, w1.y);
            ao[3] = pack_bf16x2(w1.z, w1.w);
            acc[fm][fn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ao), B,
                                                                  acc[fm][fn], 0, 0, 0);
          }
        }
      }
      // stage one 32-column slice of the accumulators at a time through this
      // wave's 8 KiB of LDS (the B buffers are free now), then finish the
      // tests in a plain loop: lanes run along columns, so every output row
      // segment is one 128-byte store per half-wave.
      float* stage = (float*)smem + wave * (WMF * 32 * 32);
#pragma unroll
      for (int fn = 0; fn < WN; ++fn) {
        const int cb = ctile * WN + fn;
        if (cb >= a.n_cblocks) break;
#pragma unroll
        for (int fm = 0; fm < WMF; ++fm)
#pragma unroll
          for (int i = 0; i < 16; ++i)
            stage[(fm * 32 + 8 * (i >> 2) + 4 * h + (i & 3)) * 32 + r32] = acc[fm][fn][i];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const ColBlock blk = a.cblocks[cb];
        const PanelDev& pdb = a.panels[blk.panel];
        const bool colok = r32 < blk.ncol;
        const float invny = colok ? gload<float>(pdb.invny + blk.col0 + r32) : 0.f;
        const float sp = colok ? gload<float>(pdb.scale + blk.col0 + r32) * a.gunit : 0.f;
        finish_block<WMF>(stage, a, blk, rowbase, h, r32, (const tab4*)pdb.table, GlobalRows{}, invny, sp);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
      __syncthreads();  // the next tile's prologue overwrites the staging area
    }
  }
}

// ---------------------------------------------------------------------------
// wide split-precision contraction: one wave per SIMD, each wave owns a
// 128 x 128 accumulator tile (256 FP32 accumulators, AGPRs); workgroup tile
// 512 markers x 128 columns.
//
// Operands move through an LDS ring, one 64-sample chunk per stage: the
// column tile's operand chunk and the packed codes of the tile's 512 markers
// (8 KiB), both copied with direct-to-LDS loads.  A chunk is requested
// NSTAGE - 1 chunks before it is used.  Within a chunk, step j's matrix-core
// instructions are interleaved with the LDS reads of step j+1's operand
// fragments and the decode of its genotypes, into the register set of the
// other parity.  One barrier per chunk, ahead of its last step: after it the
// next chunk has landed and every wave is done with this chunk's stage,
// which is refilled at once.
//
// Forms: the 16-bit splits run 2 x WMF x 4 MFMA 32x32x16 per step (hi and lo
// terms); FP16 hi + FP8 lo runs WMF x 4 FP16 MFMA per step plus a quarter of
// the chunk's block-scaled FP8 MFMA 32x32x64 (E8M0 scale of each column's lo
// term on the B side): with WMF = 4 those of marker fragment j, with WMF = 2
// those of column block j.
//
// Shapes: NW = 4, WMF = 4 (one wave per SIMD, 128 x 128 per wave, 256 AGPR
// accumulators) or NW = 8, WMF = 2 (two waves per SIMD, 64 x 128 per wave),
// so that one wave's genotype decode and epilogue overlap the other wave's
// matrix-core work.
// ---------------------------------------------------------------------------
typedef int i32x8 __attribute__((ext_vector_type(8)));

// s_waitcnt immediate: vmcnt(vm), lgkmcnt(0), expcnt unconstrained
constexpr int waitcnt_vm_lgkm0(int vm) { return (vm & 15) | ((vm >> 4) << 14) | (0x7 << 4); }
// vmcnt(vm) only (expcnt and lgkmcnt unconstrained)
constexpr int waitcnt_vm_only(int vm) { return waitcnt_vm_lgkm0(vm) | (0xF << 8); }

// G8: 8-bit dosage rows (FP16 split only): each stage holds the tile's 64
// bytes per marker; a lane reads the two dwords of its row that each K16 step
// needs and builds FP16 q - c as the register-staged kernel does.
// SEG: the accumulators are added up over segments (see kSegMin), one after the
// other, in this workgroup's part of a.part.  Each segment of a tile is a pass
// of its own through the tile loop, and moves 512 KiB against the 14 MiB that
// its chunks read (16,384 markers x 2,048 phenotypes, N = 70,001, whole scan:
// 5.66 ms with and without).
template <int PREC, int MODE, int NW, int WMF, int WN = 4, bool G8 = false, bool SEG = false>
__global__ __launch_bounds__(NW * 64) void gemm_wide_kernel(GemmArgs a) {
  static_assert(PREC != kFP32, "the wide kernel runs the split forms");
  static_assert(!G8 || PREC == kSplit16 || PREC == kSplit8, "8-bit dosages run the FP16 split forms here");
  static_assert((NW * WMF == 16 && WN == 4 && (WMF == 4 || WMF == 2)) ||
                    (NW == 4 && WMF == 2 && WN == 8 && PREC == kSplit8),
                "512 x 128 tiles, or 256 x 256 for the FP8 lo form");
  constexpr bool F8 = PREC == kSplit8;
  // 8-bit dosages in the FP16 + FP8 form: the FP8 lo operand is converted from
  // the FP16 values of the hi pass, a step at a time, and the chunk's lo
  // MFMAs run together at its last step
  constexpr bool GF = F8 && G8;
  constexpr bool W2 = WMF == 2;  // FP8 lo MFMAs by column block: both fragments, WN / 4 blocks per step
  constexpr int FNS = WN / 4;    // column blocks whose FP8 lo term runs at each step (WMF = 2)
  constexpr int NT = NW * 64;
  constexpr int TM = NW * WMF * 32;
  constexpr int BB = block_bytes(PREC);
  constexpr int NSTAGE = G8 ? 2 : (F8 ? (WN == 8 ? 3 : 4) : 3);
  constexpr int B_BYTES = WN * BB;  // operand chunk of the column tile
  constexpr int AB = G8 ? 64 : 16;  // bytes of a marker's chunk: 64 two-bit codes or 64 dosage bytes
  constexpr int A_BYTES = TM * AB;
  constexpr int STAGE_BYTES = B_BYTES + A_BYTES;
  constexpr int LDS_BYTES = NSTAGE * STAGE_BYTES;
  constexpr int PPB = BB / 1024;                // 1 KiB pieces per operand block
  constexpr int B_OPS = B_BYTES / (NT * 16);    // direct-to-LDS loads per wave per chunk
  constexpr int A_OPS = A_BYTES / (NT * 16);
  constexpr int CHUNK_OPS = B_OPS + A_OPS;
  constexpr int HI_MFMA = F8 ? WMF * WN : 2 * WMF * WN;  // 16-bit MFMA per step
  constexpr int DS_STEP = F8 ? WN : 2 * WN;              // fragment reads per step
  static_assert(NW * WMF * 32 * 32 * 4 <= LDS_BYTES, "epilogue staging must fit");
  static_assert((NSTAGE - 2) * CHUNK_OPS < 64, "vmcnt range");
  // past the stages: each row's 1/||g_res|| of the current column panel and,
  // where it fits, that panel's p-value table; the epilogue then reads
  // nothing from global memory between its output stores
  constexpr int IH_BYTES = TM * 8;
  constexpr int TAB_BYTES = kTabIntervals * 16;
  constexpr bool LT = LDS_BYTES + IH_BYTES + TAB_BYTES <= 160 * 1024;
  static_assert(WMF % 2 == 0 && LDS_BYTES + IH_BYTES <= 160 * 1024, "epilogue rows in LDS");
  __shared__ __attribute__((aligned(16))) char smem[LDS_BYTES + IH_BYTES + (LT ? TAB_BYTES : 0)];
  int tab_panel = -1;  // panel whose table is in LDS (uniform)

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int h = lane >> 5;
  const int r32 = lane & 31;

  const int G = gridDim.x;
  const int b = blockIdx.x;
  const int xcd = b & 7;
  const int slot = b >> 3;
  const int nslots = G >> 3;
  const int64_t W = (int64_t)a.n_mtiles * a.n_ctiles;
  const int64_t wlo = W * xcd / 8;
  const int64_t whi = W * (xcd + 1) / 8;

  int seg = 0;  // SEG: a tile's segments in turn
  for (int64_t w = wlo + slot; w < whi;) {
    int mtile, ctile;
    grouped_tile(w, a.n_mtiles, a.n_ctiles, mtile, ctile);
    const char* bop[WN];
    int bscale[WN];  // FP8 form: E8M0 scale of this lane's column, per block
#pragma unroll
    for (int fn = 0; fn < WN; ++fn) {
      const int cb = ctile * WN + fn;
      const ColBlock blk = a.cblocks[cb < a.n_cblocks ? cb : ctile * WN];
      bop[fn] = blk.op;
      bscale[fn] = 127;
      if constexpr (F8) {
        if (cb < a.n_cblocks && r32 < blk.ncol) bscale[fn] = a.panels[blk.panel].lscale[blk.col0 + r32];
      }
    }
    const int64_t rowbase = (int64_t)mtile * TM + wave * (WMF * 32);
    uint2 lut[WMF];
    uint32_t lut8[WMF];
#pragma unroll
    for (int fm = 0; fm < WMF; ++fm) {
      int64_t mr = rowbase + fm * 32 + r32;
      mr = mr < a.nm ? mr : a.nm - 1;
      if constexpr (F8) {
        const uint4 l4 = gload<uint4>(a.mlut + mr);
        lut[fm] = make_uint2(l4.x, l4.y);
        lut8[fm] = l4.z;
      } else {
        lut[fm] = gload<uint2>(a.mlut + mr);
        lut8[fm] = 0u;
      }
    }
    // code rows copied by this lane: markers rowbase + 64 k + lane (rows
    // past the end read the last row; their results are never stored)
    // (8-bit dosages: 16-byte piece 64 k + lane of the wave's rows, i.e.
    // quarter (64 k + lane) & 3 of marker rowbase + (64 k + lane) / 4)
    const uint8_t* arow[A_OPS];
#pragma unroll
    for (int k = 0; k < A_OPS; ++k) {
      const int piece = 64 * k + lane;
      int64_t mr = rowbase + (G8 ? piece >> 2 : piece);
      mr = mr < a.nm ? mr : a.nm - 1;
      arow[k] = a.geno + (a.m0 + mr) * a.row_bytes + (G8 ? (piece & 3) * 16 : 0);
    }

    f32x16 acc[WMF][WN];
#pragma unroll
    for (int fm = 0; fm < WMF; ++fm)
#pragma unroll
      for (int fn = 0; fn < WN; ++fn)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[fm][fn][i] = 0.0f;

    int nch = a.n_chunks, ch_lo = 0;  // chunks of the segment, its first chunk
    // chunk ch of the segment (clamped to the last one: the surplus copies land
    // in stages nobody reads again) into stage st
    auto dma = [&](int ch, int st) {
      ch = ch < nch ? ch : nch - 1;
      if constexpr (SEG) ch += ch_lo;
      char* stage = smem + st * STAGE_BYTES;
#pragma unroll
      for (int q = 0; q < B_OPS; ++q) {
        const int piece = q * NW + wave;  // 1 KiB piece of the operand chunk
        const int fn = piece / PPB;
        const int off = (piece % PPB) * 1024;
        __builtin_amdgcn_global_load_lds(
            (const __attribute__((address_space(1))) void*)(bop[fn] + (int64_t)ch * BB + off + lane * 16),
            (__attribute__((address_space(3))) void*)(stage + fn * BB + off), 16, 0, 0);
      }
#pragma unroll
      for (int k = 0; k < A_OPS; ++k)
        __builtin_amdgcn_global_load_lds(
            (const __attribute__((address_space(1))) void*)(arow[k] + (int64_t)ch * AB),
            (__attribute__((address_space(3))) void*)(stage + B_BYTES + wave * (WMF * 32 * AB) + k * 1024), 16, 0,
            0);
    };
    // whole 16-byte rows, this lane's half picked in registers (paired
    // 8-byte reads would be fused into one read that the compiler then holds
    // until every direct-to-LDS copy in flight has landed)
    auto read_a_raw = [&](int st, u32x4* raw) {
      const char* ab = smem + st * STAGE_BYTES + B_BYTES + wave * (WMF * 32 * 16);
#pragma unroll
      for (int fm = 0; fm < WMF; ++fm) raw[fm] = *(const u32x4*)(ab + (fm * 32 + r32) * 16);
    };
    auto pick_a = [&](const u32x4* raw, uint2* dst) {
#pragma unroll
      for (int fm = 0; fm < WMF; ++fm) dst[fm] = h ? make_uint2(raw[fm][2], raw[fm][3]) : make_uint2(raw[fm][0], raw[fm][1]);
    };
    auto read_a = [&](int st, uint2* dst) {
      u32x4 raw[WMF];
      read_a_raw(st, raw);
      pick_a(raw, dst);
    };
    // 8-bit dosages: dwords k0 and k0 + 2 (k0 = 4 (j >> 1) + (j & 1)) of this
    // lane half's 32 bytes of each fragment row, the two that K16 step j needs
    auto read_g8 = [&](int st, int j, uint2* dst) {
      const char* ab = smem + st * STAGE_BYTES + B_BYTES + wave * (WMF * 32 * 64) + h * 32;
      const int k0 = 4 * (j >> 1) + (j & 1);
#pragma unroll
      for (int fm = 0; fm < WMF; ++fm) {
        const char* row = ab + (fm * 32 + r32) * 64;
        dst[fm] = make_uint2(*(const uint32_t*)(row + 4 * k0), *(const uint32_t*)(row + 4 * (k0 + 2)));
      }
    };
    // slots (2d, 2d + 1) of step j take samples 16 (j >> 1) + 4 (j & 1) + d and
    // that + 8 of this lane half: byte d of the two dwords read above; FP16
    // q - c by inserting the byte under the exponent of 1024, a missing byte
    // takes mu - c
    auto decode_g8 = [&](const uint2* D, u32x4* A) {
#pragma unroll
      for (int fm = 0; fm < WMF; ++fm) {
        const uint32_t D0 = D[fm].x, D1 = D[fm].y;
        const uint32_t M0 = ff_bytes(D0), M1 = ff_bytes(D1);
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          const uint32_t x = __builtin_amdgcn_perm(D1, D0, 0x0c000c00u | ((4u + d) << 16) | d) | 0x64006400u;
          const uint32_t v =
              __builtin_bit_cast(uint32_t, __builtin_bit_cast(f16x2, x) + __builtin_bit_cast(f16x2, lut[fm].x));
          const uint32_t mk = __builtin_amdgcn_perm(M1, M0, d | (d << 8) | ((4u + d) << 16) | ((4u + d) << 24));
          A[fm][d] = (mk & lut[fm].y) | (~mk & v);
        }
      }
    };
    // 16-bit values of K16 step j: two per dword via the per-marker table
    auto decode = [&](const uint2* src2, int j, u32x4* A) {
#pragma unroll
      for (int fm = 0; fm < WMF; ++fm) {
        const uint32_t src = (j < 2) ? src2[fm].x : src2[fm].y;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          const int t = 4 * (j & 1) + d;
          const uint32_t R = (src >> (2 * t)) & 0x00030003u;
          const uint32_t sel = R * 0x101u + 0x04000400u;
          A[fm][d] = __builtin_amdgcn_perm(lut[fm].y, lut[fm].x, sel);
        }
      }
    };
    // e4m3 values of fragment fm over the whole chunk: four per dword
    auto decode8 = [&](const uint2* src2, int fm, i32x8& A8) {
#pragma unroll
      for (int part = 0; part < 2; ++part) {
        const uint32_t src = part ? src2[fm].y : src2[fm].x;
#pragma unroll
        for (int t = 0; t < 4; ++t)
          A8[4 * part + t] = (int)__builtin_amdgcn_perm(lut8[fm], lut8[fm], (src >> (2 * t)) & 0x03030303u);
      }
    };
    // FP16 hi + FP8 lo with WMF = 2: the 2-bit fields of a code dword spread
    // one per byte, Y[d] = (src >> 2d) & 0x03030303 for d = 0..3, are the e4m3
    // table selectors as they stand and, paired byte by byte with Y + 0x04040404
    // by one v_perm_b32, the FP16 table selectors; both decodes share one field
    // extraction.  Y of the first code dword (K16 steps 0, 1) is made at the
    // previous chunk's step 3, that of the second (steps 2, 3) at step 0.
    auto spread = [&](const uint2* src2, int p, uint32_t (*Y)[4]) {
#pragma unroll
      for (int fm = 0; fm < WMF; ++fm) {
        const uint32_t src = p ? src2[fm].y : src2[fm].x;
#pragma unroll
        for (int d = 0; d < 4; ++d) Y[fm][d] = (src >> (2 * d)) & 0x03030303u;
      }
    };
    // step j (of the dword that Y spreads): samples t = 4 (j & 1) + d and t + 8
    // sit in bytes (j & 1) and 2 + (j & 1) of Y[d]
    auto decode_y = [&](const uint32_t (*Y)[4], int j, u32x4* A) {
#pragma unroll
      for (int fm = 0; fm < WMF; ++fm)
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          const uint32_t y = Y[fm][d];
          const uint32_t sel = __builtin_amdgcn_perm(y + 0x04040404u, y, (j & 1) ? 0x07030501u : 0x06020400u);
          A[fm][d] = __builtin_amdgcn_perm(lut[fm].y, lut[fm].x, sel);
        }
    };
    auto decode8_y = [&](const uint32_t (*Y0)[4], const uint32_t (*Y1)[4], int fm, i32x8& A8) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        A8[k] = (int)__builtin_amdgcn_perm(lut8[fm], lut8[fm], Y0[fm][k]);
        A8[4 + k] = (int)__builtin_amdgcn_perm(lut8[fm], lut8[fm], Y1[fm][k]);
      }
    };
    auto read_b = [&](int st, int j, u32x4* bh, u32x4* bl) {
      const char* tile = smem + st * STAGE_BYTES;
#pragma unroll
      for (int fn = 0; fn < WN; ++fn) {
        bh[fn] = *(const u32x4*)(tile + fn * BB + (j * 512 + lane * 8) * 2);
        if constexpr (!F8) bl[fn] = *(const u32x4*)(tile + fn * BB + (2048 + j * 512 + lane * 8) * 2);
      }
    };
    auto read_b8_one = [&](int st, int fn, i32x8& B8f) {
      const char* tile = smem + st * STAGE_BYTES;
      const u32x4 p0 = *(const u32x4*)(tile + fn * BB + 4096 + lane * 16);
      const u32x4 p1 = *(const u32x4*)(tile + fn * BB + 4096 + 1024 + lane * 16);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        B8f[t] = (int)p0[t];
        B8f[4 + t] = (int)p1[t];
      }
    };
    auto read_b8 = [&](int st, i32x8* B8) {
#pragma unroll
      for (int fn = 0; fn < WN; ++fn) read_b8_one(st, fn, B8[fn]);
    };
    // 8-bit dosages, FP16 + FP8 form: the FP16 values of K16 step s (as
    // decode_g8 leaves them, dword d holds samples 16 (s >> 1) + 4 (s & 1) + d
    // and that + 8 of this lane half) converted to e4m3 in the lo operand's
    // layout, where dword 4 p + t holds sample 16 p + 4 k + t in byte k.  Step
    // 2p writes bytes 0 and 1 of dword 4p + d (k = 0 and 2), step 2p + 1 bytes
    // 2 and 3 (k = 1 and 3); one byte permutation then puts k in byte k.
    auto cvt8 = [&](const u32x4* Av, int s, i32x8* A8v) {
      const int p = s >> 1;
#pragma unroll
      for (int fm = 0; fm < WMF; ++fm)
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          uint32_t w = (uint32_t)A8v[fm][4 * p + d];
          if (s & 1) {
            w = cvt_pk_e4m3_hi(w, Av[fm][d]);
            w = __builtin_amdgcn_perm(w, w, 0x03010200u);
          } else {
            w = cvt_pk_e4m3_lo(w, Av[fm][d]);
          }
          A8v[fm][4 * p + d] = (int)w;
        }
    };

    if constexpr (SEG) {
      ch_lo = seg * a.seg_len;
      nch = ch_lo + a.seg_len < a.n_chunks ? a.seg_len : a.n_chunks - ch_lo;
    }
    // prologue: chunks 0..NSTAGE-1 requested, chunk 0 awaited
#pragma unroll
    for (int c = 0; c < NSTAGE; ++c) dma(c, c);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    u32x4 bh[2][WN], bl[2][WN], A[2][WMF];
    i32x8 A8[GF ? WMF : 2], B8[WN];
    uint2 acur[WMF], anext[WMF];
    u32x4 araw[WMF];  // FP8 form: the next chunk's code rows, read a step early
    constexpr bool SY = F8 && W2 && !G8;  // shared selectors (spread / decode_y / decode8_y)
    uint32_t Y0[SY ? WMF : 1][4], Y1[SY ? WMF : 1][4];  // selectors of the first / second code dword
    uint2 dg8[WMF];  // 8-bit dosages: the two dwords of the step being decoded
    if constexpr (G8) {
      read_b(0, 0, bh[0], bl[0]);
      read_g8(0, 0, dg8);
      decode_g8(dg8, A[0]);
    } else {
      read_a(0, acur);
      read_b(0, 0, bh[0], bl[0]);
    }
    if constexpr (SY) {
      spread(acur, 0, Y0);
      decode_y(Y0, 0, A[0]);
    } else if constexpr (!G8) {
      decode(acur, 0, A[0]);
    }
    if constexpr (F8 && !W2 && !G8) decode8(acur, 0, A8[0]);
    if constexpr (GF) {
#pragma unroll
      for (int fm = 0; fm < WMF; ++fm)
#pragma unroll
        for (int i = 0; i < 8; ++i) A8[fm][i] = 0;
      cvt8(A[0], 0, A8);
    }

    // the prologue's reads are complete before the loop; saying so keeps
    // the compiler from waiting for all LDS reads at the loop head
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0), vmcnt and expcnt unconstrained

    int st = 0;  // stage of chunk ch
    for (int ch = 0; ch < nch; ++ch) {
      const int st1 = st + 1 < NSTAGE ? st + 1 : 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int cs = j & 1, ns = cs ^ 1;
        if constexpr (F8 && !W2 && !G8) {
          if (j == 0) read_b8(st, B8);  // this chunk's lo fragments, used by all four steps
        }
        if constexpr (GF) {
          if (j == 3) {
            // the chunk's FP8 lo term, every fragment against every column
            // block (its e4m3 operand was completed at step 2), before the
            // barrier after which the stage is refilled
#pragma unroll
            for (int fn = 0; fn < WN; ++fn) {
              i32x8 b8;
              read_b8_one(st, fn, b8);
#pragma unroll
              for (int fm = 0; fm < WMF; ++fm)
                acc[fm][fn] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(A8[fm], b8, acc[fm][fn], 0, 0, 0, 127,
                                                                              0, bscale[fn]);
            }
          }
        }
        if constexpr (F8 && W2 && !G8) {
#pragma unroll
          for (int q = 0; q < FNS; ++q) read_b8_one(st, j * FNS + q, B8[j * FNS + q]);  // used by this step
          if (j == 0) {
            spread(acur, 1, Y1);
#pragma unroll
            for (int fm = 0; fm < WMF; ++fm) decode8_y(Y0, Y1, fm, A8[fm]);  // both fragments, whole chunk
          }
        }
        if (F8 && !G8 && j == 2) {
          // the next chunk's codes are this wave's own copies: they need
          // only its own copy of chunk ch+1 to have landed, not the barrier
          __builtin_amdgcn_s_waitcnt(waitcnt_vm_only((NSTAGE - 2) * CHUNK_OPS));
          read_a_raw(st1, araw);  // this lane's halves are picked at step 3
        }
        if (j < 3) {
          read_b(st, j + 1, bh[ns], bl[ns]);
          if constexpr (G8) {
            read_g8(st, j + 1, dg8);
            decode_g8(dg8, A[ns]);
            if constexpr (GF) cvt8(A[ns], j + 1, A8);
          } else if constexpr (SY) {
            decode_y(j + 1 < 2 ? Y0 : Y1, j + 1, A[ns]);
          } else {
            decode(acur, j + 1, A[ns]);
          }
        } else {
          // own copies of chunk ch+1 done (the NSTAGE-2 later chunks may
          // still be in flight) and own LDS reads of this chunk done; then
          // every wave's (a plain s_barrier: a workgroup fence here would
          // wait for every copy in flight)
          __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0((NSTAGE - 2) * CHUNK_OPS));
          if constexpr (!F8 && !G8) read_a(st1, anext);  // this wave's own copies: no barrier needed
          if constexpr (F8 && !G8) pick_a(araw, anext);
          asm volatile("s_barrier" ::: "memory");
          // LDS reads before the copies: a read issued after a
          // direct-to-LDS load is held until that load completes
          read_b(st1, 0, bh[ns], bl[ns]);
          if constexpr (G8) read_g8(st1, 0, dg8);  // own copies of chunk ch + 1 have landed
          if constexpr (!F8 || G8) dma(ch + NSTAGE, st);  // the 2-bit FP8 form copies beside its lo MFMAs
          if constexpr (G8) {
            decode_g8(dg8, A[ns]);
          } else if constexpr (SY) {
            spread(anext, 0, Y0);
            decode_y(Y0, 0, A[ns]);
          } else {
            decode(anext, 0, A[ns]);
          }
        }
#pragma unroll
        for (int fn = 0; fn < WN; ++fn)
#pragma unroll
          for (int fm = 0; fm < WMF; ++fm) acc[fm][fn] = mfma16<PREC>(A[cs][fm], bh[cs][fn], acc[fm][fn]);
        if constexpr (!F8) {
#pragma unroll
          for (int fn = 0; fn < WN; ++fn)
#pragma unroll
            for (int fm = 0; fm < WMF; ++fm) acc[fm][fn] = mfma16<PREC>(A[cs][fm], bl[cs][fn], acc[fm][fn]);
        }
        // issue order: copies and LDS reads early, each behind one
        // matrix-core instruction, then the decode, a few VALU ops per MFMA
        if (GF) {
          // 8-bit dosages, FP16 + FP8: no group hints
        } else if (F8 && W2) {  // WMF x WN FP16 MFMA; WN hi + 2 FNS lo fragment reads (+ code rows at step 2)
          constexpr int NDS = W2 ? WN + 2 * FNS : 0;
#pragma unroll
          for (int q = 0; q < NDS; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // DS read
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
            __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);  // VALU
          }
#pragma unroll
          for (int q = 0; q < HI_MFMA - NDS; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
            __builtin_amdgcn_sched_group_barrier(0x002, 12, 0);  // VALU
          }
        } else if (j == 3 && F8) {
#pragma unroll
          for (int q = 0; q < DS_STEP; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // DS read
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
            __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);  // VALU
          }
#pragma unroll
          for (int q = 0; q < HI_MFMA - DS_STEP; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
            __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);  // VALU
          }
        } else if (j == 3) {
#pragma unroll
          for (int q = 0; q < DS_STEP + WMF; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // DS read
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
          }
#pragma unroll
          for (int q = 0; q < CHUNK_OPS; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);  // VMEM (direct-to-LDS)
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
            __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);  // VALU
          }
#pragma unroll
          for (int q = 0; q < HI_MFMA - CHUNK_OPS - DS_STEP - WMF; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
            __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);  // VALU
          }
        } else {
          if (F8 && j == 0) {  // plus the chunk's lo fragment reads
#pragma unroll
            for (int q = 0; q < 3 * WN; ++q) {
              __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // DS read
              __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
              __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);  // VALU
            }
#pragma unroll
            for (int q = 0; q < HI_MFMA - 3 * WN; ++q) {
              __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
              __builtin_amdgcn_sched_group_barrier(0x002, 12, 0);  // VALU
            }
          } else {
            constexpr int VPD = F8 ? 3 : 0, VREST = F8 ? 5 : 3;
#pragma unroll
            for (int q = 0; q < DS_STEP; ++q) {
              __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // DS read
              __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
              if (VPD) __builtin_amdgcn_sched_group_barrier(0x002, VPD, 0);  // VALU
            }
#pragma unroll
            for (int q = 0; q < HI_MFMA - DS_STEP; ++q) {
              __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
              __builtin_amdgcn_sched_group_barrier(0x002, VREST, 0);  // VALU
            }
          }
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (GF) {
          if (j == 3) cvt8(A[ns], 0, A8);  // the next chunk's first step (after the lo MFMAs that read A8)
        }
        if constexpr (F8 && W2 && !G8) {
          // FP8 lo term of column blocks j FNS .. (j + 1) FNS - 1, both fragments, whole chunk
          if (j == 3) dma(ch + NSTAGE, st);  // the stage of chunk ch is free since the barrier
#pragma unroll
          for (int q = 0; q < FNS; ++q) {
            const int fn = j * FNS + q;
#pragma unroll
            for (int fm = 0; fm < WMF; ++fm)
              acc[fm][fn] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(A8[fm], B8[fn], acc[fm][fn], 0, 0, 0,
                                                                            127, 0, bscale[fn]);
          }
          if (j == 3) {
#pragma unroll
            for (int q = 0; q < WMF * FNS; ++q) {
              __builtin_amdgcn_sched_group_barrier(0x010, (CHUNK_OPS + WMF * FNS - 1) / (WMF * FNS), 0);  // VMEM
              __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                       // MFMA
              __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);                                       // VALU
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (F8 && !W2 && !G8) {
          // FP8 lo term of fragment fm = j over the whole chunk, after the
          // step's FP16 work (its operands were read at step 0); the decode
          // of the next fragment's e4m3 values rides along
          if (j < 3) {
            decode8(acur, j + 1, A8[ns]);
          } else {
            dma(ch + NSTAGE, st);  // the stage of chunk ch is free since the barrier
            decode8(anext, 0, A8[ns]);
          }
#pragma unroll
          for (int fn = 0; fn < WN; ++fn)
            acc[j][fn] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(A8[cs], B8[fn], acc[j][fn], 0, 0, 0, 127,
                                                                         0, bscale[fn]);
          if (j == 3) {
#pragma unroll
            for (int q = 0; q < WN; ++q) {
              __builtin_amdgcn_sched_group_barrier(0x010, CHUNK_OPS / WN, 0);  // VMEM (direct-to-LDS)
              __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);               // MFMA
              __builtin_amdgcn_sched_group_barrier(0x002, 12, 0);              // VALU
            }
          } else {
#pragma unroll
            for (int q = 0; q < WN; ++q) {
              __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
              __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);  // VALU
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int fm = 0; fm < WMF; ++fm) acur[fm] = anext[fm];
      st = st1;
      // the next chunk's first fragments landed long ago; saying so here
      // keeps the compiler from waiting for all LDS reads at the loop head
      __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0), vmcnt and expcnt unconstrained
    }
    __builtin_amdgcn_s_waitcnt(0);  // surplus copies have landed
    __syncthreads();                // all waves are done with the stages
    if constexpr (SEG) {
      // the sums so far, 16 bytes per lane and access, in this workgroup's part.
      // Every segment but the last ends here, so the accumulators don't live
      // on (kept over the segments they spill: 7.3 against 5.8 ms, 16,384
      // markers x 2,048 phenotypes, N = 70,001)
      char* ws = (char*)a.part + (int64_t)blockIdx.x * kSegTileBytes + tid * 16;
      const bool last = seg + 1 == a.n_segs;
      if (seg > 0) {
#pragma unroll
        for (int f = 0; f < WMF * WN; ++f) {
          // a few fragments' loads in flight at a time, as registers allow
          if (f % (NW == 4 ? 4 : 2) == 0) asm volatile("" : "+v"(ws)::"memory");
          f32x16& v = acc[f / WN][f % WN];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const u32x4 e = gload<u32x4>(ws + (f * 4 + i) * NT * 16);
#pragma unroll
            for (int t = 0; t < 4; ++t) v[4 * i + t] = __uint_as_float(e[t]) + v[4 * i + t];
          }
        }
      }
      if (!last) {
#pragma unroll
        for (int f = 0; f < WMF * WN; ++f) {
          asm volatile("" : "+v"(ws)::"memory");
          const f32x16& v = acc[f / WN][f % WN];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            u32x4 e;
#pragma unroll
            for (int t = 0; t < 4; ++t) e[t] = __float_as_uint(v[4 * i + t]);
            gstore(ws + (f * 4 + i) * NT * 16, e);
          }
        }
        __builtin_amdgcn_s_waitcnt(0);  // the next segment's waits count its copies alone
        ++seg;
        continue;
      }
      seg = 0;
    }
    w += nslots;

    if constexpr (MODE == kRaw) {
#pragma unroll
      for (int fn = 0; fn < WN; ++fn) {
        const int cb = ctile * WN + fn;
        if (cb >= a.n_cblocks) continue;
        const ColBlock blk = a.cblocks[cb];
        if (r32 >= blk.ncol) continue;
#pragma unroll
        for (int fm = 0; fm < WMF; ++fm)
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int64_t mr = rowbase + fm * 32 + 8 * (i >> 2) + 4 * h + (i & 3);
            if (mr < a.nm) gstore(a.raw_out + mr * a.raw_ld + blk.col0 + r32, acc[fm][fn][i]);
          }
      }
    } else {
      // this lane's column values of each block, read ahead of the stores
      float cinv[WN], csp[WN];
#pragma unroll
      for (int fn = 0; fn < WN; ++fn) {
        const int cb = ctile * WN + fn;
        const ColBlock blk = a.cblocks[cb < a.n_cblocks ? cb : ctile * WN];
        const PanelDev& pdb = a.panels[blk.panel];
        const bool colok = cb < a.n_cblocks && r32 < blk.ncol;
        cinv[fn] = colok ? gload<float>(pdb.invny + blk.col0 + r32) : 0.f;
        csp[fn] = colok ? gload<float>(pdb.scale + blk.col0 + r32) * a.gunit : 0.f;
      }
      // the wave's rows' 1/||g_res|| for panel j, one or two rows per lane
      float2* ihl = (float2*)(smem + LDS_BYTES) + __builtin_amdgcn_readfirstlane(wave) * (WMF * 32);
      auto load_rows = [&](int j) {
#pragma unroll
        for (int k = 0; k < WMF / 2; ++k) {
          int64_t mr = rowbase + 64 * k + lane;
          mr = mr < a.nm ? mr : a.nm - 1;
          ihl[64 * k + lane] = gload<float2>(a.invh + mr * a.n_panels + j);
        }
      };
      // panel j's table into LDS (all threads; the caller brackets it with barriers)
      auto load_table = [&](int j) {
        tab4* tl = (tab4*)(smem + LDS_BYTES + IH_BYTES);
        const tab4* tg = (const tab4*)a.panels[j].table;
        for (int k = tid; k < kTabIntervals; k += NT) tl[k] = gload<tab4>(tg + k);
      };
      int ih_panel = a.cblocks[ctile * WN].panel;
      load_rows(ih_panel);
      if constexpr (LT) {
        if (ih_panel != tab_panel) {  // the last tile's epilogue ended at the barrier below
          load_table(ih_panel);
          tab_panel = ih_panel;
          __syncthreads();
        }
      }
      // projection correction (see gemm_kernel)
#pragma unroll
      for (int fn = 0; fn < WN; ++fn) {
        const int cb = ctile * WN + fn;
        const ColBlock blk = a.cblocks[cb < a.n_cblocks ? cb : ctile * WN];
        const float* cwp = a.panels[blk.panel].cw + (int64_t)(blk.col0 + r32) * kSlots + 8 * h;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          const float4 c0 = gload<float4>(cwp + 16 * ks);
          const float4 c1 = gload<float4>(cwp + 16 * ks + 4);
          u32x4 bo;
          bo[0] = pack_bf16x2(c0.x, c0.y);
          bo[1] = pack_bf16x2(c0.z, c0.w);
          bo[2] = pack_bf16x2(c1.x, c1.y);
          bo[3] = pack_bf16x2(c1.z, c1.w);
          const bf16x8 B = __builtin_bit_cast(bf16x8, bo);
#pragma unroll
          for (int fm = 0; fm < WMF; ++fm) {
            int64_t mr = rowbase + fm * 32 + r32;
            mr = mr < a.nm ? mr : a.nm - 1;
            const float* wp = a.wws + (mr * a.n_panels + blk.panel) * kSlots + 16 * ks + 8 * h;
            const float4 w0 = gload<float4>(wp);
            const float4 w1 = gload<float4>(wp + 4);
            u32x4 ao;
            ao[0] = pack_bf16x2(w0.x, w0.y);
            ao[1] = pack_bf16x2(w0.z, w0.w);
            ao[2] = pack_bf16x2(w1.x, w1.y);
            ao[3] = pack_bf16x2(w1.z, w1.w);
            acc[fm][fn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ao), B,
                                                                  acc[fm][fn], 0, 0, 0);
          }
        }
      }
      // SB column blocks are staged at once (as many as the stages hold), so
      // that their accumulators are dead before the row loops run
      constexpr int SB = LDS_BYTES / (NW * WMF * 32 * 32 * 4) < WN ? LDS_BYTES / (NW * WMF * 32 * 32 * 4) : WN;
      static_assert(SB >= 1 && WN % SB == 0, "staged column blocks");
      const int wv = __builtin_amdgcn_readfirstlane(wave);  // uniform: LDS bases in scalar registers
      float* stage = (float*)smem + wv * (SB * WMF * 32 * 32);
#pragma unroll
      for (int f0 = 0; f0 < WN; f0 += SB) {
        if (ctile * WN + f0 >= a.n_cblocks) break;
#pragma unroll
        for (int s = 0; s < SB; ++s)
#pragma unroll
          for (int fm = 0; fm < WMF; ++fm)
#pragma unroll
            for (int i = 0; i < 16; ++i)
              stage[(s * WMF * 32 + fm * 32 + 8 * (i >> 2) + 4 * h + (i & 3)) * 32 + r32] = acc[fm][f0 + s][i];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int s = 0; s < SB; ++s) {
          const int fn = f0 + s;
          const int cb = ctile * WN + fn;
          if (cb >= a.n_cblocks) break;
          const ColBlock blk = a.cblocks[cb];
          if (blk.panel != ih_panel) {  // a column tile across a panel boundary
            ih_panel = blk.panel;
            load_rows(ih_panel);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
          }
          if constexpr (LT) {
            if (blk.panel != tab_panel) {
              __syncthreads();
              load_table(blk.panel);
              tab_panel = blk.panel;
              __syncthreads();
            }
          }
          const float* sb = stage + s * (WMF * 32 * 32);
          const LdsRows ihr = (LdsRows)ihl;
          if constexpr (LT)
            finish_block<WMF>(sb, a, blk, rowbase, h, r32, (LdsTable)(smem + LDS_BYTES + IH_BYTES), ihr, cinv[fn],
                              csp[fn]);
          else
            finish_block<WMF>(sb, a, blk, rowbase, h, r32, (const tab4*)a.panels[blk.panel].table, ihr, cinv[fn],
                              csp[fn]);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
    }
    __syncthreads();  // the next tile's prologue overwrites the staging area
  }
}

// ---------------------------------------------------------------------------
// tile shapes and launchers
// ---------------------------------------------------------------------------
// {waves, 32-row fragments per wave, 32-column blocks per tile}
static const TileShape kShapes[] = {
    {4, 4, 4},  // 0: 512 x 128, wide, one wave per SIMD (split forms)
    {8, 2, 4},  // 1: 512 x 128, wide, two waves per SIMD (split forms)
    {8, 2, 4},  // 2: 512 x 128
    {4, 2, 4},  // 3: 256 x 128
    {8, 1, 4},  // 4: 256 x 128, 8 waves
    {8, 2, 2},  // 5: 512 x 64
    {4, 2, 8},  // 6: 256 x 256, wide, one wave per SIMD (FP8 lo form; others run shape 0)
};
constexpr int kNumShapes = sizeof(kShapes) / sizeof(kShapes[0]);

int n_tile_shapes() { return kNumShapes; }
TileShape tile_shape(int idx) { return kShapes[idx]; }

template <int PREC, int MODE>
static const void* gemm_fn_g8(int idx) {  // 8-bit dosages: wide tiles 0 and 1 for the FP16 splits
  if constexpr (PREC == kSplit16 || PREC == kSplit8) {
    if (idx == 1) return (const void*)gemm_wide_kernel<PREC, MODE, 8, 2, 4, true>;
    if (idx == 0 || PREC == kSplit8) return (const void*)gemm_wide_kernel<PREC, MODE, 4, 4, 4, true>;
  }
  if constexpr (PREC == kFP32 || PREC == kSplit16) {  // the register-staged shapes
    switch (idx) {
      case 3: return (const void*)gemm_kernel<PREC, 4, 2, 4, MODE, true>;
      case 4: return (const void*)gemm_kernel<PREC, 8, 1, 4, MODE, true>;
      case 5: return (const void*)gemm_kernel<PREC, 8, 2, 2, MODE, true>;
      default: return (const void*)gemm_kernel<PREC, 8, 2, 4, MODE, true>;
    }
  }
  return nullptr;
}

template <int PREC, int MODE>
static const void* gemm_fn(int idx) {
  if constexpr (PREC == kSplit8) {  // the FP8 lo form exists only as the wide kernel
    if (idx == 1) return (const void*)gemm_wide_kernel<PREC, MODE, 8, 2>;
    if (idx == 6) return (const void*)gemm_wide_kernel<PREC, MODE, 4, 2, 8>;
    return (const void*)gemm_wide_kernel<PREC, MODE, 4, 4>;
  } else {
    switch (idx) {
      case 0:  // the wide kernels exist for the split forms; FP32 uses shape 2
        if constexpr (PREC != kFP32) return (const void*)gemm_wide_kernel<PREC, MODE, 4, 4>;
        return (const void*)gemm_kernel<PREC, 8, 2, 4, MODE>;
      case 1:
        if constexpr (PREC != kFP32) return (const void*)gemm_wide_kernel<PREC, MODE, 8, 2>;
        return (const void*)gemm_kernel<PREC, 8, 2, 4, MODE>;
      case 2: return (const void*)gemm_kernel<PREC, 8, 2, 4, MODE>;
      case 3: return (const void*)gemm_kernel<PREC, 4, 2, 4, MODE>;
      case 4: return (const void*)gemm_kernel<PREC, 8, 1, 4, MODE>;
      case 5: return (const void*)gemm_kernel<PREC, 8, 2, 2, MODE>;
      case 6:  // the 256 x 256 wide shape exists for the FP8 lo form only
        if constexpr (PREC != kFP32) return (const void*)gemm_wide_kernel<PREC, MODE, 4, 4>;
        return (const void*)gemm_kernel<PREC, 8, 2, 4, MODE>;
    }
    return nullptr;
  }
}

// FP32 on the small tiles (every accumulator's order of summation is the same in all shapes)
template <bool G8>
static const void* fp32_small_fn(int idx, int mode) {
  if (mode == kRaw) return idx == 0 ? (const void*)gemm_kernel<kFP32, 4, 1, 1, kRaw, G8> : nullptr;
  switch (idx) {
    case 0: return (const void*)gemm_kernel<kFP32, 4, 1, 1, kTest, G8>;
    case 1: return (const void*)gemm_kernel<kFP32, 4, 2, 1, kTest, G8>;
    case 2: return (const void*)gemm_kernel<kFP32, 4, 1, 2, kTest, G8>;
    case 3: return (const void*)gemm_kernel<kFP32, 4, 2, 2, kTest, G8>;
    case 4: return (const void*)gemm_kernel<kFP32, 4, 1, 4, kTest, G8>;
  }
  return nullptr;
}
const void* gemm_small_fp32_fn(int idx, int mode, bool g8) {
  return g8 ? fp32_small_fn<true>(idx, mode) : fp32_small_fn<false>(idx, mode);
}

static TileShape effective_shape(int idx, int prec, bool g8 = false) {
  const bool wide = idx <= 1 || idx == 6;
  if (g8 && prec == kSplit8) return kShapes[idx == 1 ? 1 : 0];
  if (g8 && prec == kSplit16 && idx <= 1) return kShapes[idx];
  if (g8) return kShapes[wide ? 2 : idx];
  if (prec == kSplit8) return kShapes[(idx == 1 || idx == 6) ? idx : 0];
  if (wide && prec == kFP32) return kShapes[2];
  if (idx == 6) return kShapes[0];
  return kShapes[idx];
}
TileShape tile_shape_for(int idx, int prec, bool g8) { return effective_shape(idx, prec, g8); }

static const void* gemm_fn_any(int idx, int prec, int mode, bool g8 = false) {
  if (g8) {
    if (prec == kSplit16) return mode == kRaw ? gemm_fn_g8<kSplit16, kRaw>(idx) : gemm_fn_g8<kSplit16, kTest>(idx);
    if (prec == kFP32) return mode == kRaw ? gemm_fn_g8<kFP32, kRaw>(idx) : gemm_fn_g8<kFP32, kTest>(idx);
    if (prec == kSplit8) return mode == kRaw ? gemm_fn_g8<kSplit8, kRaw>(idx) : gemm_fn_g8<kSplit8, kTest>(idx);
    return nullptr;
  }
  if (prec == kSplit) return mode == kRaw ? gemm_fn<kSplit, kRaw>(idx) : gemm_fn<kSplit, kTest>(idx);
  if (prec == kSplit16) return mode == kRaw ? gemm_fn<kSplit16, kRaw>(idx) : gemm_fn<kSplit16, kTest>(idx);
  if (prec == kSplit8) return mode == kRaw ? gemm_fn<kSplit8, kRaw>(idx) : gemm_fn<kSplit8, kTest>(idx);
  return mode == kRaw ? gemm_fn<kFP32, kRaw>(idx) : gemm_fn<kFP32, kTest>(idx);
}

int tile_alias(int idx, int prec, bool g8) {
  const void* fn = gemm_fn_any(idx, prec, kTest, g8);
  for (int i = 0; i < idx; ++i)
    if (gemm_fn_any(i, prec, kTest, g8) == fn) return i;
  return idx;
}

int gemm_grid(int idx, int prec, int mode, int n_cu, bool g8) {
  const void* fn = gemm_fn_any(idx, prec, mode, g8);
  if (!fn) return 8;
  int occ = 0;
  const int threads = effective_shape(idx, prec, g8).waves * 64;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, fn, threads, 0) != hipSuccess || occ < 1) occ = 1;
  int g = occ * n_cu;
  g = (g / 8) * 8;
  return g < 8 ? 8 : g;
}

// the wide tiles over segments: tiles 1 and (FP16 + FP8, 2-bit codes) 6, else
// tile 0.  The register-staged shapes have no segments: with 8-bit dosages,
// 8,192 markers x 1,024 phenotypes, N = 131,072, they take 9.7 (FP16 + FP8) and
// 10.6 ms (FP16 split) where segments on small and wide tiles take 4.5 and 5.8
static int seg_tile(int idx, int prec, bool g8) { return idx == 1 || (idx == 6 && prec == kSplit8 && !g8) ? idx : 0; }
TileShape seg_tile_shape(int idx, int prec, bool g8) { return kShapes[seg_tile(idx, prec, g8)]; }
template <int PREC, bool G8>
static const void* seg_fn(int tile) {
  if constexpr (PREC == kSplit8 && !G8)
    if (tile == 6) return (const void*)gemm_wide_kernel<PREC, kTest, 4, 2, 8, G8, true>;
  return tile == 1 ? (const void*)gemm_wide_kernel<PREC, kTest, 8, 2, 4, G8, true>
                   : (const void*)gemm_wide_kernel<PREC, kTest, 4, 4, 4, G8, true>;
}
int64_t seg_part_bytes(int n_segs, int n_cu) {
  return n_segs <= 1 ? 0 : std::max<int64_t>(n_cu * kSegTileBytes, kSegPartLeast);
}
hipError_t launch_gemm_seg(int idx, int prec, const GemmArgs& a, int n_cu, hipStream_t s, bool g8) {
  const int tile = seg_tile(idx, prec, g8);
  const void* fn = nullptr;
  if (prec == kSplit8) fn = g8 ? seg_fn<kSplit8, true>(tile) : seg_fn<kSplit8, false>(tile);
  if (prec == kSplit16) fn = g8 ? seg_fn<kSplit16, true>(tile) : seg_fn<kSplit16, false>(tile);
  const int64_t grid = std::min<int64_t>(n_cu, a.part_bytes / kSegTileBytes) / 8 * 8;
  if (!fn || grid < 8) return hipErrorInvalidValue;
  GemmArgs arg = a;
  void* params[] = {&arg};
  return hipLaunchKernel(fn, dim3((unsigned)grid), dim3(kShapes[tile].waves * 64), params, 0, s);
}

hipError_t launch_gemm(int idx, int prec, int mode, const GemmArgs& a, int grid, hipStream_t s, bool g8) {
  const void* fn = gemm_fn_any(idx, prec, mode, g8);
  if (!fn) return hipErrorInvalidValue;
  const int threads = effective_shape(idx, prec, g8).waves * 64;
  GemmArgs arg = a;
  void* params[] = {&arg};
  return hipLaunchKernel(fn, dim3(grid), dim3(threads), params, 0, s);
}

hipError_t launch_qr(const double* C, int64_t ldc, int64_t n, int64_t n_pad, int q, double* X, double* Q,
                     double* rdiag, double* scratch, int32_t* flags, hipStream_t s) {
  if (q < 1 || q > kSlots) return hipErrorInvalidValue;
  double* part = scratch;
  double* fv = scratch + kQrGrid * kSlots;
  double* vtv = fv + kSlots;
  const dim3 g(kQrGrid), b(kQrThreads);
  hipLaunchKernelGGL(qr_load_kernel, g, b, 0, s, C, ldc, n, n_pad, q, X, flags);
  for (int j = 0; j < q; ++j) {
    const double* xj = X + (int64_t)j * n_pad;
    hipLaunchKernelGGL(qr_dots_kernel, g, b, 0, s, xj, (const double*)X, n, n_pad, q, j, (int64_t)j + 1, part);
    hipLaunchKernelGGL(qr_coef_kernel, dim3(1), b, 0, s, X, n_pad, q, j, 1, (const double*)part, rdiag, fv, vtv);
    if (j + 1 < q) hipLaunchKernelGGL(qr_reflect_kernel, g, b, 0, s, xj, X, n, n_pad, q, j + 1, (int64_t)j, (const double*)fv);
  }
  hipLaunchKernelGGL(qr_qinit_kernel, g, b, 0, s, Q, n_pad, q);
  for (int j = q - 1; j >= 0; --j) {
    const double* xj = X + (int64_t)j * n_pad;
    hipLaunchKernelGGL(qr_dots_kernel, g, b, 0, s, xj, (const double*)Q, n, n_pad, q, j, (int64_t)j, part);
    hipLaunchKernelGGL(qr_coef_kernel, dim3(1), b, 0, s, X, n_pad, q, j, 0, (const double*)part, rdiag, fv, vtv);
    hipLaunchKernelGGL(qr_reflect_kernel, g, b, 0, s, xj, Q, n, n_pad, q, j, (int64_t)j, (const double*)fv);
  }
  hipLaunchKernelGGL(qr_rank_kernel, dim3(1), dim3(64), 0, s, (const double*)rdiag, q, flags);
  return hipGetLastError();
}

static int gram_waves(int64_t n_pad) {  // about four chunks a wave, at most 256 waves
  return (int)std::max<int64_t>(1, std::min<int64_t>(256, n_pad / kChunk / 4));
}

hipError_t launch_gram_qr(const double* C, int64_t ldc, int64_t n, int64_t n_pad, int q, double* Q1, double* Q,
                          double* scratch, int32_t* flags, void* wop_fp32, void* const* wop_hl, hipStream_t s) {
  if (q < 1 || q > kSlots) return hipErrorInvalidValue;
  if (q == 1) {
    hipLaunchKernelGGL(intercept_kernel, dim3((unsigned)std::min<int64_t>(1024, n_pad / kChunk)), dim3(256), 0, s, Q, n,
                       n_pad);
    return launch_cov_operands(Q, n, n_pad, q, wop_fp32, wop_hl, s);
  }
  GramArgs a{};
  a.C = C;
  a.ldc = ldc;
  a.n = n;
  a.n_pad = n_pad;
  a.q = q;
  a.waves = gram_waves(n_pad);
  a.coef = scratch;
  static_assert(2 * kSlots * kSlots + kSlots <= kQrScratch, "the factors fit in the QR's scratch");
  // the waves' tiles (6 KiB for every four chunks, or one wave's) lie in the
  // FP32 operand (8 KiB per chunk), which is written when they have been read
  a.part = (double*)wop_fp32;
  a.Q1 = Q1;
  a.Q = Q;
  a.flags = flags;
  a.wop_fp32 = (float*)wop_fp32;
  a.wop_hl[0] = (char*)wop_hl[kSplit];
  a.wop_hl[1] = (char*)wop_hl[kSplit16];
  const dim3 g(a.waves), b(64), last((unsigned)(n_pad / kChunk));
  if (q <= 16) {
    hipLaunchKernelGGL((gram_kernel<0, 1>), g, b, 0, s, a);
    hipLaunchKernelGGL(gram_factor_kernel<false>, dim3(1), dim3(1024), 0, s, a);
    hipLaunchKernelGGL((gram_kernel<1, 1>), g, b, 0, s, a);
    hipLaunchKernelGGL(gram_factor_kernel<true>, dim3(1), dim3(1024), 0, s, a);
    hipLaunchKernelGGL((gram_kernel<2, 1>), last, b, 0, s, a);
  } else {
    hipLaunchKernelGGL((gram_kernel<0, 2>), g, b, 0, s, a);
    hipLaunchKernelGGL(gram_factor_kernel<false>, dim3(1), dim3(1024), 0, s, a);
    hipLaunchKernelGGL((gram_kernel<1, 2>), g, b, 0, s, a);
    hipLaunchKernelGGL(gram_factor_kernel<true>, dim3(1), dim3(1024), 0, s, a);
    hipLaunchKernelGGL((gram_kernel<2, 2>), last, b, 0, s, a);
  }
  return hipGetLastError();
}

hipError_t launch_cov_operands(const double* Q, int64_t n, int64_t n_pad, int q, void* wop_fp32,
                               void* const* wop_hl, hipStream_t s) {
  if (!wop_fp32 || !wop_hl[kSplit] || !wop_hl[kSplit16]) return hipErrorInvalidValue;
  CovOperandArgs a{Q, n_pad, q, (float*)wop_fp32, {(char*)wop_hl[kSplit], (char*)wop_hl[kSplit16]}};
  hipLaunchKernelGGL(cov_operand_kernel, dim3((unsigned)(n_pad / kChunk)), dim3(256), 0, s, a);
  return hipGetLastError();
}

// segments of the split preparation: about 8,192 waves in all, at least two chunks each
static int prep_segments(int64_t n_pad, int64_t P) {
  const int64_t tiles = (P + 15) / 16;
  return (int)std::max<int64_t>(1, std::min<int64_t>((8192 + tiles - 1) / tiles, n_pad / kChunk / 2));
}
// cohorts from here on take the split preparation: below, its seven short
// launches (nine in the FP16 + FP8 form, about 40 us) cost more than
// prep_kernel's one (38 us at N = 2,000)
constexpr int64_t kPrepSplitMin = 64 * kChunk;

size_t prep_scratch_bytes(int64_t n_pad, int64_t P, int q) {
  if (n_pad < kPrepSplitMin) return 0;
  const int64_t nc = (P + 15) / 16 * 16;
  const int64_t sums = 16 * prep_slot_tiles(q) + kPrepMore;  // per column and segment, and twice per column
  return sizeof(double) * (size_t)(nc * (sums * (prep_segments(n_pad, P) + 2) + 2));
}

template <int PREC, int NT, bool F64>
static void launch_prep_passes(const PrepArgs& a, unsigned grid, hipStream_t s) {
  const dim3 b(256), g(grid);
  const int64_t nc = 16 * (int64_t)a.n_tiles;
  const double* part = a.part;
  hipLaunchKernelGGL((prep_project_kernel<NT, F64>), g, b, 0, s, a);
  hipLaunchKernelGGL(prep_sum_kernel<false>, dim3(a.n_tiles, a.slots + kPrepMore), b, 0, s, part, a.sums, a.segs, nc);
  hipLaunchKernelGGL((prep_residual_kernel<0, kFP32, NT, F64>), g, b, 0, s, a);
  hipLaunchKernelGGL(prep_sum_kernel<false>, dim3(a.n_tiles, 1), b, 0, s, part, a.r2, a.segs, nc);
  if (PREC == kSplit8) {
    hipLaunchKernelGGL((prep_residual_kernel<1, kSplit8, NT, F64>), g, b, 0, s, a);
    hipLaunchKernelGGL(prep_sum_kernel<true>, dim3(a.n_tiles, 1), b, 0, s, part, a.maxlo, a.segs, nc);
  }
  hipLaunchKernelGGL((prep_residual_kernel<2, PREC, NT, F64>), g, b, 0, s, a);
  hipLaunchKernelGGL(prep_sum_kernel<false>, dim3(a.n_tiles, a.slots + kPrepMore), b, 0, s, part,
                     a.sums + (a.slots + kPrepMore) * nc, a.segs, nc);
  hipLaunchKernelGGL(prep_finish_kernel, dim3((unsigned)((a.P + 3) / 4)), b, 0, s, a, PREC);
}

hipError_t launch_prep(const void* Y, int y_fp64, int64_t ldy, int64_t n, int64_t n_pad, int64_t P,
                       const double* Q, int q, int prec, void* yop, float* scale, float* invny, float* cw,
                       uint8_t* lscale, int32_t* flags, void* scratch, hipStream_t s) {
  if (scratch) {
    PrepArgs a{};
    a.Y = Y;
    a.ldy = ldy;
    a.n = n;
    a.n_pad = n_pad;
    a.P = P;
    a.Q = Q;
    a.q = q;
    a.y_fp64 = y_fp64;
    a.n_tiles = (int)((P + 15) / 16);
    a.segs = prep_segments(n_pad, P);
    a.yop = yop;
    const int64_t nc = 16 * (int64_t)a.n_tiles;
    a.sums = (double*)scratch;
    a.slots = 16 * prep_slot_tiles(q);
    a.r2 = a.sums + 2 * (a.slots + kPrepMore) * nc;
    a.maxlo = a.r2 + nc;
    a.part = a.maxlo + nc;
    a.lscale = lscale;
    a.scale = scale;
    a.invny = invny;
    a.cw = cw;
    a.flags = flags;
    const unsigned grid = (unsigned)(((int64_t)a.n_tiles * a.segs + 3) / 4);
    auto go = [&](auto p) {
      constexpr int PREC = decltype(p)::value;
      if (prep_slot_tiles(q) == 1)
        y_fp64 ? launch_prep_passes<PREC, 1, true>(a, grid, s) : launch_prep_passes<PREC, 1, false>(a, grid, s);
      else
        y_fp64 ? launch_prep_passes<PREC, 2, true>(a, grid, s) : launch_prep_passes<PREC, 2, false>(a, grid, s);
    };
    if (prec == kSplit8)
      go(std::integral_constant<int, kSplit8>{});
    else if (prec == kSplit16)
      go(std::integral_constant<int, kSplit16>{});
    else if (prec == kSplit)
      go(std::integral_constant<int, kSplit>{});
    else
      go(std::integral_constant<int, kFP32>{});
    return hipGetLastError();
  }
  // q <= QS slots; two columns per workgroup (at P = 2,048 and q = 11 this
  // beats four, which leaves two waves per SIMD, and one), one for q > 24
  auto go = [&](auto kern, int cpw) {
    hipLaunchKernelGGL(kern, dim3((unsigned)((P + cpw - 1) / cpw)), dim3(kPrepThreads), 0, s, Y, y_fp64, ldy, n,
                       n_pad, P, Q, q, prec, yop, scale, invny, cw, lscale, flags);
  };
  if (q <= 4)
    go(prep_kernel<4, 2>, 2);
  else if (q <= 8)
    go(prep_kernel<8, 2>, 2);
  else if (q <= 12)
    go(prep_kernel<12, 2>, 2);
  else if (q <= 16)
    go(prep_kernel<16, 2>, 2);
  else if (q <= 24)
    go(prep_kernel<24, 2>, 2);
  else
    go(prep_kernel<kSlots, 1>, 1);
  return hipGetLastError();
}

hipError_t launch_set_operand(const float* V, int64_t ldv, int64_t n, int64_t n_pad, int64_t P, int prec,
                              void* yop, uint8_t* lscale, hipStream_t s) {
  if (prec == kSplit8) {
    hipLaunchKernelGGL(set_lscale_kernel, dim3((unsigned)P), dim3(kPrepThreads), 0, s, V, ldv, n, lscale);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(set_operand_kernel, dim3(1024), dim3(256), 0, s, V, ldv, n, n_pad, P, prec, yop,
                     (const uint8_t*)lscale);
  return hipGetLastError();
}

hipError_t launch_table(float4* table, double df, hipStream_t s) {
  hipLaunchKernelGGL(table_kernel, dim3((kTabIntervals + kTabWave - 1) / kTabWave), dim3(64), 0, s, table, df);
  return hipGetLastError();
}

hipError_t launch_stats(const StatsArgs& a, hipStream_t s) {
  const unsigned blocks = (unsigned)((a.nm + 3) / 4);
  hipLaunchKernelGGL(stats_kernel, dim3(blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_finalize(const MarkerStat* ms, float* wws, float2* invh, int64_t nm, int n_panels, float wscale,
                           int lo_slot, RedoDev redo, hipStream_t s) {
  const int64_t total = nm * n_panels;
  hipLaunchKernelGGL(finalize_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, ms, wws, invh, nm,
                     n_panels, wscale, lo_slot, redo);
  return hipGetLastError();
}

__global__ void topk_read_kernel(const unsigned long long* __restrict__ words, int64_t n, double df,
                                 float* __restrict__ nl, int64_t* __restrict__ marker) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const unsigned long long w = words[i];
    if (w == 0ull) {
      if (nl) nl[i] = __builtin_nanf("");
      if (marker) marker[i] = -1;
      continue;
    }
    const double at = (double)__uint_as_float((uint32_t)(w >> 32));
    if (nl) nl[i] = (float)(-ln_p_two_sided(at, df) / M_LN10);
    if (marker) marker[i] = (int64_t)(0xffffffffu - (uint32_t)w);
  }
}

hipError_t launch_topk_read(const unsigned long long* words, int64_t n, int k, double df, float* nl, int64_t* marker,
                            hipStream_t s) {
  (void)k;
  const int64_t blocks = std::min<int64_t>(1024, (n + 255) / 256);
  hipLaunchKernelGGL(topk_read_kernel, dim3((unsigned)std::max<int64_t>(1, blocks)), dim3(256), 0, s, words, n, df, nl,
                     marker);
  return hipGetLastError();
}

template <bool FAR>
static void (*redo_fn(int prec, bool g8))(RedoArgs) {
  if (prec == kSplit8) return g8 ? redo_kernel<kSplit8, true, FAR> : redo_kernel<kSplit8, false, FAR>;
  if (prec == kSplit16) return g8 ? redo_kernel<kSplit16, true, FAR> : redo_kernel<kSplit16, false, FAR>;
  if (prec == kSplit && !g8) return redo_kernel<kSplit, false, FAR>;
  if (prec == kFP32) return g8 ? redo_kernel<kFP32, true, FAR> : redo_kernel<kFP32, false, FAR>;
  return nullptr;
}

hipError_t launch_redo(const RedoArgs& a, int grid, hipStream_t s) {
  // 32-bit offsets reach the last of kSlots columns below 16.7 million samples
  const bool far = (a.n_pad * kSlots) * 8 > (int64_t)UINT32_MAX;
  void (*fn)(RedoArgs) = far ? redo_fn<true>(a.prec, a.code == 2) : redo_fn<false>(a.prec, a.code == 2);
  if (!fn) return hipErrorInvalidValue;
  hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(kRedoThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_bind(const BindArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(bind_kernel, dim3(1), dim3(kMaxPanelsPerBind), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_tail_reset(TailDev t, hipStream_t s) {
  hipLaunchKernelGGL(tail_reset_kernel, dim3(1), dim3(64), 0, s, t);
  return hipGetLastError();
}

hipError_t launch_tail(TailDev t, const PanelDev* panels, const OutDev* outs, HitDev hits, int64_t m_begin,
                       hipStream_t s) {
  hipLaunchKernelGGL(tail_kernel, dim3(64), dim3(64), 0, s, t, panels, outs, hits, m_begin);
  return hipGetLastError();
}

hipError_t launch_debug_stats(const MarkerStat* ms, int64_t nm, double* shift, double* mean, double* scale,
                              hipStream_t s) {
  hipLaunchKernelGGL(debug_stats_kernel, dim3((unsigned)((nm + 255) / 256)), dim3(256), 0, s, ms, nm, shift, mean,
                     scale);
  return hipGetLastError();
}

}  // namespace tgw
