// Bayesian factorisation (BPTF, Sec. 2.2, which pairs the least-squares update with draws
// of the factor priors' parameters), in the form of the published BPMF / BPTF Gibbs sampler.
// Ratings are Gaussian with precision alpha around u . v; each row of a side has the
// prior N(mu, Lambda^{-1}); (mu, Lambda) has a Normal-Wishart hyperprior. The row draws
// reuse the half-sweep kernels (their BAYES variants): this file holds the rest.
//
//   k_prior_prepare   one workgroup, fp64: the prior image the row kernels start from
//                     (Lambda / alpha with the identity on the padding, and
//                     Lambda mu / alpha), laid out as a workspace slot (D > 20) or a
//                     packed record (D <= 20); and, when the side has rows without
//                     ratings, the Cholesky factor L of Lambda for them.
//   k_prior_rows      one lane per row without ratings: x = mu + L^{-T} z.
//   k_hyper_moments   per-block fp64 sums of x and of the upper triangle of x x^T over
//                     the side's rows (fp64 MFMA); products of two fp32
//                     values are exact in fp64, so only the summation order rounds.
//   k_hyper_reduce    the per-block partials summed in 16 fixed segments, in order.
//   k_hyper_sample    one workgroup, fp64: adds the segments in order, forms the
//                     Normal-Wishart posterior (beta* = beta0 + n, nu* = nu0 + n,
//                     mu0* = (beta0 mu0 + n xbar) / beta*, W*^{-1} = W0^{-1} + S +
//                     beta0 n / beta* (mu0 - xbar)(mu0 - xbar)^T with S the scatter
//                     about the mean), then Bartlett's draw: W* = F F^T, B lower
//                     triangular with B_ii = sqrt(chi2_i) and normal B_ij, Lambda =
//                     (F B)(F B)^T, and mu = mu0* + R^{-T} zmu with beta* Lambda = R R^T
//                     (without forming W*, F or R: see the kernel).
// The time chain of BPTF (T_0 ~ N(mu_T, Lambda_T^{-1}), T_k ~ N(T_{k-1}, Lambda_T^{-1})):
//   k_time_rhs        a bin's prior right-hand side Lambda_T (m_k + [k < K - 1] T_{k+1}) /
//                     alpha (m_k = mu_T for the first bin, else T_{k-1}) for the bins of
//                     one parity, in fp64; the bins of a parity are drawn together given
//                     the other parity.
//   k_time_moments    the moments of T_0 alone (n = 1), in the segment layout
//                     k_hyper_sample reads;
//   k_time_steps      the chain's step scatter sum_{k>=1} (T_k - T_{k-1})(T_k - T_{k-1})^T
//                     over a slice of the chain per block (the slice's bins staged in
//                     LDS, differences formed in fp64, exact for fp32 inputs), and
//   k_time_steps_sum  the slices added in order; k_hyper_sample adds the result to
//                     W*^{-1}.
// The variates (chi-square, normals) are inputs. Matrices live in fp64 in registers and LDS
// (133 KB at D = 128); the factorisations are right-looking steps with barriers between.
#include "internal.h"

namespace als {

namespace {

constexpr int kBayesBlock = 256;
constexpr int kHyperBlocks = 512;
constexpr int kReduceSegs = 16;      // the moment partials are summed in 16 segments
constexpr int kMaxD = 128;
constexpr int kStepBlocks = 64;          // slices of the time chain's step scatter
constexpr int kStepStageFloats = 15360;  // LDS stage of a slice (60 KB)
constexpr int kPacked = kMaxD * (kMaxD + 1) / 2;
// Index of (i, j), j <= i, in a packed lower triangle.
__device__ __forceinline__ int pl(int i, int j) { return i * (i + 1) / 2 + j; }

// In-place lower Cholesky factor of the packed lower triangle P (in LDS), right-looking:
// per column, the pivot's square root, the column scaled, then the trailing triangle
// updated, with barriers between. *bad is set when a pivot is not positive and finite
// (the step then continues with a unit pivot, so that every value stays defined).
__device__ void lds_cholesky(double *P, int D, int *bad) {
  for (int k = 0; k < D; ++k) {
    __syncthreads();
    const double p = P[pl(k, k)];
    const bool ok = p > 0.0 && isfinite(p);
    const double l = ok ? sqrt(p) : 1.0;
    if (!ok && threadIdx.x == 0) *bad = 1;
    __syncthreads();
    if (threadIdx.x == 0) P[pl(k, k)] = l;
    for (int i = k + 1 + threadIdx.x; i < D; i += blockDim.x) P[pl(i, k)] /= l;
    __syncthreads();
    // trailing triangle k < j <= i < D on a 16 x 16 grid of threads
    for (int i = k + 1 + (int)(threadIdx.x >> 4); i < D; i += 16) {
      const double lik = P[pl(i, k)];
      for (int j = k + 1 + (int)(threadIdx.x & 15); j <= i; j += 16)
        P[pl(i, j)] -= lik * P[pl(j, k)];
    }
  }
  __syncthreads();
}

__global__ __launch_bounds__(kBayesBlock) void k_prior_prepare(
    const double *__restrict__ Lam, const double *__restrict__ mu, int D, int DP, int LD,
    int aug_col, double alpha, int need_factor, float *__restrict__ init,
    float *__restrict__ K, float *__restrict__ mu32, int32_t *__restrict__ ok) {
  __shared__ double P1[kPacked];
  __shared__ double c[kMaxD];  // Lambda mu / alpha
  __shared__ int bad;
  if (threadIdx.x == 0) bad = 0;
  __shared__ double mus[kMaxD];
  for (int d = threadIdx.x; d < D; d += blockDim.x) {
    mus[d] = mu[d];
    mu32[d] = (float)mu[d];
  }
  // the lower triangle of Lambda (symmetric by contract) into LDS
  for (int i = (int)(threadIdx.x >> 4); i < D; i += 16)
    for (int j = (int)(threadIdx.x & 15); j <= i; j += 16) P1[pl(i, j)] = Lam[i * D + j];
  __syncthreads();
  auto lam = [&](int a, int b) -> double { return a >= b ? P1[pl(a, b)] : P1[pl(b, a)]; };
  for (int d = threadIdx.x; d < D; d += blockDim.x) {
    double t = 0.0;
    for (int e = 0; e < D; ++e) t += lam(d, e) * mus[e];
    c[d] = t / alpha;
  }
  __syncthreads();
  // entry (r, col) of the scaled prior matrix, the identity on the padding, and with the
  // augmented column (D > 20 only) holding Lambda mu / alpha
  auto entry = [&](int r, int col) -> float {
    if (r < D && col < D) return (float)(lam(r, col) / alpha);
    if (col == aug_col && r < D) return (float)c[r];
    return r == col ? 1.f : 0.f;
  };
  if (LD > 0) {
    const int ntri = LD * (LD + 1) / 2, total = ne_floats(LD);
    for (int q = threadIdx.x; q < total; q += blockDim.x) {
      float v = 0.f;
      if (q < ntri) {
        int a = 0, rem = q;
        while (rem >= LD - a) {
          rem -= LD - a;
          ++a;
        }
        v = entry(a, a + rem);
      } else if (q < ntri + LD) {
        const int d = q - ntri;
        v = d < D ? (float)c[d] : 0.f;
      }
      init[q] = v;
    }
  } else {
    const int T = DP / 16, NT = T * (T + 1) / 2;
    const int total = NT * 256 + DP;
    for (int q = threadIdx.x; q < total; q += blockDim.x) {
      float v = 0.f;
      if (q < NT * 256) {
        int t = q >> 8, I = 0;
        while (t >= T - I) {
          t -= T - I;
          ++I;
        }
        const int J = I + t, lane = (q & 255) >> 2, r = q & 3;
        v = entry(16 * I + 4 * (lane >> 4) + r, 16 * J + (lane & 15));
      } else {
        const int d = q - NT * 256;
        v = (aug_col < 0 && d < D) ? (float)c[d] : 0.f;
      }
      init[q] = v;
    }
  }
  // the Cholesky factor L of Lambda for the rows without ratings, when the side has any
  // (the image is written above, so P1 can be factored in place)
  if (need_factor) {
    lds_cholesky(P1, D, &bad);
    for (int q = threadIdx.x; q < D * D; q += blockDim.x) {
      const int i = q / D, j = q % D;
      K[q] = j <= i ? (float)P1[pl(i, j)] : 0.f;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) *ok = bad ? 0 : 1;
}

__global__ __launch_bounds__(64) void k_prior_rows(const int32_t *__restrict__ rows, int64_t n,
                                                  int D, const float *__restrict__ L,
                                                  const float *__restrict__ mu32,
                                                  const int32_t *__restrict__ ok,
                                                  const float *__restrict__ z,
                                                  float *__restrict__ X,
                                                  int32_t *__restrict__ flag_count) {
  const int64_t i = (int64_t)blockIdx.x * 64 + threadIdx.x;
  if (i >= n) return;
  const int64_t row = rows[i];
  if (*ok == 0) {
    atomicAdd(flag_count, 1);
    return;
  }
  // x = mu + L^{-T} z: back substitution with L^T into the row, then the mean added
  const float *__restrict__ zr = z + row * D;
  float *__restrict__ xr = X + row * D;
  for (int a = D - 1; a >= 0; --a) {
    float t = zr[a];
    for (int e = a + 1; e < D; ++e) t = fmaf(-L[e * D + a], xr[e], t);
    xr[a] = t / L[a * D + a];
  }
  for (int a = 0; a < D; ++a) xr[a] += mu32[a];
}

typedef double doublex4 __attribute__((ext_vector_type(4)));

// Moments: the block's rows pass through LDS as fp64, kMomentRows at a time, and its four
// waves accumulate the 16 x 16 tiles (I, J), I <= J, of x x^T on fp64 MFMA (wave w takes
// tiles w, w + 4, ...): lane (kq, c) supplies features 16 I + c and 16 J + c of row 4 s + kq
// and receives rows 4 r + kq, column c. The feature sums go two threads to a feature. Bound
// by the fp64 matrix rate and the partials' write: 39 us for 50 000 rows and 60 for 100 000 at
// D = 100. 4 x 4 tiles per thread on VALU, with one thread walking each feature's sum, took 61
// and 89 us.
// Entries are written in the packed order: the D sums of x_a, then the upper triangle of
// x x^T row by row.
constexpr int kMomentRows = 32;
constexpr int kMomentStride = kMaxD + 2;

__global__ __launch_bounds__(kBayesBlock) void k_hyper_moments(const float *__restrict__ X,
                                                               int64_t n, int D,
                                                               double *__restrict__ partials) {
  constexpr int kTiles = (kMaxD / 16) * (kMaxD / 16 + 1) / 2 / (kBayesBlock / 64);  // per wave
  __shared__ double xs[kMomentRows * kMomentStride];
  const int T = (D + 15) / 16, NT = T * (T + 1) / 2, ne = D + D * (D + 1) / 2;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, kq = lane >> 4, c = lane & 15;
  int oa[kTiles], ob[kTiles];  // first features of the wave's tiles
  doublex4 acc[kTiles];
#pragma unroll
  for (int k = 0; k < kTiles; ++k) {
    int t = w + 4 * k, I = 0;
    if (t >= NT) t = 0;
    while (t >= T - I) {
      t -= T - I;
      ++I;
    }
    oa[k] = 16 * I;
    ob[k] = 16 * (I + t);
    acc[k] = doublex4{0.0, 0.0, 0.0, 0.0};
  }
  const int feature = tid & (kMaxD - 1), half = tid / kMaxD;  // of the feature sums
  double sx = 0.0;
  const int64_t per = (n + gridDim.x - 1) / gridDim.x;
  const int64_t r0 = (int64_t)blockIdx.x * per, r1 = min(n, r0 + per);
  for (int64_t base = r0; base < r1; base += kMomentRows) {
    __syncthreads();
    // row tid / 8 of the stage, features tid % 8, + 8, ...; rows past the end are zero
    const int r = tid >> 3;
    for (int d = tid & 7; d < 16 * T; d += 8)
      xs[r * kMomentStride + d] = base + r < r1 && d < D ? (double)X[(base + r) * D + d] : 0.0;
    __syncthreads();
#pragma unroll
    for (int s = 0; s < kMomentRows / 4; ++s) {
      const double *row = xs + (4 * s + kq) * kMomentStride + c;
#pragma unroll
      for (int k = 0; k < kTiles; ++k)
        if (w + 4 * k < NT)
          acc[k] = __builtin_amdgcn_mfma_f64_16x16x4f64(row[oa[k]], row[ob[k]], acc[k], 0, 0, 0);
    }
    if (feature < D) {
#pragma unroll
      for (int q = 0; q < kMomentRows / 2; ++q)
        sx += xs[(half * (kMomentRows / 2) + q) * kMomentStride + feature];
    }
  }
  double *__restrict__ out = partials + (int64_t)blockIdx.x * ne;
  __syncthreads();
  if (half == 1) xs[feature] = sx;
  __syncthreads();
  if (half == 0 && feature < D) out[feature] = sx + xs[feature];
#pragma unroll
  for (int k = 0; k < kTiles; ++k) {
    if (w + 4 * k >= NT) continue;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int a = oa[k] + 4 * q + kq, e = ob[k] + c;
      if (a <= e && e < D) out[D + a * D - a * (a - 1) / 2 + (e - a)] = acc[k][q];
    }
  }
}

// Segment sums of the moment partials: thread (q, seg) adds entry q of the blocks of
// segment seg in block order (the loads of one thread are independent, so many are in
// flight); the draw kernel adds the segments in order.
__global__ __launch_bounds__(64) void k_hyper_reduce(const double *__restrict__ partials, int nblk,
                                                     int ne, double *__restrict__ seg_sums) {
  const int q = blockIdx.x * 64 + threadIdx.x;
  const int seg = blockIdx.y;
  if (q >= ne) return;
  const int per = (nblk + kReduceSegs - 1) / kReduceSegs;
  const int b0 = seg * per, b1 = min(nblk, b0 + per);
  double t = 0.0;
#pragma unroll 16
  for (int b = b0; b < b1; ++b) t += partials[(int64_t)b * ne + q];
  seg_sums[(int64_t)seg * ne + q] = t;
}

// 1 / sqrt(p) to about an ulp: the hardware estimate refined by Newton steps, each with about
// a third of the dependent instructions of the exactly rounded square root and division.
// Outside the range where p y y can neither overflow nor lose bits, those are used.
__device__ __forceinline__ double rsqrt_f64(double p) {
  if (!(p > 1e-280 && p < 1e280)) return 1.0 / sqrt(p);
  double y = __builtin_amdgcn_rsq(p);
#pragma unroll
  for (int it = 0; it < 3; ++it) {
    const double e = fma(-(p * y), y, 1.0);
    y = fma(0.5 * y, e, y);
  }
  return y;
}

// Normal-Wishart posterior and Bartlett draw in one workgroup of 32 x 32 threads. Thread
// (ti, tj) holds the entries (ti + 32 a, tj + 32 b), b <= a, of the lower triangle in
// registers; a step publishes one finished row through LDS, so it costs one barrier.
//   W*^{-1} = G^T G (G lower, from the last row up), hence F = G^{-1} is the lower Cholesky
//   factor of W* and needs no inverse and no second factorisation;
//   G E = B, solved from the first row down, gives E = F B;
//   Lambda = E E^T on fp64 MFMA (E staged square in LDS, zero above the diagonal);
//   sqrt(beta*) E is the Cholesky factor R of beta* Lambda, so mu = mu0* + R^{-T} zmu is one
//   back substitution.
// Bound by the latency of the 2 D dependent steps (LDS round trip, reciprocal square root,
// barrier): 106 us at D = 100 and 22 us at D = 20. Factoring W*^{-1}, inverting, multiplying
// out W* and F B with one thread per row or column and factoring twice more took 1052 and
// 67 us.
// extra (nullable): a packed upper triangle added to W*^{-1} (the time chain's steps).
// A pivot of W*^{-1} or of beta* Lambda = R R^T that is not positive and finite sets *status.
constexpr int kSampleThreads = 1024;
constexpr int kSquare = kMaxD + 2;  // doubles per row: even, and odd in units of 16 bytes

__global__ __launch_bounds__(kSampleThreads) void k_hyper_sample(
    const double *__restrict__ seg_sums, int64_t n, int D,
    const double *__restrict__ mu0, double beta0, const double *__restrict__ W0inv, double nu0,
    const double *__restrict__ chi2, const double *__restrict__ offd,
    const double *__restrict__ zmu, const double *__restrict__ extra,
    double *__restrict__ mu_out, double *__restrict__ Lam_out, int32_t *__restrict__ status) {
  constexpr int NB = kMaxD / 32;
  __shared__ double S[kMaxD * kSquare];  // the moments, then G, then E
  __shared__ double buf[2][kMaxD];       // the row published by a step
  __shared__ double xbar[kMaxD], dv[kMaxD], ginv[kMaxD];
  __shared__ int bad;
  const int tid = threadIdx.x, ti = tid >> 5, tj = tid & 31;
  const int ne = D + D * (D + 1) / 2;
  if (tid == 0) bad = 0;
  if (tid < 2 * kMaxD) buf[tid / kMaxD][tid % kMaxD] = 0.0;
  // the moments: segment sums added in segment order
  for (int q = tid; q < ne; q += kSampleThreads) {
    double t = 0.0;
#pragma unroll
    for (int g = 0; g < kReduceSegs; ++g) t += seg_sums[(int64_t)g * ne + q];
    S[q] = t;
  }
  __syncthreads();
  const double nn = (double)n;
  const double beta_s = beta0 + nn;
  const double shrink = beta_s > 0.0 ? beta0 * nn / beta_s : 0.0;
  if (tid < D) {
    xbar[tid] = n > 0 ? S[tid] / nn : 0.0;
    dv[tid] = mu0[tid] - xbar[tid];
  }
  __syncthreads();
  // W*^{-1} = W0^{-1} + (sum x x^T - n xbar xbar^T) + shrink dv dv^T (lower triangle)
  double A[NB][NB];
#pragma unroll
  for (int a = 0; a < NB; ++a) {
#pragma unroll
    for (int b = 0; b <= a; ++b) {
      const int i = ti + 32 * a, j = tj + 32 * b;
      double v = 0.0;
      if (i < D && j <= i) {
        const int q = j * D - j * (j - 1) / 2 + (i - j);
        v = W0inv[i * D + j] + (S[D + q] - nn * xbar[i] * xbar[j]) + shrink * dv[i] * dv[j] +
            (extra ? extra[q] : 0.0);
      }
      A[a][b] = v;
    }
  }
  __syncthreads();  // S is rewritten row by row from here on
  // W*^{-1} = G^T G: row k of G is row k of what the later rows leave, over its pivot's root
#pragma unroll
  for (int a = NB - 1; a >= 0; --a) {
    if (32 * a >= D) continue;
    for (int k = min(D, 32 * a + 32) - 1; k >= 32 * a; --k) {
      double *row = buf[k & 1];
      if (ti == k - 32 * a) {
#pragma unroll
        for (int b = 0; b <= a; ++b)
          if (tj + 32 * b <= k) row[tj + 32 * b] = A[a][b];
      }
      __syncthreads();
      double p = row[k];
      const bool ok = p > 0.0 && isfinite(p);
      if (!ok) p = 1.0;
      const double rs = rsqrt_f64(p), inv = rs * rs;
      // rows and columns from k on are finished: their registers no longer matter
#pragma unroll
      for (int c = 0; c <= a; ++c) {
        const double f = row[ti + 32 * c] * inv;
#pragma unroll
        for (int b = 0; b <= c; ++b) A[c][b] = fma(-f, row[tj + 32 * b], A[c][b]);
      }
      if (tid <= k) S[k * kSquare + tid] = tid == k ? p * rs : row[tid] * rs;
      if (tid == 0) {
        ginv[k] = rs;
        if (!ok) bad = 1;
      }
    }
  }
  // G E = B with Bartlett's B (B_ii = sqrt(chi2_i), B_ij normal below)
#pragma unroll
  for (int a = 0; a < NB; ++a) {
#pragma unroll
    for (int b = 0; b <= a; ++b) {
      const int i = ti + 32 * a, j = tj + 32 * b;
      A[a][b] = i < D && j <= i ? (j == i ? sqrt(chi2[i]) : offd[i * (i - 1) / 2 + j]) : 0.0;
    }
  }
  __syncthreads();  // G and ginv are complete
  bool fine = true;
#pragma unroll
  for (int a = 0; a < NB; ++a) {
    for (int k = 32 * a; k < min(D, 32 * a + 32); ++k) {
      double *row = buf[k & 1];
      if (ti == k - 32 * a) {
        const double r = ginv[k];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          const int j = tj + 32 * b;
          const double e = b <= a && j <= k ? A[a][b <= a ? b : a] * r : 0.0;
          // R's square in the entry, as a factorisation of beta* Lambda would meet it
          const double e2 = e * e * beta_s;
          fine = fine && isfinite(e2) && (j != k || (e > 0.0 && e2 > 0.0));
          row[j] = e;
        }
      }
      __syncthreads();
      // rows up to k are finished; row k of G makes place for row k of E
#pragma unroll
      for (int c = a; c < NB; ++c) {
        const double f = S[(ti + 32 * c) * kSquare + k];
#pragma unroll
        for (int b = 0; b <= a; ++b) A[c][b] = fma(-f, row[tj + 32 * b], A[c][b]);
      }
      if (tid < kMaxD) S[k * kSquare + tid] = row[tid];
    }
  }
  if (!fine) bad = 1;
  // rows past D, up to the 16-wide tiles of the product, are zero
  const int T = (D + 15) / 16;
  for (int q = tid; q < (16 * T - D) * kMaxD; q += kSampleThreads)
    S[(D + q / kMaxD) * kSquare + q % kMaxD] = 0.0;
  __syncthreads();
  if (tid < 64) {
    // mu = mu0* + R^{-T} zmu, R = sqrt(beta*) E: lane l holds the entries l and l + 64
    const double sb = sqrt(beta_s);
    double t[2], r[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int i = tid + 64 * h;
      t[h] = i < D ? zmu[i] : 0.0;
      r[h] = i < D ? 1.0 / (sb * S[i * kSquare + i]) : 0.0;
    }
#pragma unroll
    for (int h = 1; h >= 0; --h) {
      for (int i = min(D, 64 * h + 64) - 1; i >= 64 * h; --i) {
        const double y = __shfl(t[h] * r[h], i - 64 * h);
        if (tid == i - 64 * h) t[h] = y;
#pragma unroll
        for (int g = 0; g <= h; ++g)
          if (tid + 64 * g < i) t[g] = fma(-(sb * S[i * kSquare + tid + 64 * g]), y, t[g]);
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int i = tid + 64 * h;
      if (i < D) mu_out[i] = (beta0 * mu0[i] + nn * xbar[i]) / beta_s + t[h];
    }
  }
  // Lambda = E E^T: wave w takes the lower tiles w, w + 16, ...; lane (kq, c) supplies
  // row c's entry 4 s + kq of both tile rows and receives rows 4 r + kq, column c
  const int w = tid >> 6, lane = tid & 63, kq = lane >> 4, c = lane & 15;
  for (int t = w; t < T * (T + 1) / 2; t += kSampleThreads / 64) {
    int I = 0, J = t;
    while (J > I) {
      ++I;
      J -= I;
    }
    const double *ra = S + (16 * I + c) * kSquare + kq, *rb = S + (16 * J + c) * kSquare + kq;
    doublex4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int s = 0; s < 4 * (J + 1); ++s)
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(ra[4 * s], rb[4 * s], acc, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 16 * I + 4 * r + kq, j = 16 * J + c;
      if (i < D && j <= i) {
        Lam_out[i * D + j] = acc[r];
        Lam_out[j * D + i] = acc[r];
      }
    }
  }
  if (tid == 0) *status = bad ? 1 : 0;
}

// Row a and column b (a <= b) of packed upper-triangle entry t (rows in order).
__device__ inline void upper_entry(int t, int D, int &a, int &b) {
  a = 0;
  while (t >= D - a) {
    t -= D - a;
    ++a;
  }
  b = a + t;
}

__global__ __launch_bounds__(256) void k_time_rhs(const float *__restrict__ T, int64_t K, int D,
                                                  const double *__restrict__ Lam,
                                                  const double *__restrict__ mu, double inv_alpha,
                                                  int parity, float *__restrict__ h0) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t nk = (K - parity + 1) / 2;  // bins of this parity
  if (t >= nk * D) return;
  const int64_t k = parity + 2 * (t / D);
  const int a = (int)(t % D);
  double acc = 0.0;
  for (int e = 0; e < D; ++e) {
    const double prev = k == 0 ? mu[e] : (double)T[(k - 1) * D + e];
    const double next = k < K - 1 ? (double)T[(k + 1) * D + e] : 0.0;
    acc += Lam[a * D + e] * (prev + next);
  }
  h0[k * D + a] = (float)(acc * inv_alpha);
}

__global__ __launch_bounds__(256) void k_time_moments(const float *__restrict__ T, int D,
                                                      double *__restrict__ seg_sums) {
  const int ne = D + D * (D + 1) / 2;
  for (int q = blockIdx.x * 256 + threadIdx.x; q < kReduceSegs * ne; q += gridDim.x * 256) {
    const int g = q / ne, e = q % ne;
    double v = 0.0;
    if (g == 0) {
      if (e < D) {
        v = (double)T[e];
      } else {
        int a, b;
        upper_entry(e - D, D, a, b);
        v = (double)T[a] * (double)T[b];
      }
    }
    seg_sums[q] = v;
  }
}

// Block b takes the steps k = 1 + b per .. min(K, 1 + (b + 1) per) - 1, with the bins
// k - 1 .. of its slice staged in LDS (dynamic, (per + 1) D floats).
__global__ __launch_bounds__(256) void k_time_steps(const float *__restrict__ T, int64_t K, int D,
                                                    int64_t per, double *__restrict__ partials) {
  extern __shared__ float rows[];
  const int ntri = D * (D + 1) / 2;
  const int64_t k0 = 1 + (int64_t)blockIdx.x * per;
  const int64_t k1 = min(K, k0 + per);
  double *__restrict__ out = partials + (int64_t)blockIdx.x * ntri;
  const int nr = k0 < K ? (int)(k1 - k0 + 1) : 0;  // bins k0 - 1 .. k1 - 1
  for (int q = threadIdx.x; q < nr * D; q += 256) rows[q] = T[(k0 - 1) * D + q];
  __syncthreads();
  for (int q = threadIdx.x; q < ntri; q += 256) {
    int a, b;
    upper_entry(q, D, a, b);
    double acc = 0.0;
    for (int r = 1; r < nr; ++r)
      acc += ((double)rows[r * D + a] - (double)rows[(r - 1) * D + a]) *
             ((double)rows[r * D + b] - (double)rows[(r - 1) * D + b]);
    out[q] = acc;
  }
}

__global__ __launch_bounds__(256) void k_time_steps_sum(const double *__restrict__ partials,
                                                        int nblk, int ntri,
                                                        double *__restrict__ extra) {
  const int q = blockIdx.x * 256 + threadIdx.x;
  if (q >= ntri) return;
  double t = 0.0;
  for (int b = 0; b < nblk; ++b) t += partials[(int64_t)b * ntri + q];
  extra[q] = t;
}

}  // namespace

hipError_t launch_prior_prepare(const double *Lam, const double *mu, int D, int DP, double alpha,
                                bool need_factor, float *init, float *L, float *mu32, int32_t *ok,
                                hipStream_t s) {
  if (D < 1 || D > 128 || !(alpha > 0.0)) return hipErrorInvalidValue;
  const int LD = lane_width(D);
  const int aug_col = (!LD && ((D + 3) & ~3) < DP) ? ((D + 3) & ~3) : -1;
  hipLaunchKernelGGL(k_prior_prepare, dim3(1), dim3(kBayesBlock), 0, s, Lam, mu, D, DP, LD,
                     aug_col, alpha, need_factor ? 1 : 0, init, L, mu32, ok);
  return hipGetLastError();
}

hipError_t launch_prior_rows(const int32_t *rows, int64_t n, int D, const float *L,
                             const float *mu32, const int32_t *ok, const float *z, float *X,
                             int32_t *flag, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_prior_rows, dim3((unsigned)((n + 63) / 64)), dim3(64), 0, s, rows, n, D, L,
                     mu32, ok, z, X, flag);
  return hipGetLastError();
}

int hyper_blocks(int64_t n) {
  return (int)std::max<int64_t>(1, std::min<int64_t>(kHyperBlocks, (n + 63) / 64));
}

hipError_t launch_hyper_moments(const float *X, int64_t n, int D, double *partials, hipStream_t s) {
  if (D < 1 || D > 128) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_hyper_moments, dim3((unsigned)hyper_blocks(n)), dim3(kBayesBlock), 0, s, X,
                     n, D, partials);
  return hipGetLastError();
}

hipError_t launch_hyper_sample(const double *partials, int nblk, int64_t n, int D,
                               const double *mu0, double beta0, const double *W0inv, double nu0,
                               const double *chi2, const double *offd, const double *zmu,
                               double *scratch, double *mu_out, double *Lam_out, int32_t *status,
                               hipStream_t s) {
  if (D < 1 || D > 128 || nblk < 1) return hipErrorInvalidValue;
  const int ne = hyper_entries(D);
  double *seg_sums = scratch;
  hipLaunchKernelGGL(k_hyper_reduce, dim3((unsigned)((ne + 63) / 64), kReduceSegs), dim3(64), 0, s,
                     partials, nblk, ne, seg_sums);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_hyper_sample, dim3(1), dim3(kSampleThreads), 0, s, seg_sums, n, D, mu0,
                     beta0, W0inv, nu0, chi2, offd, zmu, (const double *)nullptr, mu_out, Lam_out,
                     status);
  return hipGetLastError();
}

hipError_t launch_time_rhs(const float *T, int64_t K, int D, const double *Lam, const double *mu,
                           double alpha, int parity, float *h0, hipStream_t s) {
  if (D < 1 || D > 128 || K < 1 || (parity != 0 && parity != 1) || !(alpha > 0.0))
    return hipErrorInvalidValue;
  const int64_t threads = (K - parity + 1) / 2 * D;
  if (threads == 0) return hipSuccess;
  hipLaunchKernelGGL(k_time_rhs, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, T, K,
                     D, Lam, mu, 1.0 / alpha, parity, h0);
  return hipGetLastError();
}

void time_step_blocks(int64_t K, int D, int64_t &per, int64_t &nblk) {
  const int64_t steps = std::max<int64_t>(K - 1, 0);
  const int64_t max_rows = kStepStageFloats / D;  // staged bins per block
  per = std::max<int64_t>(1, std::min<int64_t>((steps + kStepBlocks - 1) / kStepBlocks,
                                               max_rows - 1));
  nblk = std::max<int64_t>(1, (steps + per - 1) / per);
}

hipError_t launch_time_hyper(const float *T, int64_t K, int D, const double *mu0, double beta0,
                             const double *W0inv, double nu0, const double *chi2,
                             const double *offd, const double *zmu, double *scratch,
                             double *step_partials, double *extra, double *mu_out,
                             double *Lam_out, int32_t *status, hipStream_t s) {
  if (D < 1 || D > 128 || K < 1) return hipErrorInvalidValue;
  const int ne = hyper_entries(D), ntri = D * (D + 1) / 2;
  double *seg_sums = scratch;
  hipLaunchKernelGGL(k_time_moments, dim3((unsigned)((kReduceSegs * ne + 255) / 256)), dim3(256),
                     0, s, T, D, seg_sums);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  int64_t per = 0, nblk = 0;
  time_step_blocks(K, D, per, nblk);
  hipLaunchKernelGGL(k_time_steps, dim3((unsigned)nblk), dim3(256),
                     (size_t)(per + 1) * D * sizeof(float), s, T, K, D, per, step_partials);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_time_steps_sum, dim3((unsigned)((ntri + 255) / 256)), dim3(256), 0, s,
                     step_partials, (int)nblk, ntri, extra);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_hyper_sample, dim3(1), dim3(kSampleThreads), 0, s, seg_sums, (int64_t)1, D,
                     mu0, beta0, W0inv, nu0, chi2, offd, zmu, (const double *)extra, mu_out, Lam_out,
                     status);
  return hipGetLastError();
}

}  // namespace als
