// Held-out predictions r_hat = u_u . v_i (Sec. 2.2) and the squared errors of
// the validation RMSE (Sec. 4.1), for a list of (user, item) pairs.
//
// The work is two gathered D-vectors and one dot product per pair, so it is
// bound by memory. Rows are read with the widest loads that every row's alignment
// allows (float4 when D % 4 == 0, then float2, then float). A group of 4 or 8 lanes
// shares a pair, so that each load instruction reads contiguous row segments (the
// wave's 64 lanes touch 16 or 8 rows instead of 64), and the group's partial sums are
// added by shuffles; rows of fewer than four loads take one lane per pair, which has
// them all in flight before any arithmetic. The dot
// product runs with fused multiply-adds in fp32 (in feature order for one lane per
// pair; strided per lane, then a shuffle tree, for a group). Pairs whose
// indices fall outside the factor tables give NaN and read nothing. With
// ratings, each 256-lane block writes the fp64 sum of its pairs' squared
// errors; a fixed-order reduction follows, so the sum is reproducible.
#include <algorithm>

#include "internal.h"

namespace als {

namespace {

constexpr int kPairBlock = 256;
constexpr int kGroupLoads = 4;  // loads a row from which on a group of lanes shares a pair

// Floats per load: the widest that every row's alignment allows (16-byte aligned tables).
int predict_vec(int D) { return D % 4 == 0 ? 4 : D % 2 == 0 ? 2 : 1; }

// Lanes per pair: eight from 24 loads a row on, four from four, else one (float4 loads measured
// on the full-size workload's pairs: D = 20 0.106 ms with one lane and 0.072 with four, D = 100
// 0.735 and, with eight, 0.250). Us for 3M pairs with one lane and grouped: D = 5 39 and 32, 10
// 50 and 40, 13 111 and 42, 33 318 and 83, 50 286 and 105, 89 932 and 128, 127 1360 and 173.
int predict_group(int D) {
  const int nv = D / predict_vec(D);
  return nv >= 24 ? 8 : (nv >= kGroupLoads ? 4 : 1);
}

template <int VW> struct Vec;
template <> struct Vec<4> {
  using T = float4;
  static __device__ __forceinline__ float fma_dot(T a, T b, float acc) {
    acc = fmaf(a.x, b.x, acc);
    acc = fmaf(a.y, b.y, acc);
    acc = fmaf(a.z, b.z, acc);
    return fmaf(a.w, b.w, acc);
  }
};
template <> struct Vec<2> {
  using T = float2;
  static __device__ __forceinline__ float fma_dot(T a, T b, float acc) {
    acc = fmaf(a.x, b.x, acc);
    return fmaf(a.y, b.y, acc);
  }
};
template <> struct Vec<1> {
  using T = float;
  static __device__ __forceinline__ float fma_dot(T a, T b, float acc) { return fmaf(a, b, acc); }
};

// u . v over D features (D % VW == 0, fewer than kGroupLoads loads a row, both rows
// VW * 4-byte aligned), in feature order.
template <int VW>
__device__ __forceinline__ float row_dot(const float *__restrict__ u, const float *__restrict__ v,
                                         int D) {
  using T = typename Vec<VW>::T;
  const T *__restrict__ a = reinterpret_cast<const T *>(u);
  const T *__restrict__ b = reinterpret_cast<const T *>(v);
  const int nv = D / VW;
  T x[kGroupLoads - 1], y[kGroupLoads - 1];
#pragma unroll
  for (int k = 0; k < kGroupLoads - 1; ++k) {
    if (k < nv) {
      x[k] = a[k];
      y[k] = b[k];
    }
  }
  float acc = 0.f;
#pragma unroll
  for (int k = 0; k < kGroupLoads - 1; ++k)
    if (k < nv) acc = Vec<VW>::fma_dot(x[k], y[k], acc);
  return acc;
}

// G lanes share a pair (G a power of two, 1 < G <= 16, D % VW == 0): lane g of the group
// loads vectors g, g + G, ... of both rows, so that one load instruction of the wave reads
// whole contiguous row segments; the G partial sums are then added across the group.
template <int VW, int G, bool SSE>
__global__ __launch_bounds__(kPairBlock) void k_predict_group(
    const float *__restrict__ U, const float *__restrict__ V, int64_t M, int64_t N, int D,
    int64_t n, const int32_t *__restrict__ users, const int32_t *__restrict__ items,
    const uint8_t *__restrict__ r, float *__restrict__ pred, double *__restrict__ sse_blocks) {
  const int g = (int)threadIdx.x & (G - 1);
  const int64_t p = ((int64_t)blockIdx.x * kPairBlock + threadIdx.x) / G;
  double e2 = 0.0;
  float acc = 0.f;
  bool ok = false;
  double rv = 0.0;
  if (p < n) {
    const uint32_t u = (uint32_t)users[p], i = (uint32_t)items[p];
    rv = SSE ? (double)r[p] : 0.0;
    ok = ((uint64_t)u < (uint64_t)M) & ((uint64_t)i < (uint64_t)N);
    if (ok) {
      using T = typename Vec<VW>::T;
      const T *__restrict__ a = reinterpret_cast<const T *>(U + (int64_t)u * D);
      const T *__restrict__ b = reinterpret_cast<const T *>(V + (int64_t)i * D);
      const int nv = D / VW;
      constexpr int kIn = 4;  // vectors of each row in flight per lane
      for (int c0 = g; c0 < nv; c0 += kIn * G) {
        T x[kIn], y[kIn];
#pragma unroll
        for (int k = 0; k < kIn; ++k) {
          if (c0 + k * G < nv) {
            x[k] = a[c0 + k * G];
            y[k] = b[c0 + k * G];
          }
        }
#pragma unroll
        for (int k = 0; k < kIn; ++k)
          if (c0 + k * G < nv) acc = Vec<VW>::fma_dot(x[k], y[k], acc);
      }
    }
  }
#pragma unroll
  for (int o = G / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
  if (p < n && g == 0) {
    const float dot = ok ? acc : __builtin_nanf("");
    if (pred) pred[p] = dot;
    if (SSE) {
      const double e = rv - (double)dot;
      e2 = e * e;
    }
  }
  if (SSE) {
    __shared__ double wsum[kPairBlock / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) e2 += __shfl_xor(e2, o);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = e2;
    __syncthreads();
    if (threadIdx.x == 0) {
      double s = 0.0;
#pragma unroll
      for (int w = 0; w < kPairBlock / 64; ++w) s += wsum[w];
      sse_blocks[blockIdx.x] = s;
    }
  }
}

template <int VW, bool SSE>
__global__ __launch_bounds__(kPairBlock) void k_predict(
    const float *__restrict__ U, const float *__restrict__ V, int64_t M, int64_t N, int D,
    int64_t n, const int32_t *__restrict__ users, const int32_t *__restrict__ items,
    const uint8_t *__restrict__ r, float *__restrict__ pred, double *__restrict__ sse_blocks) {
  const int64_t p = (int64_t)blockIdx.x * kPairBlock + threadIdx.x;
  double e2 = 0.0;
  if (p < n) {
    // both indices (and the rating) are loaded before either is tested, so the two
    // index loads overlap; a negative index wraps to a large unsigned value
    const uint32_t u = (uint32_t)users[p], i = (uint32_t)items[p];
    const double rv = SSE ? (double)r[p] : 0.0;
    float dot = __builtin_nanf("");
    if (((uint64_t)u < (uint64_t)M) & ((uint64_t)i < (uint64_t)N))
      dot = row_dot<VW>(U + (int64_t)u * D, V + (int64_t)i * D, D);
    if (pred) pred[p] = dot;
    if (SSE) {
      const double e = rv - (double)dot;
      e2 = e * e;
    }
  }
  if (SSE) {
    __shared__ double wsum[kPairBlock / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) e2 += __shfl_xor(e2, o);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = e2;
    __syncthreads();
    if (threadIdx.x == 0) {
      double s = 0.0;
#pragma unroll
      for (int w = 0; w < kPairBlock / 64; ++w) s += wsum[w];
      sse_blocks[blockIdx.x] = s;
    }
  }
}

template <int VW, int G>
hipError_t launch_predict_group(const float *U, const float *V, int64_t M, int64_t N, int D,
                                int64_t n, const int32_t *users, const int32_t *items,
                                const uint8_t *r, float *pred, double *sse_blocks,
                                hipStream_t s) {
  const unsigned blocks = (unsigned)pair_blocks(n, D);
  if (sse_blocks)
    hipLaunchKernelGGL((k_predict_group<VW, G, true>), dim3(blocks), dim3(kPairBlock), 0, s, U, V,
                       M, N, D, n, users, items, r, pred, sse_blocks);
  else
    hipLaunchKernelGGL((k_predict_group<VW, G, false>), dim3(blocks), dim3(kPairBlock), 0, s, U,
                       V, M, N, D, n, users, items, r, pred, sse_blocks);
  return hipGetLastError();
}

template <int VW>
hipError_t launch_predict_vw(const float *U, const float *V, int64_t M, int64_t N, int D,
                             int64_t n, const int32_t *users, const int32_t *items,
                             const uint8_t *r, float *pred, double *sse_blocks, hipStream_t s) {
  const int G = predict_group(D);
  if (G == 8)
    return launch_predict_group<VW, 8>(U, V, M, N, D, n, users, items, r, pred, sse_blocks, s);
  if (G == 4)
    return launch_predict_group<VW, 4>(U, V, M, N, D, n, users, items, r, pred, sse_blocks, s);
  const unsigned blocks = (unsigned)pair_blocks(n, D);
  if (sse_blocks)
    hipLaunchKernelGGL((k_predict<VW, true>), dim3(blocks), dim3(kPairBlock), 0, s, U, V, M, N, D,
                       n, users, items, r, pred, sse_blocks);
  else
    hipLaunchKernelGGL((k_predict<VW, false>), dim3(blocks), dim3(kPairBlock), 0, s, U, V, M, N,
                       D, n, users, items, r, pred, sse_blocks);
  return hipGetLastError();
}

}  // namespace

int64_t pair_blocks(int64_t n, int D) {
  return (n * predict_group(D) + kPairBlock - 1) / kPairBlock;
}

hipError_t launch_predict(const float *U, const float *V, int64_t M, int64_t N, int D, int64_t n,
                          const int32_t *users, const int32_t *items, const uint8_t *r,
                          float *pred, double *sse_blocks, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (sse_blocks && !r) return hipErrorInvalidValue;
  const int vw = predict_vec(D), G = predict_group(D);
  const int64_t blocks = max_blocks(kPairBlock), per = blocks * kPairBlock / G;  // a launch's
  for (int64_t first = 0; first < n; first += per) {
    const int64_t k = std::min(per, n - first);
    const uint8_t *rk = r ? r + first : nullptr;
    float *pk = pred ? pred + first : nullptr;
    double *sk = sse_blocks ? sse_blocks + first / per * blocks : nullptr;
    const auto launch = vw == 4   ? launch_predict_vw<4>
                        : vw == 2 ? launch_predict_vw<2>
                                  : launch_predict_vw<1>;
    const hipError_t e =
        launch(U, V, M, N, D, k, users + first, items + first, rk, pk, sk, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace als
