// Device helpers shared by the kernel files.
#pragma once

#include "common.hpp"

namespace dc {
namespace {

constexpr int kWave = 64;

template <typename T>
__device__ inline T shfl_xor(T v, int m) {
  return __shfl_xor(v, m, kWave);
}

__device__ inline double gam(int i, int n) { return i < (n >> 1) ? 1.0 : -1.0; }

// Block-wide sum of W doubles per thread (blockDim.x a multiple of 64, <= 1024),
// written as this block's partial: partials[w * nblk + block].  A second
// kernel (k_finalize) sums the partials of each value in a fixed order, so
// every reduction is deterministic.
template <int W>
__device__ void block_partials_at(double (&v)[W], double* partials, int bid, int nblk) {
  __shared__ double sh[16][W];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int nw = blockDim.x / kWave;
#pragma unroll
  for (int t = 0; t < W; ++t) {
    double s = v[t];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += shfl_xor(s, o);
    if (lane == 0) sh[wave][t] = s;
  }
  __syncthreads();
  if (threadIdx.x < W) {
    double s = 0.0;
    for (int w = 0; w < nw; ++w) s += sh[w][threadIdx.x];
    partials[size_t(threadIdx.x) * nblk + bid] = s;
  }
}

template <int W>
__device__ void block_partials(double (&v)[W], double* partials) {
  block_partials_at<W>(v, partials, blockIdx.x + blockIdx.y * gridDim.x, gridDim.x * gridDim.y);
}

// result[v] = sum_b partials[v * nparts + b]; one 64-lane wave per value.
__device__ inline void finalize_value(const double* __restrict__ partials, int nparts,
                                      double* __restrict__ result, int v) {
  const double* p = partials + size_t(v) * nparts;
  double s = 0.0;
  for (int b = threadIdx.x; b < nparts; b += 512) {   // eight loads in flight, added in order
    double t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) t[u] = p[min(b + 64 * u, nparts - 1)];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (b + 64 * u < nparts) s += t[u];
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += shfl_xor(s, o);
  if (threadIdx.x == 0) result[v] = s;
}

inline unsigned grid_for(size_t N, int threads, unsigned cap = 4096) {
  size_t b = (N + threads - 1) / threads;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return unsigned(b);
}

// blocks of a single-value reduction over N elements: >= 4 elements per
// thread, at most 512 partials
inline unsigned red_blocks(size_t N) {
  size_t b = (N + 1023) / 1024;
  if (b < 1) b = 1;
  if (b > 512) b = 512;
  return unsigned(b);
}

// Lane exchanges by DPP: lane ^ 1, lane ^ 2, the half-row mirror and a rotation
// of a 16-lane row by 8.
__device__ inline int dpp_xor1(int v) { return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, false); }
__device__ inline int dpp_xor2(int v) { return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, false); }
__device__ inline int dpp_hmirror(int v) { return __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, false); }
__device__ inline int dpp_ror8(int v) { return __builtin_amdgcn_mov_dpp(v, 0x128, 0xF, 0xF, false); }

// The two FP16 values of a packed 32-bit word, widened.
__device__ inline float lo_h(uint32_t w) {
  return float(__builtin_bit_cast(_Float16, static_cast<unsigned short>(w & 0xffffu)));
}
__device__ inline float hi_h(uint32_t w) {
  return float(__builtin_bit_cast(_Float16, static_cast<unsigned short>(w >> 16)));
}

// 16x16x4 matrix products with accumulators of the operand type.
template <typename VT>
struct Mfma;
template <>
struct Mfma<float> {
  using acc_t = __attribute__((ext_vector_type(4))) float;
  __device__ static acc_t mma(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  __device__ static int row(int lk, int q) { return lk * 4 + q; }
};
template <>
struct Mfma<double> {
  using acc_t = __attribute__((ext_vector_type(4))) double;
  __device__ static acc_t mma(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  __device__ static int row(int lk, int q) { return lk + 4 * q; }
};

}  // namespace
}  // namespace dc
