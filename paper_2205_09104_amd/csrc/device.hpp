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
