// Operator set-up: the tiled block layouts and the self-block inverses.
#include "kernels.hpp"
#include "device.hpp"

namespace dc {

namespace {

// ------------------------------------------------------------------ layout
// Tiled layout: block = 8 x 8 lane grid of T x T sub-tiles; lane l = lr*8+lc
// owns rows lr*T .. lr*T+T-1 and columns lc*T .. lc*T+T-1; its element
// e = a*T + b is (lr*T + a, lc*T + b).  Element e of lane l lives in 16-byte
// unit (e / EPL)*64 + l, slot e % EPL.

__device__ uint16_t f64_to_f16_rne(double x) {
  const uint64_t b = __double_as_longlong(x);
  const uint16_t sign = uint16_t((b >> 48) & 0x8000u);
  const int exp = int((b >> 52) & 0x7ff);
  const uint64_t mant = b & ((uint64_t(1) << 52) - 1);
  if (exp == 0x7ff) return sign | 0x7c00u | (mant ? 0x200u : 0u);
  if (exp == 0) return sign;  // FP64 subnormals are far below the FP16 range
  const int e = exp - 1023;
  if (e > 15) return sign | 0x7c00u;
  const uint64_t m = mant | (uint64_t(1) << 52);
  const int shift = (e >= -14) ? 42 : 42 + (-14 - e);
  if (shift >= 64) return sign;
  uint64_t keep = m >> shift;
  const uint64_t rem = m & ((uint64_t(1) << shift) - 1);
  const uint64_t half = uint64_t(1) << (shift - 1);
  if (rem > half || (rem == half && (keep & 1))) keep += 1;
  if (e >= -14) {
    uint32_t hexp = uint32_t(e + 15);
    if (keep >= (uint64_t(1) << 11)) {
      keep >>= 1;
      hexp += 1;
    }
    if (hexp >= 31) return sign | 0x7c00u;
    return uint16_t(sign | (hexp << 10) | uint32_t(keep & 0x3ffu));
  }
  return uint16_t(sign | uint32_t(keep));  // subnormal (or the smallest normal)
}

// FP16 code of z / s, rounded to nearest even from the exact quotient (rs = 1 / s).
// z rs is within 2^-51 of the quotient, so rounding it to FP32 and then to FP16
// gives the same code unless the FP32 value is an FP16 midpoint; those (one in
// 8192), FP16 subnormals and values out of range take the exact division and
// the rounding on its bits.  (With a division per entry the conversion, not
// HBM, bound the kernels below.)
__device__ inline uint32_t f16_code(double z, double s, double rs) {
  const float q = float(z * rs);
  const uint32_t b = __float_as_uint(q), e = b & 0x7fffffffu;
  uint32_t h = __builtin_bit_cast(unsigned short, _Float16(q));
  if ((b & 0x1fffu) == 0x1000u || (e < 0x38800000u && e != 0u) || e >= 0x40000000u)
    h = f64_to_f16_rne(z / s);
  return h;
}

// A block entry as two FP16 codes of the block's scale (re low, im high).
__device__ inline uint32_t f16_pair(z64 z, double dscale, double rs) {
  return dscale > 0.0 ? f16_code(z.re, dscale, rs) | (f16_code(z.im, dscale, rs) << 16) : 0u;
}

// Largest of the 256 threads' values, in every thread.
__device__ inline double block_max(double v) {
  __shared__ double sh[4];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, shfl_xor(v, o));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  return fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
}

// The n x n matrix M (LDS, row-major) into block `blk` of each requested tiled
// layout, in whole 16-byte units; mx: its largest |Re|, |Im|.  256 threads.
template <int T>
__device__ inline void write_tiled(const z64* M, int n, double mx, size_t blk, z64* o64, z32* o32,
                                   float* mx32, uint32_t* o16, float* sc16) {
  constexpr int TT = T * T, U32 = (TT + 1) / 2, U16 = (TT + 3) / 4;
  const float scale = float(mx);
  const double dscale = double(scale), rs = 1.0 / dscale;
  if (threadIdx.x == 0) {
    if (o16) sc16[blk] = scale;
    if (mx32) mx32[blk] = scale;
  }
  auto entry = [&](int e, int lane) {
    const int a = e / T, b = e - a * T;
    const int i = (lane >> 3) * T + a, j = (lane & 7) * T + b;
    return e < TT && i < n && j < n ? M[i * n + j] : mk(0.0, 0.0);
  };
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (o64)
    for (int e = wave; e < TT; e += 4) o64[(blk * TT + e) * 64 + lane] = entry(e, lane);
  if (o32)
    for (int u = wave; u < U32; u += 4) {
      const z64 x = entry(2 * u, lane), y = entry(2 * u + 1, lane);
      reinterpret_cast<float4*>(o32)[(blk * U32 + u) * 64 + lane] =
          make_float4(float(x.re), float(x.im), float(y.re), float(y.im));
    }
  if (o16)
    for (int u = wave; u < U16; u += 4) {
      uint32_t w[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) w[q] = f16_pair(entry(4 * u + q, lane), dscale, rs);
      reinterpret_cast<uint4*>(o16)[(blk * U16 + u) * 64 + lane] = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// One workgroup per stored block (site, slot: 0 the self block, 1 + mu a hop
// block).  HBM bound: the block is read once, coalesced, into LDS, where its
// largest entry is found, and every layout is written from there in whole
// 16-byte units.  8^4, n = 48, FP64 and FP16 (1.7 GB): 465 -> 312 us, 5.4 TB/s.
template <int T>
__global__ __launch_bounds__(256) void k_layout(const z64* __restrict__ self_in,
                                                const z64* __restrict__ hops_in, int n, z64* o64,
                                                z32* o32, float* mx32, uint32_t* o16, float* sc16) {
  extern __shared__ z64 M[];               // n*n entries
  const size_t blk = blockIdx.x;           // site*5 + slot
  const size_t site = blk / 5, slot = blk - 5 * site;
  const int nn = n * n;
  const z64* src = slot == 0 ? self_in + site * nn : hops_in + (site * 4 + (slot - 1)) * nn;
  double mx = 0.0;
  for (int t = threadIdx.x; t < nn; t += 256) {
    const z64 z = src[t];
    M[t] = z;
    mx = fmax(mx, fmax(fabs(z.re), fabs(z.im)));
  }
  mx = block_max(mx);   // its barrier also completes M
  write_tiled<T>(M, n, mx, blk, o64, o32, mx32, o16, sc16);
}

// ------------------------------------------------------------------ inverses
// Gauss-Jordan inversion with partial pivoting of each site's self block A_x +
// i*tm*Gamma5, one wave per site.  The matrix stays in the registers of the tiled
// layout (lane (lr, lc) holds the T x T entries (lr T + a, lc T + b)), so it is read
// and written as whole units without staging, and a step exchanges one column
// (multipliers and pivot search) and the pivot row through LDS, with no barrier
// between waves.  The pivot search takes one lane per row and compares |Re| + |Im|
// by the FP64 exponent and 14 leading bits (a pivot within 2^-14 of the largest
// serves the same purpose), ties to the lower row.  Row interchanges are made as
// they come, the column interchanges that undo them in one permutation at the
// end, a strip of eight rows at a time through LDS.
// Bound by instruction issue (about 450 per column, 4 T^2 of them FMAs) at two
// waves per SIMD.  8^4, n = 48, FP64 and FP16 outputs: 990 us (matrix in LDS,
// four waves and barriers per column, bound by LDS passes) -> 340 us (registers
// of four waves, two barriers) -> 279-286 us.
template <int T>
__global__ __launch_bounds__(64) void k_invert_blocks(const z64* __restrict__ tiled64, int n,
                                                      double tm, z64* o64, z32* o32,
                                                      uint32_t* o16, float* sc16,
                                                      int* __restrict__ singular) {
  constexpr int TT = T * T, U32 = (TT + 1) / 2, U16 = (TT + 3) / 4;
  // entry i of a column or row sits at (i / T) S + i % T: the eight lanes that read
  // T entries each start S = T or T + 1 (odd) entries apart, without bank conflicts
  constexpr int S = T | 1;
  __shared__ z64 strip[8 * 8 * S];
  z64* const col = strip;              // column k
  z64* const prow = strip + 8 * S;     // pivot row
  z64* const krow = strip + 16 * S;    // row k, which goes where the pivot row was
  const size_t site = blockIdx.x;
  const int lane = threadIdx.x, lr = lane >> 3, lc = lane & 7;
  const z64* src = tiled64 + site * 5 * TT * 64;  // slot 0 of the site: A_x
  z64 m[T][T];
#pragma unroll
  for (int a = 0; a < T; ++a)
#pragma unroll
    for (int b = 0; b < T; ++b) m[a][b] = src[(a * T + b) * 64 + lane];
  if (lr == lc) {
#pragma unroll
    for (int a = 0; a < T; ++a)
      if (lr * T + a < n) m[a][a].im += (lr * T + a < (n >> 1)) ? tm : -tm;
  }
  int swapped = lane;   // lane k: the row exchanged with row k
  for (int kt = 0; kt < 8; ++kt) {
#pragma unroll
    for (int kb = 0; kb < T; ++kb) {
      const int k = kt * T + kb;
      if (k < n) {
        if (lc == kt) {
#pragma unroll
          for (int a = 0; a < T; ++a) col[lr * S + a] = m[a][kb];
        }
        __syncthreads();
        const z64 cv = lane < 8 * T ? col[lane / T * S + lane % T] : mk(0.0, 0.0);
        const double mag = fabs(cv.re) + fabs(cv.im);
        const bool in = lane >= k && lane < n, can = in && mag > 0.0;
        uint32_t key = in ? uint32_t(63 - lane) : 0u;
        if (can) key |= uint32_t(__double_as_longlong(mag) >> 32) & ~63u;
        key = max(key, uint32_t(dpp_xor1(int(key))));
        key = max(key, uint32_t(dpp_xor2(int(key))));
        key = max(key, uint32_t(dpp_hmirror(int(key))));
        key = max(key, uint32_t(dpp_ror8(int(key))));
        const auto r16 = __builtin_amdgcn_permlane16_swap(key, key, false, false);
        key = max(uint32_t(r16[0]), uint32_t(r16[1]));
        const auto r32 = __builtin_amdgcn_permlane32_swap(key, key, false, false);
        key = max(uint32_t(r32[0]), uint32_t(r32[1]));
        const int p = __builtin_amdgcn_readfirstlane(63 - int(key & 63u));
        const int lp = p / T, ap = p - lp * T;
        if (__builtin_amdgcn_ballot_w64(can) == 0 && lane == 0) *singular = 1;
        if (lane == k) swapped = p;
#pragma unroll
        for (int a = 0; a < T; ++a)
          if (a == ap && lr == lp) {
#pragma unroll
            for (int b = 0; b < T; ++b) prow[lc * S + b] = m[a][b];
          }
        if (lr == kt) {
#pragma unroll
          for (int b = 0; b < T; ++b) krow[lc * S + b] = m[kb][b];
        }
        z64 f[T], pr[T];
#pragma unroll
        for (int a = 0; a < T; ++a) f[a] = col[lr * S + a];
        const z64 akk = col[lp * S + ap], ck = col[kt * S + kb];
        const double den = akk.re * akk.re + akk.im * akk.im;
        const z64 d = den > 0.0 ? mk(akk.re / den, -akk.im / den) : mk(0.0, 0.0);  // 1 / a_kk
        __syncthreads();
#pragma unroll
        for (int b = 0; b < T; ++b) {
          z64 v = prow[lc * S + b];
          if (lc == kt && b == kb) v = mk(1.0, 0.0);
          pr[b] = mk(v.re * d.re - v.im * d.im, v.re * d.im + v.im * d.re);
        }
        if (p != k) {
#pragma unroll
          for (int a = 0; a < T; ++a)
            if (a == ap && lr == lp) {
              f[a] = ck;
#pragma unroll
              for (int b = 0; b < T; ++b) m[a][b] = krow[lc * S + b];
            }
        }
        // M[i][j] = (j == k ? 0 : M[i][j]) - f_i pr_j, and row k becomes the scaled pivot
        // row: 0 - (-1) pr_j
        if (lc == kt) {
#pragma unroll
          for (int a = 0; a < T; ++a) m[a][kb] = mk(0.0, 0.0);
        }
        if (lr == kt) {
          f[kb] = mk(-1.0, 0.0);
#pragma unroll
          for (int b = 0; b < T; ++b) m[kb][b] = mk(0.0, 0.0);
        }
#pragma unroll
        for (int a = 0; a < T; ++a)
#pragma unroll
          for (int b = 0; b < T; ++b) {
            m[a][b].re -= f[a].re * pr[b].re - f[a].im * pr[b].im;
            m[a][b].im -= f[a].re * pr[b].im + f[a].im * pr[b].re;
          }
        __syncthreads();
      }
    }
  }
  // where each column goes when the interchanges are undone, last first
  int dest = lane;
  for (int k = n - 1; k >= 0; --k) {
    const int p = __builtin_amdgcn_readlane(swapped, k);
    dest = dest == k ? p : (dest == p ? k : dest);
  }
  int dj[T];
#pragma unroll
  for (int b = 0; b < T; ++b) {
    const int j = __shfl(dest, lc * T + b, kWave);
    dj[b] = j / T * S + j % T;
  }
  double mx = 0.0;
#pragma unroll
  for (int a = 0; a < T; ++a) {
#pragma unroll
    for (int b = 0; b < T; ++b) strip[lr * 8 * S + dj[b]] = m[a][b];
    __syncthreads();
#pragma unroll
    for (int b = 0; b < T; ++b) {
      z64 z = strip[lr * 8 * S + lc * S + b];
      if (lr * T + a >= n || lc * T + b >= n) z = mk(0.0, 0.0);
      m[a][b] = z;
      mx = fmax(mx, fmax(fabs(z.re), fabs(z.im)));
    }
    __syncthreads();
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, shfl_xor(mx, o));
  const float scale = float(mx);
  const double dscale = double(scale), rs = 1.0 / dscale;
  auto entry = [&](int e) { return e < TT ? m[e / T][e % T] : mk(0.0, 0.0); };
  if (o64) {
#pragma unroll
    for (int e = 0; e < TT; ++e) o64[(site * TT + e) * 64 + lane] = m[e / T][e % T];
  }
  if (o32) {
#pragma unroll
    for (int u = 0; u < U32; ++u) {
      const z64 x = entry(2 * u), y = entry(2 * u + 1);
      reinterpret_cast<float4*>(o32)[(site * U32 + u) * 64 + lane] =
          make_float4(float(x.re), float(x.im), float(y.re), float(y.im));
    }
  }
  if (o16) {
    if (lane == 0) sc16[site] = scale;
#pragma unroll
    for (int u = 0; u < U16; ++u) {
      uint32_t w[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) w[q] = f16_pair(entry(4 * u + q), dscale, rs);
      reinterpret_cast<uint4*>(o16)[(site * U16 + u) * 64 + lane] = make_uint4(w[0], w[1], w[2], w[3]);
    }
  }
}

template <typename K>
void allow_lds(K kernel, size_t bytes) {
  DC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                             hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes)));
}

}  // namespace

void launch_layout_blocks(const z64* self_in, const z64* hops_in, int V, int n, void* out64,
                          void* out32, float* max32, void* out16, float* scales16,
                          hipStream_t st) {
  const size_t lds = size_t(n) * n * sizeof(z64);
  switch (tile_T(n)) {
#define DC_CASE(TV)                                                                              \
  case TV:                                                                                       \
    allow_lds(&k_layout<TV>, lds);                                                               \
    hipLaunchKernelGGL(k_layout<TV>, dim3(unsigned(V) * 5u), dim3(256), lds, st, self_in,        \
                       hops_in, n, static_cast<z64*>(out64), static_cast<z32*>(out32),           \
                       out32 ? max32 : nullptr, static_cast<uint32_t*>(out16), scales16);        \
    break;
    DC_CASE(1) DC_CASE(2) DC_CASE(3) DC_CASE(4) DC_CASE(5) DC_CASE(6) DC_CASE(7) DC_CASE(8)
#undef DC_CASE
    default:
      throw InvalidArg("block size n > 64 is not supported");
  }
  DC_HIP(hipGetLastError());
}

void launch_invert_blocks(const void* tiled64, int V, int n, double tm, void* out64, void* out32,
                          void* out16, float* scales16, int* singular, hipStream_t st) {
  switch (tile_T(n)) {
#define DC_CASE(TV)                                                                             \
  case TV:                                                                                      \
    hipLaunchKernelGGL(k_invert_blocks<TV>, dim3(unsigned(V)), dim3(64), 0, st,                 \
                       static_cast<const z64*>(tiled64), n, tm, static_cast<z64*>(out64),       \
                       static_cast<z32*>(out32), static_cast<uint32_t*>(out16), scales16,       \
                       singular);                                                               \
    break;
    DC_CASE(1) DC_CASE(2) DC_CASE(3) DC_CASE(4) DC_CASE(5) DC_CASE(6) DC_CASE(7) DC_CASE(8)
#undef DC_CASE
    default:
      throw InvalidArg("block size n > 64 is not supported");
  }
  DC_HIP(hipGetLastError());
}

}  // namespace dc
