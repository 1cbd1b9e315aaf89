// Krylov-space kernels: Gram-Schmidt reductions, tall-skinny combinations,
// conversions and the Arnoldi bookkeeping.
#include "kernels.hpp"
#include "device.hpp"

#include <algorithm>

namespace dc {

namespace {

__global__ __launch_bounds__(64) void k_finalize(const double* __restrict__ partials, int nparts,
                                                 double* __restrict__ result,
                                                 const int* __restrict__ done) {
  if (done && *done) return;
  finalize_value(partials, nparts, result, blockIdx.x);
}

// ------------------------------------------------------------------ BLAS
// Dot products and updates against a basis of Q vectors.  Each thread takes
// E elements per pass and issues the loads of all G basis vectors of a chunk
// before any arithmetic, so 2*G*E independent loads are in flight per lane
// (a load-use-load chain would leave one).  Accumulation is in FP64.
constexpr int kDotE = 2;     // elements per thread per pass
constexpr int kAxpyG = 16;   // basis vectors per chunk of the update kernel

template <typename VR>
__device__ inline const cx<VR>* basis_ptr(const cx<VR>* b0, int q0, const cx<VR>* b1, size_t N,
                                          int q) {
  return q < q0 ? b0 + size_t(q) * N : b1 + size_t(q - q0) * N;
}

// Wave sums of V per-lane values (V a power of two, at most 64) by halving
// exchanges: at each step a lane keeps one half of its values, sends the other
// half to its partner and adds what it receives, so after log2(V) steps lane l
// holds one value, index l / (64 / V), summed over V lanes; the remaining
// steps are a plain butterfly.  V - 1 + 6 - log2(V) exchanges instead of 6 V,
// in a fixed order.
template <int V, int S = 0>
__device__ inline void halving_steps(double (&acc)[V], int lane) {
  if constexpr ((V >> S) > 1) {
    constexpr int half = V >> (S + 1);
    constexpr int o = 32 >> S;
    const bool upper = (lane & o) != 0;
#pragma unroll
    for (int i = 0; i < half; ++i) {
      const double send = upper ? acc[i] : acc[i + half];
      const double keep = upper ? acc[i + half] : acc[i];
      acc[i] = keep + shfl_xor(send, o);
    }
    halving_steps<V, S + 1>(acc, lane);
  }
}

template <int V>
__device__ inline double wave_sum_many(double (&acc)[V], int lane) {
  halving_steps<V>(acc, lane);
  double v = acc[0];
#pragma unroll
  for (int o = 32 / V; o > 0; o >>= 1) v += shfl_xor(v, o);
  return v;
}

// result value v = by * 2G + t of the group; t = 2*(q - g0) + re/im.  Block
// bx of gx along the vector, by along the values (blockIdx of a plain launch).
template <typename VR, int G>
__device__ __forceinline__ void multidot_body(const cx<VR>* __restrict__ b0, int q0,
                                              const cx<VR>* __restrict__ b1, int q1, size_t N,
                                              const cx<VR>* __restrict__ w,
                                              double* __restrict__ partials, int bx, int gx,
                                              int by) {
  const int Qb = q0 + q1;
  const int g0 = by * G;
  const cx<VR>* ptr[G];
#pragma unroll
  for (int t = 0; t < G; ++t) {
    const int q = g0 + t;
    ptr[t] = q < Qb ? basis_ptr(b0, q0, b1, N, q) : w;  // past the basis: w itself (the norm)
  }
  double acc[2 * G];
#pragma unroll
  for (int t = 0; t < 2 * G; ++t) acc[t] = 0.0;
  const size_t chunk = size_t(blockDim.x) * kDotE;
  const size_t stride = size_t(gx) * chunk;
  for (size_t base = size_t(bx) * chunk + threadIdx.x; base < N; base += stride) {
    size_t idx[kDotE];
    double wr[kDotE], wi[kDotE];
#pragma unroll
    for (int e = 0; e < kDotE; ++e) {
      const size_t i = base + size_t(e) * blockDim.x;
      idx[e] = i < N ? i : N - 1;
    }
    cx<VR> v[G][kDotE], wv[kDotE];
#pragma unroll
    for (int e = 0; e < kDotE; ++e) wv[e] = w[idx[e]];
#pragma unroll
    for (int t = 0; t < G; ++t)
#pragma unroll
      for (int e = 0; e < kDotE; ++e) v[t][e] = ptr[t][idx[e]];
    __builtin_amdgcn_sched_barrier(0);  // keep every load ahead of the arithmetic
#pragma unroll
    for (int e = 0; e < kDotE; ++e) {
      const bool ok = base + size_t(e) * blockDim.x < N;
      wr[e] = ok ? double(wv[e].re) : 0.0;
      wi[e] = ok ? double(wv[e].im) : 0.0;
    }
#pragma unroll
    for (int t = 0; t < G; ++t)
#pragma unroll
      for (int e = 0; e < kDotE; ++e) {
        const double vr = v[t][e].re, vi = v[t][e].im;
        acc[2 * t] = fma(vr, wr[e], fma(vi, wi[e], acc[2 * t]));        // Re conj(v) w
        acc[2 * t + 1] = fma(vr, wi[e], fma(-vi, wr[e], acc[2 * t + 1]));  // Im conj(v) w
      }
  }
  __shared__ double sh[4][2 * G];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const double s = wave_sum_many<2 * G>(acc, lane);
  constexpr int kSpan = 64 / (2 * G);   // lanes holding the same value
  if (lane % kSpan == 0) sh[wave][lane / kSpan] = s;
  __syncthreads();
  if (threadIdx.x < 2 * G) {
    double s = 0.0;
    for (int wv2 = 0; wv2 < int(blockDim.x >> 6); ++wv2) s += sh[wv2][threadIdx.x];
    partials[(size_t(by) * 2 * G + threadIdx.x) * gx + bx] = s;
  }
}

template <typename VR, int G>
__global__ __launch_bounds__(256) void k_multidot(const cx<VR>* __restrict__ b0, int q0,
                                                  const cx<VR>* __restrict__ b1, int q1,
                                                  size_t N, const cx<VR>* __restrict__ w,
                                                  Reducer red, const int* __restrict__ done,
                                                  int* go, int step) {
  if (done && *done) return;
  if (go && blockIdx.x + blockIdx.y + threadIdx.x == 0) *go = step;
  multidot_body<VR, G>(b0, q0, b1, q1, N, w, red.partials, blockIdx.x, gridDim.x, blockIdx.y);
}

// The update kernels split the basis between the kSplitWaves waves of a
// workgroup: each wave takes every kSplitWaves-th chunk of kAxpyG vectors (the
// loads of a chunk issued before their arithmetic) for the same 64 kDotE
// elements, so a wave waits on a quarter of the chunks; the partial sums are
// then combined through LDS in a fixed order.  Elements of a pass:
// base + e 64 + lane.
constexpr int kSplitWaves = 4;   // waves per workgroup (256 threads)

template <typename VR, int G>
__device__ inline void split_sums(const cx<VR>* __restrict__ b0, int q0,
                                  const cx<VR>* __restrict__ b1, size_t N, int Q,
                                  const double* __restrict__ coef, size_t base, int lane,
                                  int wave, size_t (&idx)[kDotE], double (&sr)[kDotE],
                                  double (&si)[kDotE]) {
#pragma unroll
  for (int e = 0; e < kDotE; ++e) {
    const size_t i = base + size_t(e) * 64 + lane;
    idx[e] = i < N ? i : N - 1;
    sr[e] = si[e] = 0.0;
  }
  for (int qc = wave * G; qc < Q; qc += kSplitWaves * G) {
    cx<VR> v[G][kDotE];
#pragma unroll
    for (int t = 0; t < G; ++t) {
      const int q = min(qc + t, Q - 1);
      const cx<VR>* p = basis_ptr(b0, q0, b1, N, q);
#pragma unroll
      for (int e = 0; e < kDotE; ++e) v[t][e] = p[idx[e]];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < G; ++t) {
      const int q = qc + t;
      const double cr = q < Q ? coef[2 * q] : 0.0, ci = q < Q ? coef[2 * q + 1] : 0.0;
#pragma unroll
      for (int e = 0; e < kDotE; ++e) {
        const double vr = v[t][e].re, vi = v[t][e].im;
        sr[e] = fma(cr, vr, fma(-ci, vi, sr[e]));
        si[e] = fma(cr, vi, fma(ci, vr, si[e]));
      }
    }
  }
}

// out = (w - sum_q coef_q basis_q) sc; out may be w.  Block bx of gx (blockIdx.x /
// gridDim.x of a plain launch).
template <typename VR, int G = kAxpyG>
__device__ __forceinline__ void multiaxpy_split_body(const cx<VR>* w, cx<VR>* out,
                                                     const cx<VR>* __restrict__ b0, int q0,
                                                     const cx<VR>* __restrict__ b1, int q1,
                                                     size_t N, const double* __restrict__ coef,
                                                     int want_norm, double* partials, double sc,
                                                     int bx, int gx) {
  const int Q = q0 + q1;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __shared__ double part[kSplitWaves][kDotE][2][64];
  double nacc[1] = {0.0};
  const size_t span = size_t(64) * kDotE;
  for (size_t base = size_t(bx) * span; base < N; base += size_t(gx) * span) {
    size_t idx[kDotE];
    double sr[kDotE], si[kDotE];
    split_sums<VR, G>(b0, q0, b1, N, Q, coef, base, lane, wave, idx, sr, si);
#pragma unroll
    for (int e = 0; e < kDotE; ++e) {
      part[wave][e][0][lane] = sr[e];
      part[wave][e][1][lane] = si[e];
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int e = 0; e < kDotE; ++e) {
        if (base + size_t(e) * 64 + lane < N) {
          const cx<VR> wv = w[idx[e]];
          double r = wv.re, im = wv.im;
#pragma unroll
          for (int v2 = 0; v2 < kSplitWaves; ++v2) {
            r -= part[v2][e][0][lane];
            im -= part[v2][e][1][lane];
          }
          const cx<VR> o = mk(VR(r * sc), VR(im * sc));
          out[idx[e]] = o;
          nacc[0] += double(o.re) * double(o.re) + double(o.im) * double(o.im);
        }
      }
    }
    __syncthreads();
  }
  if (want_norm) block_partials_at<1>(nacc, partials, bx, gx);
}

template <typename VR>
__global__ __launch_bounds__(256) void k_multiaxpy(const cx<VR>* w, cx<VR>* out,
                                                   const cx<VR>* __restrict__ b0, int q0,
                                                   const cx<VR>* __restrict__ b1, int q1,
                                                   size_t N, const double* __restrict__ coef,
                                                   int want_norm, Reducer red,
                                                   const int* __restrict__ done) {
  if (done && *done) return;
  multiaxpy_split_body<VR>(w, out, b0, q0, b1, q1, N, coef, want_norm, red.partials,
                           1.0, blockIdx.x, gridDim.x);
}

// Bases of at most one chunk (kAxpyG vectors): nothing to split between the
// waves, so each thread takes its own kDotE elements through the whole basis.
template <typename VR>
__device__ __forceinline__ void multiaxpy_flat_body(const cx<VR>* w, cx<VR>* out,
                                                    const cx<VR>* __restrict__ b0, int q0,
                                                    const cx<VR>* __restrict__ b1, int q1,
                                                    size_t N, const double* __restrict__ coef,
                                                    int want_norm, double* partials, double sc,
                                                    int bx, int gx) {
  const int Q = q0 + q1;
  double nacc[1] = {0.0};
  const size_t chunk = size_t(blockDim.x) * kDotE;
  const size_t stride = size_t(gx) * chunk;
  for (size_t base = size_t(bx) * chunk + threadIdx.x; base < N; base += stride) {
    size_t idx[kDotE];
    double sr[kDotE], si[kDotE];
#pragma unroll
    for (int e = 0; e < kDotE; ++e) {
      const size_t i = base + size_t(e) * blockDim.x;
      idx[e] = i < N ? i : N - 1;
      const cx<VR> wv = w[idx[e]];
      sr[e] = wv.re;
      si[e] = wv.im;
    }
    for (int qc = 0; qc < Q; qc += kAxpyG) {
      cx<VR> v[kAxpyG][kDotE];
#pragma unroll
      for (int t = 0; t < kAxpyG; ++t) {
        const int q = min(qc + t, Q - 1);
        const cx<VR>* p = basis_ptr(b0, q0, b1, N, q);
#pragma unroll
        for (int e = 0; e < kDotE; ++e) v[t][e] = p[idx[e]];
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < kAxpyG; ++t) {
        const int q = qc + t;
        const double cr = q < Q ? coef[2 * q] : 0.0, ci = q < Q ? coef[2 * q + 1] : 0.0;
#pragma unroll
        for (int e = 0; e < kDotE; ++e) {
          const double vr = v[t][e].re, vi = v[t][e].im;
          sr[e] = fma(-cr, vr, fma(ci, vi, sr[e]));
          si[e] = fma(-cr, vi, fma(-ci, vr, si[e]));
        }
      }
    }
#pragma unroll
    for (int e = 0; e < kDotE; ++e) {
      if (base + size_t(e) * blockDim.x < N) {
        const cx<VR> o = mk(VR(sr[e] * sc), VR(si[e] * sc));
        out[idx[e]] = o;
        nacc[0] += double(o.re) * double(o.re) + double(o.im) * double(o.im);
      }
    }
  }
  if (want_norm) block_partials_at<1>(nacc, partials, bx, gx);
}

template <typename VR>
__global__ __launch_bounds__(256) void k_multiaxpy_flat(const cx<VR>* w, cx<VR>* out,
                                                   const cx<VR>* __restrict__ b0, int q0,
                                                   const cx<VR>* __restrict__ b1, int q1,
                                                   size_t N, const double* __restrict__ coef,
                                                   int want_norm, Reducer red,
                                                   const int* __restrict__ done) {
  if (done && *done) return;
  multiaxpy_flat_body<VR>(w, out, b0, q0, b1, q1, N, coef, want_norm, red.partials,
                          1.0, blockIdx.x, gridDim.x);
}

constexpr int kCombR = 16;  // outputs per pass of the combine kernel
constexpr int kCombMfmaMin = 16;   // from this many outputs on: the MFMA block update

template <typename VR>
__global__ __launch_bounds__(256) void k_combine(const cx<VR>* __restrict__ b0, int q0,
                                                 const cx<VR>* __restrict__ b1, int q1,
                                                 size_t N, const double* __restrict__ coef,
                                                 int R, cx<VR>* __restrict__ out, int accumulate) {
  const int Q = q0 + q1;
  const int r0 = blockIdx.y * kCombR;
  const size_t stride = size_t(gridDim.x) * blockDim.x;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < N; i += stride) {
    double ar[kCombR], ai[kCombR];
#pragma unroll
    for (int t = 0; t < kCombR; ++t) ar[t] = ai[t] = 0.0;
    for (int q = 0; q < Q; ++q) {
      const cx<VR> v = (q < q0) ? b0[size_t(q) * N + i] : b1[size_t(q - q0) * N + i];
      const double vr = v.re, vi = v.im;
#pragma unroll
      for (int t = 0; t < kCombR; ++t) {
        const int r = r0 + t;
        if (r < R) {
          const double cr = coef[2 * (size_t(r) * Q + q)], ci = coef[2 * (size_t(r) * Q + q) + 1];
          ar[t] += cr * vr - ci * vi;
          ai[t] += cr * vi + ci * vr;
        }
      }
    }
#pragma unroll
    for (int t = 0; t < kCombR; ++t) {
      const int r = r0 + t;
      if (r < R) {
        cx<VR>* o = out + size_t(r) * N + i;
        if (accumulate) {
          const cx<VR> old = *o;
          *o = mk(VR(double(old.re) + ar[t]), VR(double(old.im) + ai[t]));
        } else {
          *o = mk(VR(ar[t]), VR(ai[t]));
        }
      }
    }
  }
}

// One output (R = 1): out (+)= sum_q coef_q basis_q with the basis split
// between the waves as in the update kernel (the general kernel above walks
// the basis one load at a time).
template <typename VR>
__global__ __launch_bounds__(256) void k_combine1(const cx<VR>* __restrict__ b0, int q0,
                                                  const cx<VR>* __restrict__ b1, int q1,
                                                  size_t N, const double* __restrict__ coef,
                                                  cx<VR>* __restrict__ out, int accumulate) {
  const int Q = q0 + q1;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __shared__ double part[kSplitWaves][kDotE][2][64];
  const size_t span = size_t(64) * kDotE;
  for (size_t base = size_t(blockIdx.x) * span; base < N; base += size_t(gridDim.x) * span) {
    size_t idx[kDotE];
    double sr[kDotE], si[kDotE];
    split_sums<VR, kAxpyG>(b0, q0, b1, N, Q, coef, base, lane, wave, idx, sr, si);
#pragma unroll
    for (int e = 0; e < kDotE; ++e) {
      part[wave][e][0][lane] = sr[e];
      part[wave][e][1][lane] = si[e];
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int e = 0; e < kDotE; ++e) {
        if (base + size_t(e) * 64 + lane < N) {
          double r = 0.0, im = 0.0;
          if (accumulate) {
            const cx<VR> old = out[idx[e]];
            r = old.re;
            im = old.im;
          }
#pragma unroll
          for (int v2 = 0; v2 < kSplitWaves; ++v2) {
            r += part[v2][e][0][lane];
            im += part[v2][e][1][lane];
          }
          out[idx[e]] = mk(VR(r), VR(im));
        }
      }
    }
    __syncthreads();
  }
}

template <typename VR>
__global__ void k_scale(const cx<VR>* __restrict__ in, cx<VR>* __restrict__ out, size_t N,
                        const double* __restrict__ sdev, double s, const int* __restrict__ done) {
  if (done && *done) return;
  const double sc = sdev ? *sdev : s;
  const size_t stride = size_t(gridDim.x) * blockDim.x;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < N; i += stride) {
    const cx<VR> z = in[i];
    out[i] = mk(VR(z.re * sc), VR(z.im * sc));
  }
}

template <typename VR>
__global__ void k_cscale(const cx<VR>* in, cx<VR>* out, size_t N, z64 c,
                         const int* __restrict__ done) {
  if (done && *done) return;
  const size_t stride = size_t(gridDim.x) * blockDim.x;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < N; i += stride) {
    const cx<VR> z = in[i];
    out[i] = mk(VR(c.re * double(z.re) - c.im * double(z.im)),
                VR(c.re * double(z.im) + c.im * double(z.re)));
  }
}

template <typename VR>
__global__ void k_scale_step(cx<VR>* v, size_t N, const double* __restrict__ inv_h,
                             const int* __restrict__ jdone, int j) {
  if (*jdone != j + 1) return;
  const double sc = *inv_h;
  const size_t stride = size_t(gridDim.x) * blockDim.x;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < N; i += stride) {
    const cx<VR> z = v[i];
    v[i] = mk(VR(double(z.re) * sc), VR(double(z.im) * sc));
  }
}

template <typename VR>
__global__ void k_zero(cx<VR>* x, size_t N) {
  const size_t stride = size_t(gridDim.x) * blockDim.x;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < N; i += stride)
    x[i] = mk(VR(0), VR(0));
}

template <typename VR>
__global__ void k_axpy(z64 a, const cx<VR>* __restrict__ x, cx<VR>* __restrict__ y, size_t N) {
  const size_t stride = size_t(gridDim.x) * blockDim.x;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < N; i += stride) {
    const cx<VR> xv = x[i];
    cx<VR> yv = y[i];
    yv.re = VR(double(yv.re) + a.re * double(xv.re) - a.im * double(xv.im));
    yv.im = VR(double(yv.im) + a.re * double(xv.im) + a.im * double(xv.re));
    y[i] = yv;
  }
}

template <typename VR>
__global__ __launch_bounds__(256) void k_norm2(const cx<VR>* __restrict__ x, size_t N,
                                               Reducer red) {
  // column blockIdx.y of [q][N]; partial of block (bx, by) at by * gx + bx
  const cx<VR>* col = x + size_t(blockIdx.y) * N;
  double acc[1] = {0.0};
  const size_t stride = size_t(gridDim.x) * blockDim.x;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < N; i += stride) {
    const cx<VR> z = col[i];
    acc[0] += double(z.re) * double(z.re) + double(z.im) * double(z.im);
  }
  block_partials<1>(acc, red.partials);
}

template <typename VR>
__global__ void k_gamma5(const cx<VR>* in, cx<VR>* out, size_t N, int n) {
  const size_t stride = size_t(gridDim.x) * blockDim.x;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < N; i += stride) {
    const int c = int(i % n);
    const cx<VR> z = in[i];
    out[i] = (c < (n >> 1)) ? z : mk(VR(-z.re), VR(-z.im));
  }
}

__global__ void k_cvt64to32(const z64* __restrict__ in, z32* __restrict__ out, size_t N, int n,
                            int g5) {
  const size_t stride = size_t(gridDim.x) * blockDim.x;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < N; i += stride) {
    const z64 z = in[i];
    const double s = (g5 && int(i % n) >= (n >> 1)) ? -1.0 : 1.0;
    out[i] = mk(float(s * z.re), float(s * z.im));
  }
}

__global__ void k_cvt32to64(const z32* __restrict__ in, z64* __restrict__ out, size_t N, int n,
                            int g5) {
  const size_t stride = size_t(gridDim.x) * blockDim.x;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < N; i += stride) {
    const z32 z = in[i];
    const double s = (g5 && int(i % n) >= (n >> 1)) ? -1.0 : 1.0;
    out[i] = mk(s * double(z.re), s * double(z.im));
  }
}

// Philox4x32-10 (Salmon et al., SC'11) and Box-Muller, as in the input generator.
__device__ void philox(uint32_t c[4], uint32_t k0, uint32_t k1) {
  for (int r = 0; r < 10; ++r) {
    const uint32_t hi0 = __umulhi(0xD2511F53u, c[0]), lo0 = 0xD2511F53u * c[0];
    const uint32_t hi1 = __umulhi(0xCD9E8D57u, c[2]), lo1 = 0xCD9E8D57u * c[2];
    const uint32_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
    c[0] = n0;
    c[1] = lo1;
    c[2] = n2;
    c[3] = lo0;
    if (r < 9) {
      k0 += 0x9E3779B9u;
      k1 += 0xBB67AE85u;
    }
  }
}

__global__ void k_gaussian(z64* out, size_t N, uint64_t seed, uint32_t stream_id) {
  const size_t stride = size_t(gridDim.x) * blockDim.x;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < N; i += stride) {
    uint32_t c[4] = {uint32_t(i), uint32_t(uint64_t(i) >> 32), stream_id, 0u};
    philox(c, uint32_t(seed), uint32_t(seed >> 32));
    const double two53 = 9007199254740992.0;
    const double u1 = (double(uint64_t(c[0] >> 5) * 67108864ull + (c[1] >> 6)) + 0.5) / two53;
    const double u2 = (double(uint64_t(c[2] >> 5) * 67108864ull + (c[3] >> 6)) + 0.5) / two53;
    const double r = sqrt(-2.0 * log(u1)) * 0.70710678118654752440;
    double sn, cs;
    sincos(6.283185307179586477 * u2, &sn, &cs);
    out[i] = mk(r * cs, r * sn);
  }
}

// ------------------------------------------------------------------ block products
// The tall-skinny complex products of block GMRES (one Krylov space shared by
// many right-hand sides) and of the recycle-space construction and refresh:
// Gram matrices A^H B of two blocks of vectors and block updates
// C = beta C + alpha A S with a small coefficient matrix S.  Both stage
// 64-wide panels in LDS as real and imaginary planes with a padded stride and
// multiply on 16x16x4 MFMA tiles with three real products per complex one;
// wave w owns output row tile w and all four column tiles of a 64 x 64 output
// tile.  VS is the storage type of the vectors, VC the type the products are
// formed and accumulated in (FP32 vectors may be combined in FP64).
constexpr int kBpT = 64;          // output tile edge
constexpr int kBpK = 32;          // inner-dimension rows staged per LDS round
constexpr int kBpLD = kBpK + 1;   // padded plane stride
constexpr int kGramMaxParts = 256;

// part[c] = A_c^H B_c for row chunk c = blockIdx.x (rows [c L, min(c L + L, N))),
// output tile (blockIdx.y % tq, blockIdx.y / tq) of the qa x rb result, tq =
// ceil(qa / 64); part layout [chunk][j qa + i].  A: qa vectors, B: rb vectors,
// each N long with stride N.
template <typename VS, typename VC>
__global__ __launch_bounds__(256) void k_block_gram(const cx<VS>* __restrict__ A, int qa,
                                                     const cx<VS>* __restrict__ B, int rb,
                                                     size_t N, size_t L,
                                                     cx<VC>* __restrict__ part) {
  using acc_t = typename Mfma<VC>::acc_t;
  __shared__ VC Ar[kBpT * kBpLD], Ai[kBpT * kBpLD], Br[kBpT * kBpLD], Bi[kBpT * kBpLD];
  const int tq = (qa + kBpT - 1) / kBpT;
  const int i0 = int(blockIdx.y % unsigned(tq)) * kBpT, j0 = int(blockIdx.y / unsigned(tq)) * kBpT;
  const int ni = min(kBpT, qa - i0), nj = min(kBpT, rb - j0);
  const size_t r0 = size_t(blockIdx.x) * L, r1 = min(N, r0 + L);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int l16 = lane & 15, lk = lane >> 4;
  const int nct = (nj + 15) / 16;    // column tiles with at least one column
  acc_t prr[4], pii[4], pss[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    prr[t] = acc_t{0, 0, 0, 0};
    pii[t] = acc_t{0, 0, 0, 0};
    pss[t] = acc_t{0, 0, 0, 0};
  }
  // panels: column c of the tile, rows k0 .. k0 + 31 (consecutive threads
  // read consecutive rows of one vector); thread t holds elements
  // u = t + 256 e, e < 8, of each panel in registers: those of the next round
  // are loaded while the current one multiplies
  constexpr int EPT = kBpT * kBpK / 256;
  cx<VS> ra[EPT], rb_[EPT];
  auto fetch = [&](size_t k0) {
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const int u = int(threadIdx.x) + 256 * e;
      const int c = u / kBpK, r = u % kBpK;
      const size_t row = k0 + size_t(r);
      ra[e] = mk(VS(0), VS(0));
      rb_[e] = mk(VS(0), VS(0));
      if (row < r1) {
        if (c < ni) ra[e] = A[size_t(i0 + c) * N + row];
        if (c < nj) rb_[e] = B[size_t(j0 + c) * N + row];
      }
    }
  };
  if (r0 < r1) fetch(r0);
  for (size_t k0 = r0; k0 < r1; k0 += kBpK) {
#pragma unroll
    for (int e = 0; e < EPT; ++e) {   // A is conjugated here
      const int u = int(threadIdx.x) + 256 * e;
      const int c = u / kBpK, r = u % kBpK;
      Ar[c * kBpLD + r] = VC(ra[e].re);
      Ai[c * kBpLD + r] = -VC(ra[e].im);
      Br[c * kBpLD + r] = VC(rb_[e].re);
      Bi[c * kBpLD + r] = VC(rb_[e].im);
    }
    __syncthreads();
    if (k0 + kBpK < r1) fetch(k0 + kBpK);
    if (wave * 16 < ni) {
#pragma unroll 2
      for (int kk = 0; kk < kBpK; kk += 4) {
        const int ao = (wave * 16 + l16) * kBpLD + kk + lk;
        const VC a_r = Ar[ao], a_i = Ai[ao];
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) {
          if (ct < nct) {
            const int bo = (ct * 16 + l16) * kBpLD + kk + lk;
            const VC b_r = Br[bo], b_i = Bi[bo];
            prr[ct] = Mfma<VC>::mma(a_r, b_r, prr[ct]);
            pii[ct] = Mfma<VC>::mma(a_i, b_i, pii[ct]);
            pss[ct] = Mfma<VC>::mma(a_r + a_i, b_r + b_i, pss[ct]);
          }
        }
      }
    }
    __syncthreads();
  }
  const size_t qr = size_t(qa) * size_t(rb);
  cx<VC>* out = part + size_t(blockIdx.x) * qr;
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) {
    const int j = ct * 16 + l16;
    if (ct >= nct || j >= nj) continue;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = wave * 16 + Mfma<VC>::row(lk, q);
      if (i < ni)
        out[size_t(j0 + j) * qa + (i0 + i)] =
            mk(VC(prr[ct][q] - pii[ct][q]), VC(pss[ct][q] - prr[ct][q] - pii[ct][q]));
    }
  }
}

// out[e] = sum over the P chunks of part[c][e] (FP64, chunk order fixed)
template <typename VC>
__global__ void k_block_gram_sum(const cx<VC>* __restrict__ part, int P, size_t qr,
                                 z64* __restrict__ out) {
  const size_t e = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= qr) return;
  double re = 0.0, im = 0.0;
  for (int c = 0; c < P; ++c) {
    const cx<VC> z = part[size_t(c) * qr + e];
    re += double(z.re);
    im += double(z.im);
  }
  out[e] = mk(re, im);
}

// C[:, j] = beta C[:, j] + alpha sum_i A_i S[i + j ldS] for j < r, over the
// k = q0 + q1 vectors A_i = b0 + i N (i < q0), b1 + (i - q0) N (after); C has r
// vectors (each N long, stride N); S is column-major in the product type.
// Workgroup t: column tile t % nct (nct = ceil(r / 64)), rows 64 (t / nct)
// .. + 63, so the workgroups that share a row panel of the A_i run together.
// C must not overlap the A_i.
template <typename VS, typename VC>
__global__ __launch_bounds__(256) void k_block_update(const cx<VS>* __restrict__ b0, int q0,
                                                       const cx<VS>* __restrict__ b1, int q1,
                                                       const cx<VC>* __restrict__ S, int ldS,
                                                       cx<VS>* C, int r, size_t N, z64 alpha,
                                                       z64 beta) {
  using acc_t = typename Mfma<VC>::acc_t;
  // four planes while multiplying ([row][kk] of A, [col][kk] of S); the
  // 64 x 64 output planes ([col][row], stride 65) reuse them afterwards
  constexpr int PL = kBpT * kBpLD;
  __shared__ VC sm[4 * PL];
  static_assert(2 * kBpT * (kBpT + 1) <= 4 * PL, "output planes fit");
  VC* Ar = sm;
  VC* Ai = sm + PL;
  VC* Sr = sm + 2 * PL;
  VC* Si = sm + 3 * PL;
  const int k = q0 + q1;
  const int nctile = (r + kBpT - 1) / kBpT;
  const size_t row0 = size_t(blockIdx.x / unsigned(nctile)) * kBpT;
  const int j0 = int(blockIdx.x % unsigned(nctile)) * kBpT;
  const int nj = min(kBpT, r - j0);
  const int nrow = int(min(size_t(kBpT), N - row0));
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int l16 = lane & 15, lk = lane >> 4;
  const int nct = (nj + 15) / 16;
  acc_t prr[4], pii[4], pss[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    prr[t] = acc_t{0, 0, 0, 0};
    pii[t] = acc_t{0, 0, 0, 0};
    pss[t] = acc_t{0, 0, 0, 0};
  }
  // A panel: vector k0 + kk, rows row0 .. row0 + 63 (consecutive threads,
  // consecutive rows); S panel: column j, rows k0 .. k0 + 31.  Thread t holds
  // elements u = t + 256 e of each in registers; the next round's are loaded
  // while the current one multiplies.
  constexpr int EPT = kBpT * kBpK / 256;
  cx<VS> ra[EPT];
  cx<VC> rs[EPT];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const int u = int(threadIdx.x) + 256 * e;
      const int kk = u / kBpT, rr = u % kBpT;
      const int i = k0 + kk;
      ra[e] = mk(VS(0), VS(0));
      if (i < k && rr < nrow)
        ra[e] = (i < q0 ? b0 + size_t(i) * N : b1 + size_t(i - q0) * N)[row0 + rr];
      const int j = u / kBpK, kq = u % kBpK;
      rs[e] = mk(VC(0), VC(0));
      if (j < nj && k0 + kq < k) rs[e] = S[size_t(j0 + j) * ldS + k0 + kq];
    }
  };
  if (k > 0) fetch(0);
  for (int k0 = 0; k0 < k; k0 += kBpK) {
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const int u = int(threadIdx.x) + 256 * e;
      const int kk = u / kBpT, rr = u % kBpT;
      Ar[rr * kBpLD + kk] = VC(ra[e].re);
      Ai[rr * kBpLD + kk] = VC(ra[e].im);
      const int j = u / kBpK, kq = u % kBpK;
      Sr[j * kBpLD + kq] = rs[e].re;
      Si[j * kBpLD + kq] = rs[e].im;
    }
    __syncthreads();
    if (k0 + kBpK < k) fetch(k0 + kBpK);
#pragma unroll 2
    for (int kk = 0; kk < kBpK; kk += 4) {
      const int ao = (wave * 16 + l16) * kBpLD + kk + lk;
      const VC a_r = Ar[ao], a_i = Ai[ao];
#pragma unroll
      for (int ct = 0; ct < 4; ++ct) {
        if (ct < nct) {
          const int bo = (ct * 16 + l16) * kBpLD + kk + lk;
          const VC b_r = Sr[bo], b_i = Si[bo];
          prr[ct] = Mfma<VC>::mma(a_r, b_r, prr[ct]);
          pii[ct] = Mfma<VC>::mma(a_i, b_i, pii[ct]);
          pss[ct] = Mfma<VC>::mma(a_r + a_i, b_r + b_i, pss[ct]);
        }
      }
    }
    __syncthreads();
  }
  // accumulators -> output planes [col][row] -> coalesced column stores
  constexpr int OL = kBpT + 1;
  VC* Or = sm;
  VC* Oi = sm + kBpT * OL;
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) {
    if (ct >= nct) continue;
    const int col = ct * 16 + l16;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int row = wave * 16 + Mfma<VC>::row(lk, q);
      Or[col * OL + row] = prr[ct][q] - pii[ct][q];
      Oi[col * OL + row] = pss[ct][q] - prr[ct][q] - pii[ct][q];
    }
  }
  __syncthreads();
  const bool keep = beta.re != 0.0 || beta.im != 0.0;
  for (int u = threadIdx.x; u < kBpT * kBpT; u += 256) {
    const int col = u / kBpT, rr = u % kBpT;
    if (col >= nj || rr >= nrow) continue;
    const double pr = double(Or[col * OL + rr]), pi = double(Oi[col * OL + rr]);
    double yr = alpha.re * pr - alpha.im * pi, yi = alpha.re * pi + alpha.im * pr;
    cx<VS>* c = C + size_t(j0 + col) * N + row0 + rr;
    if (keep) {
      const cx<VS> z = *c;
      yr += beta.re * double(z.re) - beta.im * double(z.im);
      yi += beta.re * double(z.im) + beta.im * double(z.re);
    }
    *c = mk(VS(yr), VS(yi));
  }
}

// ------------------------------------------------------------------ Arnoldi
__global__ void k_arnoldi_init(ArnoldiDev a, double beta, const double* __restrict__ beta_dev) {
  if (threadIdx.x == 0) {
    if (beta_dev) beta = *beta_dev;
    *a.done = 0;
    *a.jdone = 0;
    if (a.go) *a.go = 0;
    *a.brk_flag = 0;
    *a.est = beta;
    double* g = a.giv;
    for (int i = 0; i < 2 * (a.ldh + 1); ++i) g[i] = 0.0;
    g[0] = beta;
  }
}

// Givens storage in a.giv: g[0..ldh] (complex), then c[0..ldh) (real, stored
// in the even slots of complex entries), then s[0..ldh) (complex).
constexpr int kFinishLds = 512;  // Hessenberg column length staged in LDS

// Coefficients of the two passes and the norm of the new vector, as the first 64
// threads of a workgroup see them; every lane returns the same value.
// nrm2 given: h_{j+1,j}^2 = *nrm2.  Without it, single-sync process (c2 null,
// Sec. 3.5): the coefficients come from one pass and h^2 = ||A v_j||^2 - sum |c1|^2;
// a value at or below (brk ||A v_j||)^2 is a breakdown.  Two passes without nrm2: c2
// carries ||w||^2 of the vector after the first pass, h^2 = ||w||^2 - sum |c2|^2.
// The difference is the norm of the final vector but for d sum |c2|^2, d the basis's
// distance from orthonormality, and c2 itself is about d ||A v_j||: relative to h^2 at
// most d (d / brk)^2 above the breakdown threshold.  Measured, recycle space included, d
// is below 2e-7 in FP32 (brk 1e-6) and 4e-14 in FP64 (1e-14): below 1e-8 and 1e-12.  Where
// h is larger the difference keeps the precision of its terms.
struct StepNorm {
  double h;   // 0 for a breakdown
  bool breakdown;
};
__device__ __forceinline__ StepNorm step_norm(const double* c1, const double* c2,
                                              const double* nrm2, int Q, double brk) {
  const double wn2 = c1[2 * Q];   // ||A v_j||^2 before orthogonalisation
  const double* c = c2 ? c2 : c1;
  double sq = 0.0;
  if (!nrm2) {
    for (int i = int(threadIdx.x); i < 2 * Q; i += 64) sq += c[i] * c[i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sq += shfl_xor(sq, o);
  }
  StepNorm r;
  if (!c2) {
    const double t = wn2 - sq;
    r.breakdown = !(t > brk * brk * wn2);
    r.h = r.breakdown ? 0.0 : sqrt(t);
  } else {
    const double h = sqrt(fmax(nrm2 ? *nrm2 : c2[2 * Q] - sq, 0.0));
    r.breakdown = !(h > brk * sqrt(fmax(wn2, 0.0)));
    r.h = r.breakdown ? 0.0 : h;
  }
  return r;
}

// The bookkeeping of Arnoldi step j: the first 64 threads of one workgroup combine
// the passes' coefficients in parallel and stage the new column and the stored
// rotations in LDS; thread 0 then runs the (inherently serial) Givens update.
__device__ __forceinline__ void arnoldi_finish_body(const ArnoldiDev& a, int steps, int kC, int j,
                                                    const double* c1, const double* c2,
                                                    const StepNorm& nm, double target) {
  if (*a.done) return;
  const int tid = threadIdx.x < 64 ? int(threadIdx.x) : 1 << 30;
  __shared__ double hcol[2 * (kFinishLds + 2)], csl[kFinishLds], snl[2 * kFinishLds];
  const bool staged = j + 2 <= kFinishLds;
  double* Hc = a.H + 2 * size_t(j) * a.ldh;
  double* g = a.giv;
  double* cs = a.giv + 2 * (a.ldh + 1);
  double* sn = cs + 2 * a.ldh;
  const bool ss = (c2 == nullptr);
  for (int i = tid; i < kC; i += 64) {
    a.Bk[2 * (size_t(j) * a.ldb + i)] = c1[2 * i] + (ss ? 0.0 : c2[2 * i]);
    a.Bk[2 * (size_t(j) * a.ldb + i) + 1] = c1[2 * i + 1] + (ss ? 0.0 : c2[2 * i + 1]);
  }
  for (int i = tid; i <= j; i += 64) {
    const double hr = c1[2 * (kC + i)] + (ss ? 0.0 : c2[2 * (kC + i)]);
    const double hi = c1[2 * (kC + i) + 1] + (ss ? 0.0 : c2[2 * (kC + i) + 1]);
    Hc[2 * i] = hr;
    Hc[2 * i + 1] = hi;
    if (staged) {
      hcol[2 * i] = hr;
      hcol[2 * i + 1] = hi;
    }
  }
  if (staged)
    for (int i = tid; i < j; i += 64) {
      csl[i] = cs[2 * i];
      snl[2 * i] = sn[2 * i];
      snl[2 * i + 1] = sn[2 * i + 1];
    }
  __syncthreads();
  if (threadIdx.x != 0) return;
  const double* hsrc = staged ? hcol : Hc;
  const bool breakdown = nm.breakdown;
  const double hh = nm.h;
  Hc[2 * (j + 1)] = hh;
  Hc[2 * (j + 1) + 1] = 0.0;
  *a.inv_h = breakdown ? 0.0 : 1.0 / hh;
  // carry the running entry through the previous rotations:
  // [h_i; h_{i+1}] <- [[c_i, s_i], [-conj(s_i), c_i]] [h_i; h_{i+1}]
  double xr = hsrc[0], xi = hsrc[1];
  for (int i = 0; i < j; ++i) {
    const double c = staged ? csl[i] : cs[2 * i];
    const double sr = staged ? snl[2 * i] : sn[2 * i];
    const double si = staged ? snl[2 * i + 1] : sn[2 * i + 1];
    const double yr = hsrc[2 * (i + 1)], yi = hsrc[2 * (i + 1) + 1];
    const double nyr = -(sr * xr + si * xi) + c * yr;
    const double nyi = -(sr * xi - si * xr) + c * yi;
    xr = nyr;
    xi = nyi;
  }
  const double ax = sqrt(xr * xr + xi * xi);
  double c, sr, si;
  if (hh == 0.0) {
    c = 1.0;
    sr = si = 0.0;
  } else if (ax == 0.0) {
    c = 0.0;
    sr = 1.0;
    si = 0.0;
  } else {
    const double r = sqrt(ax * ax + hh * hh);
    c = ax / r;
    sr = (xr / ax) * hh / r;  // s = (x/|x|) h / r
    si = (xi / ax) * hh / r;
  }
  cs[2 * j] = c;
  cs[2 * j + 1] = 0.0;
  sn[2 * j] = sr;
  sn[2 * j + 1] = si;
  const double gr = g[2 * j], gi = g[2 * j + 1];
  g[2 * j] = c * gr;
  g[2 * j + 1] = c * gi;
  g[2 * (j + 1)] = -(sr * gr + si * gi);  // -conj(s) g_j
  g[2 * (j + 1) + 1] = -(sr * gi - si * gr);
  const double est = sqrt(g[2 * (j + 1)] * g[2 * (j + 1)] + g[2 * (j + 1) + 1] * g[2 * (j + 1) + 1]);
  *a.est = est;
  if (a.hest) a.hest[j] = est;
  *a.jdone = j + 1;
  if (breakdown) *a.brk_flag = 1;
  if (a.target_dev) target = *a.target_dev;
  if (breakdown || est <= target || j + 1 >= steps) {
    *a.done = 1;
    if (a.hdone) *a.hdone = 1;
  }
}

__global__ __launch_bounds__(64) void k_arnoldi_finish(ArnoldiDev a, int steps, int kC, int j,
                                                       const double* c1, const double* c2,
                                                       const double* nrm2, double target,
                                                       double brk) {
  arnoldi_finish_body(a, steps, kC, j, c1, c2, step_norm(c1, c2, nrm2, kC + j + 1, brk), target);
}

// ------------------------------------------------------------------ Gram-Schmidt, single column
// A step's kernels are small next to the launches between them, so each kernel
// sums the reduction partials of the one before by itself (every workgroup the
// same, from L2), the second pass's coefficients and the norm come out of the
// kernel that applies the first's, and one extra workgroup of the last kernel
// does the bookkeeping beside the update.  Three launches per step where separate
// passes take nine, three passes over the basis where they take four, and none for
// the norm and the scaling: 30 steps on 8^4 (FP64, n = 48) 6.85 -> 6.27 ms, of them
// 4.7 ms in the operator's applies (5.55 ms with 4.2 ms of applies since); an odd-even
// GCRO-DR solve on 4^4, n = 16, 6.6 -> 4.8 ms; 120 steps on 16^4, n = 16 140.8 -> 127.9
// ms.  Finishing the reductions in the last workgroup to arrive was slower (7.3 and
// 5.1 ms): its fences write back and invalidate each die's L2.

constexpr int kFoldQ = 64;        // vectors of the basis that k_update_dot holds in registers
// Partials per value that the next kernel sums itself; more are summed by a launch of
// their own.  Every workgroup reads all of them, so the line lies where that read
// costs what the launch does: with a basis of 30 in FP64 the folded sums of 32
// partials save 0.4 of 5.4 ms of a 4^4 solve, those of 192 partials cost 0.1 of
// 36.2 ms of an 8^4 one.
constexpr int kFoldParts = 64;

// result[v] = sum over b of partials[v * nparts + b] for v < nvals: eight lanes per
// value, 256 threads.
__device__ __forceinline__ void sum_partials(const double* __restrict__ partials, int nvals,
                                             int nparts, double* result) {
  const int l = threadIdx.x & 7;
  for (int v = int(threadIdx.x >> 3); v < nvals; v += 32) {
    const double* p = partials + size_t(v) * nparts;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    int b = l;
    for (; b + 24 < nparts; b += 32) {
#pragma unroll
      for (int u = 0; u < 4; ++u) s[u] += p[b + 8 * u];
    }
    for (; b < nparts; b += 8) s[0] += p[b];
    double t = (s[0] + s[1]) + (s[2] + s[3]);
#pragma unroll
    for (int o = 4; o > 0; o >>= 1) t += shfl_xor(t, o);
    if (l == 0) result[v] = t;
  }
}

// w -= [b0 b1] c1, then the partials of [b0 b1]^H w and ||w||^2 of the updated w, for a
// basis of Q <= kFoldQ vectors read once: wave v of a workgroup holds vectors 16 v ..
// 16 v + 15 of a tile of 64 entries, the waves' shares of the update meet in LDS,
// and each wave forms its own products with the updated tile from the same
// registers.  Accumulators stay in registers over the workgroup's tiles.  FOLD: c1
// comes as nparts partials per value and is kept in res1 for the bookkeeping.
template <typename VR, bool FOLD>
__global__ __launch_bounds__(256) void k_update_dot(const cx<VR>* __restrict__ b0, int q0,
                                                    const cx<VR>* __restrict__ b1, int q1,
                                                    size_t N, cx<VR>* w,
                                                    const double* __restrict__ parts, int nparts,
                                                    double* __restrict__ res1,
                                                    double* __restrict__ out,
                                                    const int* __restrict__ done) {
  constexpr int G = 16;
  if (done && *done) return;
  const int Q = q0 + q1, nvals = 2 * Q + 1;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));   // uniform basis addresses
  __shared__ double part[2][4][2][64];
  __shared__ double sums[4 * 2 * G + 1];
  if constexpr (FOLD) {
    sum_partials(parts, nvals, nparts, sums);
    __syncthreads();
    if (blockIdx.x == 0)
      for (int u = threadIdx.x; u < nvals; u += 256) res1[u] = sums[u];
  }
  const bool mine = wave * G < Q;
  double acc[2 * G], nacc = 0.0;
#pragma unroll
  for (int t = 0; t < 2 * G; ++t) acc[t] = 0.0;
  int ph = 0;
  for (size_t base = size_t(blockIdx.x) * 64; base < N; base += size_t(gridDim.x) * 64, ph ^= 1) {
    const bool in = base + lane < N;
    const size_t i = in ? base + lane : N - 1;
    cx<VR> v[G];
    const cx<VR> wv = w[i];
    double sr = 0.0, si = 0.0;
    if (mine) {
#pragma unroll
      for (int t = 0; t < G; ++t) v[t] = basis_ptr(b0, q0, b1, N, min(wave * G + t, Q - 1))[i];
      __builtin_amdgcn_sched_barrier(0);   // keep every load ahead of the arithmetic
#pragma unroll
      for (int t = 0; t < G; ++t) {
        const int q = wave * G + t;
        double cr = 0.0, ci = 0.0;
        if (q < Q) {
          cr = FOLD ? sums[2 * q] : res1[2 * q];
          ci = FOLD ? sums[2 * q + 1] : res1[2 * q + 1];
        }
        const double vr = v[t].re, vi = v[t].im;
        sr = fma(cr, vr, fma(-ci, vi, sr));
        si = fma(cr, vi, fma(ci, vr, si));
      }
    }
    part[ph][wave][0][lane] = sr;
    part[ph][wave][1][lane] = si;
    __syncthreads();
    double r = wv.re, im = wv.im;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      r -= part[ph][u][0][lane];
      im -= part[ph][u][1][lane];
    }
    const cx<VR> o = mk(VR(r), VR(im));
    const double orr = in ? double(o.re) : 0.0, oi = in ? double(o.im) : 0.0;
    if (wave == 0) {
      if (in) w[i] = o;
      nacc += orr * orr + oi * oi;
    }
    if (mine) {
#pragma unroll
      for (int t = 0; t < G; ++t) {
        const double vr = v[t].re, vi = v[t].im;
        acc[2 * t] = fma(vr, orr, fma(vi, oi, acc[2 * t]));            // Re conj(v) w
        acc[2 * t + 1] = fma(vr, oi, fma(-vi, orr, acc[2 * t + 1]));   // Im conj(v) w
      }
    }
  }
  __syncthreads();   // the coefficients in sums have been read
  if (mine) {
    const double s = wave_sum_many<2 * G>(acc, lane);
    if ((lane & 1) == 0) sums[wave * 2 * G + (lane >> 1)] = s;
  }
  if (wave == 0) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) nacc += shfl_xor(nacc, o);
    if (lane == 0) sums[4 * 2 * G] = nacc;
  }
  __syncthreads();
  for (int u = threadIdx.x; u < nvals; u += 256)
    out[size_t(u) * gridDim.x + blockIdx.x] = sums[u < 2 * Q ? u : 4 * 2 * G];
}

// Bookkeeping of Arnoldi step j.
struct StepEnd {
  ArnoldiDev a;
  const double* c1;   // the first pass's coefficients and ||A v_j||^2; null: single-sync
  double target, brk;
  int steps, kC, j;
};

// w = (w - [b0 b1] c) / h_{j+1,j} with the last pass's coefficients c (FOLD: nparts
// partials per value at src, else at src itself), for the step whose first kernel
// set the flag; workgroup 0 runs the step's bookkeeping meanwhile.
// G: vectors per chunk of the split update (0: the flat one).
template <typename VR, int G, bool FOLD>
__global__ __launch_bounds__(256) void k_step_end(cx<VR>* w, const cx<VR>* __restrict__ b0, int q0,
                                                  const cx<VR>* __restrict__ b1, int q1, size_t N,
                                                  const double* __restrict__ src, int nparts,
                                                  StepEnd e) {
  if (*e.a.go != e.j + 1) return;
  const int Q = q0 + q1;
  __shared__ double cf[2 * kFoldQ + 1];
  __shared__ double inv;
  if constexpr (FOLD) {
    sum_partials(src, 2 * Q + 1, nparts, cf);
    __syncthreads();
  }
  const double* c = FOLD ? cf : src;
  StepNorm nm{};
  if (threadIdx.x < 64) {
    nm = step_norm(e.c1 ? e.c1 : c, e.c1 ? c : nullptr, nullptr, Q, e.brk);
    if (threadIdx.x == 0) inv = nm.breakdown ? 0.0 : 1.0 / nm.h;
  }
  if (blockIdx.x == 0) {
    arnoldi_finish_body(e.a, e.steps, e.kC, e.j, e.c1 ? e.c1 : c, e.c1 ? c : nullptr, nm, e.target);
    return;
  }
  __syncthreads();
  const int bx = int(blockIdx.x) - 1, gx = int(gridDim.x) - 1;
  if constexpr (G != 0)
    multiaxpy_split_body<VR, G>(w, w, b0, q0, b1, q1, N, FOLD ? cf : src, 0, nullptr, inv, bx, gx);
  else
    multiaxpy_flat_body<VR>(w, w, b0, q0, b1, q1, N, FOLD ? cf : src, 0, nullptr, inv, bx, gx);
}

// ------------------------------------------------------------------ batched Gram-Schmidt
// The launches of one classical Gram-Schmidt step for up to kOrthCols
// independent columns (a lockstep batch) at once: blockIdx.z is the column,
// and each column runs exactly the blocks, partial layout and sums of its own
// single launch (its grid extent gx; the launch covers the largest), so its
// results are those of the per-column launches bit for bit.
template <typename VR, int G>
__global__ __launch_bounds__(256) void k_multidot_cols(OrthCols t) {
  if (int(blockIdx.z) >= t.count) return;
  const OrthCol& a = t.c[blockIdx.z];
  if (a.done && *a.done) return;
  if (blockIdx.x >= a.gx) return;
  multidot_body<VR, G>(static_cast<const cx<VR>*>(a.b0), a.q0, static_cast<const cx<VR>*>(a.b1),
                       a.q1, a.N, static_cast<const cx<VR>*>(a.w), a.partials, int(blockIdx.x),
                       int(a.gx), int(blockIdx.y));
}

__global__ __launch_bounds__(64) void k_finalize_cols(OrthCols t) {
  if (int(blockIdx.z) >= t.count) return;
  const OrthCol& a = t.c[blockIdx.z];
  if (a.done && *a.done) return;
  finalize_value(a.partials, int(a.gx), a.result, int(blockIdx.x));
}

template <typename VR, bool SPLIT>
__global__ __launch_bounds__(256) void k_multiaxpy_cols(OrthCols t, int want_norm) {
  if (int(blockIdx.z) >= t.count) return;
  const OrthCol& a = t.c[blockIdx.z];
  if (a.done && *a.done) return;
  if (blockIdx.x >= a.gx) return;
  cx<VR>* w = static_cast<cx<VR>*>(a.w);
  const cx<VR>* b0 = static_cast<const cx<VR>*>(a.b0);
  const cx<VR>* b1 = static_cast<const cx<VR>*>(a.b1);
  if constexpr (SPLIT)
    multiaxpy_split_body<VR>(w, w, b0, a.q0, b1, a.q1, a.N, a.coef, want_norm, a.partials, 1.0,
                             int(blockIdx.x), int(a.gx));
  else
    multiaxpy_flat_body<VR>(w, w, b0, a.q0, b1, a.q1, a.N, a.coef, want_norm, a.partials, 1.0,
                            int(blockIdx.x), int(a.gx));
}

__global__ __launch_bounds__(64) void k_arnoldi_finish_cols(FinishCols t, int steps, int j,
                                                            double brk) {
  if (int(blockIdx.x) >= t.count) return;
  const FinishCol& f = t.c[blockIdx.x];
  arnoldi_finish_body(f.a, steps, f.kC, j, f.c1, f.c2,
                      step_norm(f.c1, f.c2, f.nrm2, f.kC + j + 1, brk), f.target);
}

template <typename VR>
__global__ void k_scale_step_cols(ScaleCols t, int j) {
  if (int(blockIdx.z) >= t.count) return;
  const int c = int(blockIdx.z);
  if (*t.jdone[c] != j + 1) return;
  const double sc = *t.inv_h[c];
  cx<VR>* v = static_cast<cx<VR>*>(t.v[c]);
  const size_t N = t.N[c];
  const size_t stride = size_t(gridDim.x) * blockDim.x;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < N; i += stride) {
    const cx<VR> z = v[i];
    v[i] = mk(VR(double(z.re) * sc), VR(double(z.im) * sc));
  }
}

}  // namespace

// ====================================================================== launchers

void launch_finalize(const double* partials, int nvals, int nparts, double* result,
                     const int* done, hipStream_t st) {
  hipLaunchKernelGGL(k_finalize, dim3(unsigned(nvals)), dim3(64), 0, st, partials, nparts, result,
                     done);
  DC_HIP(hipGetLastError());
}

// blocks per dot group: about one pass per thread, bounded by the partials
// capacity over all groups and values
static unsigned dot_blocks(size_t N, int values) {
  size_t b = (N + 256 * kDotE - 1) / (256 * kDotE);
  const size_t cap = size_t(kRedCap) / size_t(values > 0 ? values : 1);
  if (b > cap) b = cap;
  if (b > 1024) b = 1024;
  if (b < 1) b = 1;
  return unsigned(b);
}

template <typename VR, int G>
static void multidot_g(const void* b0, int q0, const void* b1, int q1, size_t N, const void* w,
                       Reducer red, const int* done, int Q, hipStream_t st, unsigned* gx_out,
                       int* go, int step) {
  const int gy = (Q + G - 1) / G;
  const unsigned gx = dot_blocks(N, gy * 2 * G);
  hipLaunchKernelGGL((k_multidot<VR, G>), dim3(gx, unsigned(gy)), dim3(256), 0, st,
                     static_cast<const cx<VR>*>(b0), q0, static_cast<const cx<VR>*>(b1), q1, N,
                     static_cast<const cx<VR>*>(w), red, done, go, step);
  *gx_out = gx;
}

template <typename VR>
static unsigned multidot_t(const void* b0, int q0, const void* b1, int q1, size_t N,
                           const void* w, Reducer red, const int* done, int Q, hipStream_t st,
                           int* go = nullptr, int step = 0) {
  unsigned gx = 0;
  if (Q <= 2) multidot_g<VR, 2>(b0, q0, b1, q1, N, w, red, done, Q, st, &gx, go, step);
  else if (Q <= 4) multidot_g<VR, 4>(b0, q0, b1, q1, N, w, red, done, Q, st, &gx, go, step);
  else if (Q <= 8) multidot_g<VR, 8>(b0, q0, b1, q1, N, w, red, done, Q, st, &gx, go, step);
  else multidot_g<VR, 16>(b0, q0, b1, q1, N, w, red, done, Q, st, &gx, go, step);
  return gx;
}

void launch_multidot(Prec p, const void* b0, int q0, const void* b1, int q1, size_t N,
                     const void* w, int want_norm, Reducer red, double* result, const int* done,
                     hipStream_t st) {
  const int Q = q0 + q1 + (want_norm ? 1 : 0);
  if (Q == 0) return;
  const unsigned gx = p == P64 ? multidot_t<double>(b0, q0, b1, q1, N, w, red, done, Q, st)
                               : multidot_t<float>(b0, q0, b1, q1, N, w, red, done, Q, st);
  DC_HIP(hipGetLastError());
  // value v of the launch is result v (value = group * 2G + 2*(q - g0) + re/im = 2q + re/im)
  launch_finalize(red.partials, 2 * Q, int(gx), result, done, st);
}

// Workgroups of the update over Q basis vectors: the wave-split kernel when the
// basis has more than one chunk, else the flat one.
static unsigned axpy_blocks(size_t N, bool split) {
  const size_t per = split ? size_t(64) * kDotE : size_t(256) * kDotE;
  const size_t nb = std::min<size_t>((N + per - 1) / per, split ? 4096 : 2048);
  return unsigned(std::max<size_t>(nb, 1));
}

void launch_multiaxpy(Prec p, void* w, const void* b0, int q0, const void* b1, int q1, size_t N,
                      const double* coef, int want_norm, Reducer red, double* result,
                      const int* done, hipStream_t st) {
  if (q0 + q1 == 0 && !want_norm) return;
  const bool split = q0 + q1 > kAxpyG;
  const unsigned nb = axpy_blocks(N, split);
  if (p == P64) {
    auto k = split ? k_multiaxpy<double> : k_multiaxpy_flat<double>;
    hipLaunchKernelGGL(k, dim3(nb), dim3(256), 0, st, static_cast<const z64*>(w),
                       static_cast<z64*>(w), static_cast<const z64*>(b0), q0,
                       static_cast<const z64*>(b1), q1, N, coef, want_norm, red, done);
  } else {
    auto k = split ? k_multiaxpy<float> : k_multiaxpy_flat<float>;
    hipLaunchKernelGGL(k, dim3(nb), dim3(256), 0, st, static_cast<const z32*>(w),
                       static_cast<z32*>(w), static_cast<const z32*>(b0), q0,
                       static_cast<const z32*>(b1), q1, N, coef, want_norm, red, done);
  }
  DC_HIP(hipGetLastError());
  if (want_norm) launch_finalize(red.partials, 1, int(nb), result, done, st);
}

template <typename VR>
static void gram_schmidt_t(const void* b0, int q0, const void* b1, int q1, size_t N, void* w,
                           Reducer red, double* res1, double* res2, const ArnoldiDev& a,
                           bool single_sync, int steps, int kC, int j, double target, double brk,
                           hipStream_t st) {
  const Prec p = sizeof(VR) == 8 ? P64 : P32;
  const int Q = q0 + q1, nvals = 2 * Q + 1;
  const cx<VR>*v0 = static_cast<const cx<VR>*>(b0), *v1 = static_cast<const cx<VR>*>(b1);
  // partials per value of the launch before, 0 if they were summed to `result`
  auto settle = [&](unsigned gx, const double* parts, double* result) {
    if (Q <= kFoldQ && gx <= unsigned(kFoldParts)) return int(gx);
    launch_finalize(parts, nvals, int(gx), result, a.done, st);
    return 0;
  };
  const double* last = red.partials;
  double* cres = res1;
  unsigned gx = multidot_t<VR>(b0, q0, b1, q1, N, w, red, a.done, Q + 1, st, a.go, j + 1);
  DC_HIP(hipGetLastError());
  int np = settle(gx, red.partials, res1);
  if (!single_sync) {
    cres = res2;
    // behind the partials that the next kernel still sums (of at most kFoldQ + 1 vectors,
    // rounded up to a group of 16)
    constexpr int kept = 2 * (kFoldQ + 16) * kFoldParts;
    static_assert(kept <= kRedCap / 2, "room for the second kernel's partials");
    double* second = red.partials + (np > 0 ? kept : 0);
    const int cap = kRedCap - (np > 0 ? kept : 0);
    last = second;
    if (Q <= kFoldQ) {
      // at most two workgroups per CU (their registers allow no more), with equal
      // numbers of tiles
      const size_t tiles = (N + 63) / 64;
      const size_t most = std::min<size_t>(512, size_t(cap) / size_t(nvals));
      const size_t rounds = (tiles + most - 1) / most;
      gx = unsigned(std::max<size_t>((tiles + rounds - 1) / std::max<size_t>(rounds, 1), 1));
      auto k = np > 0 ? k_update_dot<VR, true> : k_update_dot<VR, false>;
      hipLaunchKernelGGL(k, dim3(gx), dim3(256), 0, st, v0, q0, v1, q1, N, static_cast<cx<VR>*>(w),
                         red.partials, np, res1, second, a.done);
      DC_HIP(hipGetLastError());
    } else {
      // more vectors than a workgroup's registers hold: the update and its dots
      // each read the basis
      launch_multiaxpy(p, w, b0, q0, b1, q1, N, res1, 0, red, nullptr, a.done, st);
      gx = multidot_t<VR>(b0, q0, b1, q1, N, w, red, a.done, Q + 1, st);
      DC_HIP(hipGetLastError());
    }
    np = settle(gx, second, res2);
  }
  StepEnd e{};
  e.a = a;
  e.c1 = single_sync ? nullptr : res1;
  e.target = target;
  e.brk = brk;
  e.steps = steps;
  e.kC = kC;
  e.j = j;
  const bool split = Q > kAxpyG;
  // up to 32 vectors in chunks of 8, so that all four waves have one (8^4, n = 48, FP64,
  // 17 to 30 vectors: 18.7 -> 16.2 us)
  auto k = !split ? (np > 0 ? k_step_end<VR, 0, true> : k_step_end<VR, 0, false>)
           : Q <= 32 ? (np > 0 ? k_step_end<VR, 8, true> : k_step_end<VR, 8, false>)
                     : (np > 0 ? k_step_end<VR, kAxpyG, true> : k_step_end<VR, kAxpyG, false>);
  // (the sums and the norm once per workgroup: at most two per CU)
  hipLaunchKernelGGL(k, dim3(std::min(axpy_blocks(N, split), 512u) + 1), dim3(256), 0, st,
                     static_cast<cx<VR>*>(w), v0, q0, v1, q1, N, np > 0 ? last : cres, np, e);
  DC_HIP(hipGetLastError());
}

void launch_gram_schmidt(Prec p, const void* b0, int q0, const void* b1, int q1, size_t N, void* w,
                         Reducer red, double* res1, double* res2, const ArnoldiDev& a,
                         bool single_sync, int steps, int kC, int j, double target, double brk,
                         hipStream_t st) {
  if (p == P64)
    gram_schmidt_t<double>(b0, q0, b1, q1, N, w, red, res1, res2, a, single_sync, steps, kC, j,
                           target, brk, st);
  else
    gram_schmidt_t<float>(b0, q0, b1, q1, N, w, red, res1, res2, a, single_sync, steps, kC, j,
                          target, brk, st);
}

namespace {
int g_batch_launches = 1;
}

void set_batch_launches(int batched) {
  if (batched != 0 && batched != 1) throw InvalidArg("batched launch mode must be 0 or 1");
  g_batch_launches = batched;
}

int batch_launches() { return g_batch_launches; }

static void check_cols(int count) {
  if (count < 0 || count > kOrthCols) throw InvalidArg("column table holds 0..16 columns");
}

static int common_q(const OrthCols& t) {
  const int Q = t.c[0].q0 + t.c[0].q1;
  for (int c = 1; c < t.count; ++c)
    if (t.c[c].q0 + t.c[c].q1 != Q) throw InvalidArg("batched columns need equal basis sizes");
  return Q;
}

template <typename VR, int G>
static void multidot_cols_g(OrthCols t, int Q, hipStream_t st) {
  const int gy = (Q + G - 1) / G;
  unsigned gmax = 1;
  for (int c = 0; c < t.count; ++c) {
    t.c[c].gx = dot_blocks(t.c[c].N, gy * 2 * G);   // as its own launch would take
    gmax = std::max(gmax, t.c[c].gx);
  }
  hipLaunchKernelGGL((k_multidot_cols<VR, G>), dim3(gmax, unsigned(gy), unsigned(t.count)),
                     dim3(256), 0, st, t);
  DC_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_finalize_cols, dim3(unsigned(2 * Q), 1u, unsigned(t.count)), dim3(64), 0,
                     st, t);
  DC_HIP(hipGetLastError());
}

template <typename VR>
static void multidot_cols_t(const OrthCols& t, int Q, hipStream_t st) {
  if (Q <= 2) multidot_cols_g<VR, 2>(t, Q, st);
  else if (Q <= 4) multidot_cols_g<VR, 4>(t, Q, st);
  else if (Q <= 8) multidot_cols_g<VR, 8>(t, Q, st);
  else multidot_cols_g<VR, 16>(t, Q, st);
}

void launch_multidot_cols(Prec p, const OrthCols& t, int want_norm, hipStream_t st) {
  check_cols(t.count);
  if (t.count == 0) return;
  const int Q = common_q(t) + (want_norm ? 1 : 0);
  if (Q == 0) return;
  if (p == P64) multidot_cols_t<double>(t, Q, st);
  else multidot_cols_t<float>(t, Q, st);
}

void launch_multiaxpy_cols(Prec p, const OrthCols& t0, int want_norm, hipStream_t st) {
  check_cols(t0.count);
  if (t0.count == 0) return;
  const int Q = common_q(t0);
  if (Q == 0 && !want_norm) return;
  OrthCols t = t0;
  // the grid of each column's own launch (multiaxpy_any)
  const bool split = Q > kAxpyG;
  const size_t per = split ? size_t(64) * kDotE : size_t(256) * kDotE;
  const size_t cap = split ? 4096 : 2048;
  unsigned gmax = 1;
  for (int c = 0; c < t.count; ++c) {
    size_t nb = (t.c[c].N + per - 1) / per;
    if (nb > cap) nb = cap;
    if (nb < 1) nb = 1;
    t.c[c].gx = unsigned(nb);
    gmax = std::max(gmax, t.c[c].gx);
  }
  const dim3 grid(gmax, 1u, unsigned(t.count));
  if (p == P64) {
    if (split) hipLaunchKernelGGL((k_multiaxpy_cols<double, true>), grid, dim3(256), 0, st, t, want_norm);
    else hipLaunchKernelGGL((k_multiaxpy_cols<double, false>), grid, dim3(256), 0, st, t, want_norm);
  } else {
    if (split) hipLaunchKernelGGL((k_multiaxpy_cols<float, true>), grid, dim3(256), 0, st, t, want_norm);
    else hipLaunchKernelGGL((k_multiaxpy_cols<float, false>), grid, dim3(256), 0, st, t, want_norm);
  }
  DC_HIP(hipGetLastError());
  if (want_norm) {
    hipLaunchKernelGGL(k_finalize_cols, dim3(1u, 1u, unsigned(t.count)), dim3(64), 0, st, t);
    DC_HIP(hipGetLastError());
  }
}

void launch_arnoldi_finish_cols(const FinishCols& t, int steps, int j, double brk,
                                hipStream_t st) {
  check_cols(t.count);
  if (t.count == 0) return;
  hipLaunchKernelGGL(k_arnoldi_finish_cols, dim3(unsigned(t.count)), dim3(64), 0, st, t, steps, j,
                     brk);
  DC_HIP(hipGetLastError());
}

void launch_scale_step_cols(Prec p, const ScaleCols& t, int j, hipStream_t st) {
  check_cols(t.count);
  if (t.count == 0) return;
  size_t nmax = 1;
  for (int c = 0; c < t.count; ++c) nmax = std::max(nmax, t.N[c]);
  const dim3 grid(grid_for(nmax, 256), 1u, unsigned(t.count)), block(256);
  if (p == P64) hipLaunchKernelGGL(k_scale_step_cols<double>, grid, block, 0, st, t, j);
  else hipLaunchKernelGGL(k_scale_step_cols<float>, grid, block, 0, st, t, j);
  DC_HIP(hipGetLastError());
}

int block_gram_parts(size_t N, int qa, int rb, size_t part_cap) {
  // enough chunks that chunks x output tiles fill the chip twice over, each
  // chunk at least 8 LDS rounds long, within the partials' capacity
  const size_t tiles = size_t((qa + kBpT - 1) / kBpT) * size_t((rb + kBpT - 1) / kBpT);
  size_t P = (2048 + tiles - 1) / std::max<size_t>(tiles, 1);
  P = std::min<size_t>(P, kGramMaxParts);
  P = std::min<size_t>(P, std::max<size_t>(N / (8 * kBpK), 1));
  if (part_cap) P = std::min<size_t>(P, part_cap / std::max<size_t>(size_t(qa) * size_t(rb), 1));
  return int(std::max<size_t>(P, 1));
}

template <typename VS, typename VC>
static void block_gram_t(const void* A, int qa, const void* B, int rb, size_t N, size_t part_cap,
                         void* part, z64* out, hipStream_t st) {
  const int P0 = block_gram_parts(N, qa, rb, part_cap);
  size_t L = (N + size_t(P0) - 1) / size_t(P0);
  L = (L + kBpK - 1) / kBpK * kBpK;
  const int P = int((N + L - 1) / L);
  const unsigned tiles = unsigned((qa + kBpT - 1) / kBpT) * unsigned((rb + kBpT - 1) / kBpT);
  const size_t qr = size_t(qa) * size_t(rb);
  hipLaunchKernelGGL((k_block_gram<VS, VC>), dim3(unsigned(P), tiles), dim3(256), 0, st,
                     static_cast<const cx<VS>*>(A), qa, static_cast<const cx<VS>*>(B), rb, N, L,
                     static_cast<cx<VC>*>(part));
  DC_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_block_gram_sum<VC>, dim3(unsigned((qr + 255) / 256)), dim3(256), 0, st,
                     static_cast<const cx<VC>*>(part), P, qr, out);
  DC_HIP(hipGetLastError());
}

void launch_block_gram(Prec p, const void* A, int qa, const void* B, int rb, size_t N, void* part,
                       z64* out, hipStream_t st, bool fp64_products, size_t part_cap) {
  if (qa <= 0 || rb <= 0) return;
  if (p == P64)
    block_gram_t<double, double>(A, qa, B, rb, N, part_cap, part, out, st);
  else if (fp64_products)
    block_gram_t<float, double>(A, qa, B, rb, N, part_cap, part, out, st);
  else
    block_gram_t<float, float>(A, qa, B, rb, N, part_cap, part, out, st);
}

template <typename VS, typename VC>
static void block_update_t(const void* b0, int q0, const void* b1, int q1, const void* S, int ldS,
                           void* C, int r, size_t N, z64 alpha, z64 beta, hipStream_t st) {
  const size_t tiles = ((N + kBpT - 1) / kBpT) * size_t((r + kBpT - 1) / kBpT);
  if (tiles > 0xffffffffull) throw InvalidArg("block update too large");
  hipLaunchKernelGGL((k_block_update<VS, VC>), dim3(unsigned(tiles)), dim3(256), 0, st,
                     static_cast<const cx<VS>*>(b0), q0, static_cast<const cx<VS>*>(b1), q1,
                     static_cast<const cx<VC>*>(S), ldS, static_cast<cx<VS>*>(C), r, N, alpha,
                     beta);
  DC_HIP(hipGetLastError());
}

void launch_block_update(Prec p, const void* A, int k, const void* S, void* C, int r, size_t N,
                         z64 alpha, z64 beta, hipStream_t st) {
  if (r <= 0 || N == 0) return;
  if (p == P64)
    block_update_t<double, double>(A, k, nullptr, 0, S, k, C, r, N, alpha, beta, st);
  else
    block_update_t<float, float>(A, k, nullptr, 0, S, k, C, r, N, alpha, beta, st);
}

void launch_combine(Prec p, const void* b0, int q0, const void* b1, int q1, size_t N,
                    const double* coef, int R, void* out, int accumulate, hipStream_t st) {
  if (R <= 0) return;
  if (R == 1) {
    size_t nb = (N + 64 * kDotE - 1) / (64 * kDotE);
    if (nb > 4096) nb = 4096;
    if (nb < 1) nb = 1;
    const dim3 grid{static_cast<unsigned>(nb)}, block{256};
    if (q0 + q1 == 0) {
      if (!accumulate) launch_zero(p, out, N, st);
      return;
    }
    if (p == P64)
      hipLaunchKernelGGL(k_combine1<double>, grid, block, 0, st, static_cast<const z64*>(b0), q0,
                         static_cast<const z64*>(b1), q1, N, coef, static_cast<z64*>(out),
                         accumulate);
    else
      hipLaunchKernelGGL(k_combine1<float>, grid, block, 0, st, static_cast<const z32*>(b0), q0,
                         static_cast<const z32*>(b1), q1, N, coef, static_cast<z32*>(out),
                         accumulate);
    DC_HIP(hipGetLastError());
    return;
  }
  if (R >= kCombMfmaMin && q0 + q1 > 0) {
    // many outputs: the MFMA block update with FP64 products and sums (the
    // coefficients are FP64), out = sum + (accumulate ? out : 0)
    const z64 one = mk(1.0, 0.0), beta = mk(accumulate ? 1.0 : 0.0, 0.0);
    if (p == P64)
      block_update_t<double, double>(b0, q0, b1, q1, coef, q0 + q1, out, R, N, one, beta, st);
    else
      block_update_t<float, double>(b0, q0, b1, q1, coef, q0 + q1, out, R, N, one, beta, st);
    return;
  }
  const int gy = (R + kCombR - 1) / kCombR;
  const dim3 grid(grid_for(N, 256, 2048), unsigned(gy)), block(256);
  if (p == P64)
    hipLaunchKernelGGL(k_combine<double>, grid, block, 0, st, static_cast<const z64*>(b0), q0,
                       static_cast<const z64*>(b1), q1, N, coef, R, static_cast<z64*>(out),
                       accumulate);
  else
    hipLaunchKernelGGL(k_combine<float>, grid, block, 0, st, static_cast<const z32*>(b0), q0,
                       static_cast<const z32*>(b1), q1, N, coef, R, static_cast<z32*>(out),
                       accumulate);
  DC_HIP(hipGetLastError());
}

void launch_scale(Prec p, const void* in, void* out, size_t N, const double* scale_dev, double s,
                  const int* done, hipStream_t st) {
  const dim3 grid(grid_for(N, 256)), block(256);
  if (p == P64)
    hipLaunchKernelGGL(k_scale<double>, grid, block, 0, st, static_cast<const z64*>(in),
                       static_cast<z64*>(out), N, scale_dev, s, done);
  else
    hipLaunchKernelGGL(k_scale<float>, grid, block, 0, st, static_cast<const z32*>(in),
                       static_cast<z32*>(out), N, scale_dev, s, done);
  DC_HIP(hipGetLastError());
}

void launch_cscale(Prec p, const void* in, void* out, size_t N, z64 c, const int* done,
                   hipStream_t st) {
  const dim3 grid(grid_for(N, 256)), block(256);
  if (p == P64)
    hipLaunchKernelGGL(k_cscale<double>, grid, block, 0, st, static_cast<const z64*>(in),
                       static_cast<z64*>(out), N, c, done);
  else
    hipLaunchKernelGGL(k_cscale<float>, grid, block, 0, st, static_cast<const z32*>(in),
                       static_cast<z32*>(out), N, c, done);
  DC_HIP(hipGetLastError());
}

void launch_scale_step(Prec p, void* v, size_t N, const double* inv_h, const int* jdone, int j,
                       hipStream_t st) {
  const dim3 grid(grid_for(N, 256)), block(256);
  if (p == P64)
    hipLaunchKernelGGL(k_scale_step<double>, grid, block, 0, st, static_cast<z64*>(v), N, inv_h,
                       jdone, j);
  else
    hipLaunchKernelGGL(k_scale_step<float>, grid, block, 0, st, static_cast<z32*>(v), N, inv_h,
                       jdone, j);
  DC_HIP(hipGetLastError());
}

// 4-byte words from src to dst; one side is host-mapped pinned memory (the
// staged transfers between the solver's host logic and the device, which as
// kernels queue without the host-side cost of a copy call).
__global__ void k_copy_words(const uint32_t* __restrict__ src, uint32_t* __restrict__ dst,
                             size_t n) {
  const size_t stride = size_t(gridDim.x) * blockDim.x;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride)
    dst[i] = src[i];
}

void launch_copy_words(const void* src, void* dst, size_t bytes, hipStream_t st) {
  if (bytes == 0) return;
  if (bytes % 4 != 0 || reinterpret_cast<uintptr_t>(src) % 4 != 0 ||
      reinterpret_cast<uintptr_t>(dst) % 4 != 0)
    throw std::invalid_argument("staged copies move aligned 4-byte words");
  const size_t n = bytes / 4;
  const dim3 grid(grid_for(n, 256, 2048)), block(256);
  hipLaunchKernelGGL(k_copy_words, grid, block, 0, st, static_cast<const uint32_t*>(src),
                     static_cast<uint32_t*>(dst), n);
  DC_HIP(hipGetLastError());
}

// Several segments of 4-byte words in one launch (blockIdx.y = segment).
__global__ void k_copy_segments(CopySegments s) {
  const int g = blockIdx.y;
  const uint32_t* __restrict__ src = s.src[g];
  uint32_t* __restrict__ dst = s.dst[g];
  const size_t n = s.words[g];
  const size_t stride = size_t(gridDim.x) * blockDim.x;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) dst[i] = src[i];
}

void launch_copy_segments(const CopySegments& s, hipStream_t st) {
  if (s.count <= 0) return;
  if (s.count > kCopySegMax) throw std::invalid_argument("too many copy segments");
  size_t most = 0;
  for (int g = 0; g < s.count; ++g) most = std::max(most, s.words[g]);
  const dim3 grid(grid_for(most, 256, 256), unsigned(s.count)), block(256);
  hipLaunchKernelGGL(k_copy_segments, grid, block, 0, st, s);
  DC_HIP(hipGetLastError());
}

void launch_zero(Prec p, void* x, size_t N, hipStream_t st) {
  const dim3 grid(grid_for(N, 256)), block(256);
  if (p == P64)
    hipLaunchKernelGGL(k_zero<double>, grid, block, 0, st, static_cast<z64*>(x), N);
  else
    hipLaunchKernelGGL(k_zero<float>, grid, block, 0, st, static_cast<z32*>(x), N);
  DC_HIP(hipGetLastError());
}

void launch_axpy(Prec p, z64 a, const void* x, void* y, size_t N, hipStream_t st) {
  const dim3 grid(grid_for(N, 256)), block(256);
  if (p == P64)
    hipLaunchKernelGGL(k_axpy<double>, grid, block, 0, st, a, static_cast<const z64*>(x),
                       static_cast<z64*>(y), N);
  else
    hipLaunchKernelGGL(k_axpy<float>, grid, block, 0, st, a, static_cast<const z32*>(x),
                       static_cast<z32*>(y), N);
  DC_HIP(hipGetLastError());
}

void launch_colnorm2(Prec p, const void* x, int q, size_t N, Reducer red, double* result,
                     hipStream_t st) {
  if (q <= 0) return;
  unsigned nb = red_blocks(N);
  const unsigned cap = unsigned(size_t(kRedCap) / size_t(q));
  if (nb > cap) nb = cap;
  const dim3 grid(nb, unsigned(q)), block(256);
  if (p == P64)
    hipLaunchKernelGGL(k_norm2<double>, grid, block, 0, st, static_cast<const z64*>(x), N, red);
  else
    hipLaunchKernelGGL(k_norm2<float>, grid, block, 0, st, static_cast<const z32*>(x), N, red);
  DC_HIP(hipGetLastError());
  launch_finalize(red.partials, q, int(nb), result, nullptr, st);
}

void launch_norm2(Prec p, const void* x, size_t N, Reducer red, double* result, hipStream_t st) {
  launch_colnorm2(p, x, 1, N, red, result, st);
}

void launch_gamma5(Prec p, const void* in, void* out, int V, int n, hipStream_t st) {
  const size_t N = size_t(V) * n;
  const dim3 grid(grid_for(N, 256)), block(256);
  if (p == P64)
    hipLaunchKernelGGL(k_gamma5<double>, grid, block, 0, st, static_cast<const z64*>(in),
                       static_cast<z64*>(out), N, n);
  else
    hipLaunchKernelGGL(k_gamma5<float>, grid, block, 0, st, static_cast<const z32*>(in),
                       static_cast<z32*>(out), N, n);
  DC_HIP(hipGetLastError());
}

void launch_convert_64to32(const z64* in, z32* out, size_t N, int n, int g5, hipStream_t st) {
  hipLaunchKernelGGL(k_cvt64to32, dim3(grid_for(N, 256)), dim3(256), 0, st, in, out, N, n, g5);
  DC_HIP(hipGetLastError());
}

void launch_convert_32to64(const z32* in, z64* out, size_t N, int n, int g5, hipStream_t st) {
  hipLaunchKernelGGL(k_cvt32to64, dim3(grid_for(N, 256)), dim3(256), 0, st, in, out, N, n, g5);
  DC_HIP(hipGetLastError());
}

void launch_gaussian(z64* out, size_t N, uint64_t seed, uint32_t stream_id, hipStream_t st) {
  hipLaunchKernelGGL(k_gaussian, dim3(grid_for(N, 256)), dim3(256), 0, st, out, N, seed,
                     stream_id);
  DC_HIP(hipGetLastError());
}

void launch_arnoldi_finish(ArnoldiDev a, int steps, int kC, int j, const double* c1,
                           const double* c2, const double* nrm2, double target, double brk,
                           hipStream_t st) {
  hipLaunchKernelGGL(k_arnoldi_finish, dim3(1), dim3(64), 0, st, a, steps, kC, j, c1, c2, nrm2,
                     target, brk);
  DC_HIP(hipGetLastError());
}

void launch_arnoldi_init(ArnoldiDev a, double beta, hipStream_t st, const double* beta_dev) {
  hipLaunchKernelGGL(k_arnoldi_init, dim3(1), dim3(64), 0, st, a, beta, beta_dev);
  DC_HIP(hipGetLastError());
}

// out[0] = sqrt(max(*nrm2, 0)), out[1] = 1 / out[0] (0 for a zero norm)
__global__ void k_norm_root(const double* __restrict__ nrm2, double* __restrict__ out) {
  if (threadIdx.x == 0) {
    const double b = sqrt(fmax(*nrm2, 0.0));
    out[0] = b;
    out[1] = b > 0.0 ? 1.0 / b : 0.0;
  }
}

void launch_norm_root(const double* nrm2, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_norm_root, dim3(1), dim3(64), 0, st, nrm2, out);
  DC_HIP(hipGetLastError());
}

}  // namespace dc
