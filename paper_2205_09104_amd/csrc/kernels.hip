// HIP kernels for gfx950 (CDNA4): coarse-operator apply, reduced operator and the
// gradient kernel.
#include "kernels.hpp"
#include "device.hpp"

#include <hip/hip_ext.h>

#include <algorithm>
#include <mutex>


// Scratch of the no-allocation reduced apply (dc_apply_reduced_noalloc): the
// odd-row temporary t_o lives in this file-scope device array, one copy per
// GPU, held until the process ends.  Host code never passes `scratch` itself
// to a kernel (in host code it names a host-side stand-in): it passes the
// device address that hipGetSymbolAddress returned for the current device.
static __device__ __align__(256) unsigned char scratch[dc::kNoAllocScratchBytes];

namespace dc {

namespace {
std::mutex g_scratch_mu;
void* g_scratch_dev[kMaxDevices] = {};
}  // namespace

void* noalloc_scratch(bool setup) {
  int dev = 0;
  DC_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) throw InvalidArg("device index out of range");
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    if (!setup) return nullptr;
    void* p = nullptr;
    DC_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) throw HipError("hipGetSymbolAddress returned a null address for the scratch array");
    g_scratch_dev[dev] = p;
  }
  return g_scratch_dev[dev];
}

namespace {

__global__ void k_neighbours(int* nbr, int L0, int L1, int L2, int L3) {
  const int V = L0 * L1 * L2 * L3;
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  if (x >= V) return;
  int c[4];
  c[0] = x % L0;
  c[1] = (x / L0) % L1;
  c[2] = (x / (L0 * L1)) % L2;
  c[3] = x / (L0 * L1 * L2);
  const int L[4] = {L0, L1, L2, L3};
  for (int mu = 0; mu < 4; ++mu) {
    for (int dir = 0; dir < 2; ++dir) {
      int d[4] = {c[0], c[1], c[2], c[3]};
      d[mu] = dir == 0 ? (d[mu] + 1) % L[mu] : (d[mu] + L[mu] - 1) % L[mu];
      nbr[(dir * 4 + mu) * V + x] = d[0] + L0 * (d[1] + L1 * (d[2] + L2 * d[3]));
    }
  }
}

// ------------------------------------------------------------------ apply
// Element loaders of one lane's sub-tile for each storage precision.
template <int T, int P>
struct Tile;

template <int T>
struct Tile<T, P64> {
  using A = double;
  static constexpr int TT = T * T;
  static constexpr int UNITS = TT;  // one complex double per 16-byte unit
  __device__ static void load(const void* base, int lane, cx<double> (&m)[TT]) {
    const double2* p = static_cast<const double2*>(base);
#pragma unroll
    for (int e = 0; e < TT; ++e) {
      const double2 v = p[e * 64 + lane];
      m[e] = mk(v.x, v.y);
    }
  }
};

template <int T>
struct Tile<T, P32> {
  using A = float;
  static constexpr int TT = T * T;
  static constexpr int UNITS = (TT + 1) / 2;
  __device__ static void load(const void* base, int lane, cx<float> (&m)[TT]) {
    const float4* p = static_cast<const float4*>(base);
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
      const float4 v = p[u * 64 + lane];
      m[2 * u] = mk(v.x, v.y);
      if (2 * u + 1 < TT) m[2 * u + 1] = mk(v.z, v.w);
    }
  }
};

template <int T>
struct Tile<T, P16S> {
  using A = float;
  static constexpr int TT = T * T;
  static constexpr int UNITS = (TT + 3) / 4;
};

template <int P>
struct VecOf {
  using R = float;
};
template <>
struct VecOf<P64> {
  using R = double;
};

// Cross-lane sums inside a wavefront.  Lanes are l = lr*8 + lc.  Row sums
// (over lc, lanes l^1, l^2, l^4) use DPP quad permutes and the half-row mirror;
// column sums (over lr, lanes l^8, l^16, l^32) use a DPP row rotation by 8 and
// the gfx950 permlane16/32 swaps, whose two outputs add to v[l] + v[l^16]
// (resp. v[l^32]) in every lane.
template <int CTL>
__device__ inline float dppf(float v) {
  int i = __float_as_int(v);
  if (CTL == 1) i = dpp_xor1(i);
  if (CTL == 2) i = dpp_xor2(i);
  if (CTL == 4) i = dpp_hmirror(i);
  if (CTL == 8) i = dpp_ror8(i);
  return __int_as_float(i);
}
template <int CTL>
__device__ inline double dppd(double v) {
  const long long b = __double_as_longlong(v);
  const float lo = dppf<CTL>(__int_as_float(int(b & 0xffffffff)));
  const float hi = dppf<CTL>(__int_as_float(int(b >> 32)));
  return __longlong_as_double((long long)(unsigned(__float_as_int(lo))) |
                              ((long long)(__float_as_int(hi)) << 32));
}
__device__ inline float sum_row8(float v) {  // over lc
  v += dppf<1>(v);
  v += dppf<2>(v);
  v += dppf<4>(v);
  return v;
}
__device__ inline double sum_row8(double v) {
  v += dppd<1>(v);
  v += dppd<2>(v);
  v += dppd<4>(v);
  return v;
}
__device__ inline float swap_sum16(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ inline float swap_sum32(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ inline double swap_pair16(double v, double& other) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = unsigned(b & 0xffffffff), hi = unsigned(b >> 32);
  const auto rl = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
  const auto rh = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
  other = __longlong_as_double((long long)rl[1] | ((long long)rh[1] << 32));
  return __longlong_as_double((long long)rl[0] | ((long long)rh[0] << 32));
}
__device__ inline double swap_pair32(double v, double& other) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = unsigned(b & 0xffffffff), hi = unsigned(b >> 32);
  const auto rl = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
  const auto rh = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
  other = __longlong_as_double((long long)rl[1] | ((long long)rh[1] << 32));
  return __longlong_as_double((long long)rl[0] | ((long long)rh[0] << 32));
}
__device__ inline float sum_col8(float v) {  // over lr
  v += dppf<8>(v);
  v = swap_sum16(v);
  return swap_sum32(v);
}
__device__ inline double sum_col8(double v) {
  v += dppd<8>(v);
  double o;
  double a = swap_pair16(v, o);
  v = a + o;
  a = swap_pair32(v, o);
  return a + o;
}

// gbuf slots per site: 0..3 receive the backward hops Gamma5 B[x-mu,mu]^H
// Gamma5 psi_{x-mu}; 4 the self block (with i*tm*Gamma5 psi_x); 5..8 the
// forward hops B[x,mu] psi_{x+mu}.
constexpr int kSlots = 9;

// Block element access: FP64 / FP32 tiles are decoded into complex values,
// FP16 tiles stay packed (re in the low, im in the high half of a 32-bit
// word) and are widened inside the mixed-precision FMAs.
template <int T, int P>
struct TileRegs {
  using A = typename Tile<T, P>::A;
  static constexpr int TT = T * T;
  static constexpr int UNITS = Tile<T, P>::UNITS;
  cx<A> m[TT];
  __device__ void load(const void* base, int lane) { Tile<T, P>::load(base, lane, m); }
  // the same with non-temporal loads, for tiles that one launch reads once
  __device__ void load_stream(const void* base, int lane) {
    typedef A avec __attribute__((ext_vector_type(16 / sizeof(A))));
    const avec* p = static_cast<const avec*>(base);
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
      const avec v = __builtin_nontemporal_load(p + u * 64 + lane);
      if constexpr (P == P64) {
        m[u] = mk(v.x, v.y);
      } else {
        m[2 * u] = mk(v.x, v.y);
        if (2 * u + 1 < TT) m[2 * u + 1] = mk(v.z, v.w);
      }
    }
  }
};

template <int T>
struct TileRegs<T, P16S> {
  static constexpr int TT = T * T;
  static constexpr int UNITS = (TT + 3) / 4;
  uint32_t w[UNITS * 4];
  __device__ void load(const void* base, int lane) {
    const uint4* p = static_cast<const uint4*>(base);
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
      const uint4 v = p[u * 64 + lane];
      w[4 * u] = v.x;
      w[4 * u + 1] = v.y;
      w[4 * u + 2] = v.z;
      w[4 * u + 3] = v.w;
    }
  }
  // the same with non-temporal loads, for tiles that one launch reads once
  __device__ void load_stream(const void* base, int lane) {
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    const u32x4* p = static_cast<const u32x4*>(base);
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
      const u32x4 v = __builtin_nontemporal_load(p + u * 64 + lane);
      w[4 * u] = v.x;
      w[4 * u + 1] = v.y;
      w[4 * u + 2] = v.z;
      w[4 * u + 3] = v.w;
    }
  }
};

// Accumulate one lane's sub-tile: f_a += z_ac pc_c and (hop blocks)
// g_c += conj(z_ac) pr_a.  npc_im = -Im(pc), npr_re = -Re(pr) avoid sign flips
// per element.
// f += M pc (row products, DOF) and g += M^T pr (column products, DOG) over one
// lane's T x T sub-tile.
template <int T, int P, bool DOF, bool DOG, typename A>
__device__ inline void tile_products(const TileRegs<T, P>& R, const cx<A> (&pc)[T],
                                     const A (&npc_im)[T], const cx<A> (&pr)[T],
                                     const A (&npr_re)[T], cx<A> (&f)[T], cx<A> (&g)[T]) {
#pragma unroll
  for (int a = 0; a < T; ++a)
#pragma unroll
    for (int c = 0; c < T; ++c) {
      A zr, zi;
      if constexpr (P == P16S) {
        zr = lo_h(R.w[a * T + c]);
        zi = hi_h(R.w[a * T + c]);
      } else {
        zr = R.m[a * T + c].re;
        zi = R.m[a * T + c].im;
      }
      if constexpr (DOF) {
        f[a].re = fma(zr, pc[c].re, f[a].re);
        f[a].re = fma(zi, npc_im[c], f[a].re);
        f[a].im = fma(zr, pc[c].im, f[a].im);
        f[a].im = fma(zi, pc[c].re, f[a].im);
      }
      if constexpr (DOG) {
        g[c].re = fma(zr, pr[a].re, g[c].re);
        g[c].re = fma(zi, pr[a].im, g[c].re);
        g[c].im = fma(zr, pr[a].im, g[c].im);
        g[c].im = fma(zi, npr_re[a], g[c].im);
      }
    }
}

// One stored block of one site, processed by one wave.  Full lattice (the
// default): the self block writes slot 4 of gbuf[x]; a hop block B[x,mu]
// writes B psi_{x+mu} into slot 5+mu of gbuf[x] and Gamma5 B^H Gamma5 psi_x
// into slot mu of gbuf[x+mu].  G5: Gamma5 before and after (the adjoint through
// Gamma5 D(-mu) Gamma5), as signs of the products' inputs and outputs.
template <int T, int P, bool FULL, bool HOP, bool G5>
__device__ __forceinline__ void apply_one_block(
    const uint4* __restrict__ bp, const float* __restrict__ scales,
    const cx<typename VecOf<P>::R>* __restrict__ psi, cx<typename VecOf<P>::R>* __restrict__ gbuf,
    int item, int site, int slot, int src, int n, double tm, int stream) {
  using A = typename Tile<T, P>::A;
  using VR = typename VecOf<P>::R;
  constexpr bool DOG = HOP;
  const int lane = threadIdx.x;
  const int lr = lane >> 3, lc = lane & 7;
  TileRegs<T, P> R;
  if (stream) R.load_stream(bp, lane);
  else R.load(bp, lane);
  cx<A> pc[T], pr[T];
  A npc_im[T], npr_re[T];
#pragma unroll
  for (int q = 0; q < T; ++q) {
    const int col = lc * T + q;
    pc[q] = mk(A(0), A(0));
    if (FULL || col < n) {
      const cx<VR> z = psi[size_t(HOP ? src : site) * n + col];
      pc[q] = (G5 && col >= (n >> 1)) ? mk(A(-z.re), A(-z.im)) : mk(A(z.re), A(z.im));
    }
    npc_im[q] = -pc[q].im;
    pr[q] = mk(A(0), A(0));
    if (DOG) {
      const int row = lr * T + q;
      if (FULL || row < n) {
        const cx<VR> z = psi[size_t(site) * n + row];
        pr[q] = (G5 || row < (n >> 1)) ? mk(A(z.re), A(z.im)) : mk(A(-z.re), A(-z.im));
      }
    }
    npr_re[q] = -pr[q].re;
  }
  cx<A> f[T], g[T];
#pragma unroll
  for (int q = 0; q < T; ++q) {
    f[q] = mk(A(0), A(0));
    g[q] = mk(A(0), A(0));
  }
  tile_products<T, P, true, DOG>(R, pc, npc_im, pr, npr_re, f, g);
  A s = A(1);
  if (P == P16S) s = A(scales[item]);
#pragma unroll
  for (int q = 0; q < T; ++q) {
    f[q].re = sum_row8(f[q].re) * s;
    f[q].im = sum_row8(f[q].im) * s;
  }
  if (lc == 0) {
    cx<VR>* dst = gbuf + (size_t(site) * kSlots + (HOP ? 4 + slot : 4)) * n;
#pragma unroll
    for (int q = 0; q < T; ++q) {
      const int row = lr * T + q;
      if (FULL || row < n) {
        const bool low = row >= (n >> 1);
        cx<A> v = f[q];
        if (G5 && low) v = mk(-v.re, -v.im);
        if (!HOP && tm != 0.0) {  // i * tm * Gamma5 psi_x in the accumulation precision
          const A t = A(low ? -tm : tm);
          const cx<VR> z = psi[size_t(site) * n + row];
          v.re -= t * A(z.im);
          v.im += t * A(z.re);
        }
        dst[row] = mk(VR(v.re), VR(v.im));
      }
    }
  }
  if constexpr (DOG) {
#pragma unroll
    for (int q = 0; q < T; ++q) {
      g[q].re = sum_col8(g[q].re) * s;
      g[q].im = sum_col8(g[q].im) * s;
    }
    if (lr == 0) {
      cx<VR>* dst = gbuf + (size_t(src) * kSlots + (slot - 1)) * n;  // x + mu receives it
#pragma unroll
      for (int q = 0; q < T; ++q) {
        const int col = lc * T + q;
        if (FULL || col < n) {
          const A gg = (G5 || col < (n >> 1)) ? A(1) : A(-1);
          dst[col] = mk(VR(gg * g[q].re), VR(gg * g[q].im));
        }
      }
    }
  }
}

// One 64-lane workgroup per (site, stored block).  The wave reads its block
// once with 16-byte loads (1 KB contiguous per load instruction) and forms
// from registers both the forward product B psi_{x+mu} (row sums) and the
// backward product Gamma5 B^H Gamma5 psi_x (column sums).  No barrier: waves
// of different sites overlap their loads with each other's arithmetic.  HBM bound
// with blocks beyond the last-level cache: 16^4, n = 48, FP16: 572 us, 5.5 TB/s of
// block and vector bytes (607 with cached loads); 8^4, n = 48, FP64: 133 us (149).
template <int T, int P, bool FULL, bool G5>
__global__ __launch_bounds__(64) void k_apply_blocks(
    const void* __restrict__ blocks, const float* __restrict__ scales,
    const cx<typename VecOf<P>::R>* __restrict__ psi, cx<typename VecOf<P>::R>* __restrict__ gbuf,
    const int* __restrict__ nbr, int V, int n, int chunk, double tm,
    int stream, const int* __restrict__ done) {
  if (done && *done) return;
  // XCD-aware order: workgroup b runs on XCD b % 8; each XCD gets a
  // contiguous range of (site, block) items, so a site's blocks are streamed
  // together and neighbour vectors are shared through that XCD's L2.
  const int b = blockIdx.x;
  const int item = (b & 7) * chunk + (b >> 3);
  if (item >= 5 * V) return;
  const int site = item / 5, slot = item - 5 * site;  // slot 0 = A, 1 + mu = B[x, mu]
  const size_t blk_units = size_t(Tile<T, P>::UNITS) * 64;
  const uint4* bp = static_cast<const uint4*>(blocks) + size_t(item) * blk_units;
  if (slot == 0) {
    apply_one_block<T, P, FULL, false, G5>(bp, scales, psi, gbuf, item, site, 0, site, n, tm, stream);
  } else {
    const int src = nbr[(slot - 1) * V + site];
    apply_one_block<T, P, FULL, true, G5>(bp, scales, psi, gbuf, item, site, slot, src, n, tm, stream);
  }
}

// ------------------------------------------------------------------ odd-even reduction
// S = A_e - D_eo A_o^{-1} D_oe (Sec. 2.2) in factored form over compressed
// vectors (the site x of either parity sits at row x / 2).  A hop block
// B[x,mu] couples an even and an odd site, and each factor needs it in one
// direction only, so both kernels are site-centric: one workgroup per row, one
// wave per block of that row (every block is read once per launch), each
// wave's n-vector product into LDS, then a fixed-order sum (deterministic).

// One wave's product of a stored block (registers R, scale s) with the
// n-vector v, into dst (LDS): DIR 1 forward B v (row sums), DIR 2 backward
// Gamma5 B^H Gamma5 v (column sums), DIR 0 self block B v + i tm Gamma5 v.
// g5 bit 0 multiplies v by Gamma5 first, bit 1 the product.
template <int T, int P, bool FULL, int DIR>
__device__ __forceinline__ void wave_product(const TileRegs<T, P>& R, typename Tile<T, P>::A s,
                                             const cx<typename VecOf<P>::R>* __restrict__ v,
                                             cx<typename VecOf<P>::R>* dst, int n, double tm,
                                             int lane, int g5 = 0) {
  using A = typename Tile<T, P>::A;
  using VR = typename VecOf<P>::R;
  constexpr bool DOF = DIR != 2, DOG = DIR == 2;
  const int lr = lane >> 3, lc = lane & 7;
  cx<A> pc[T], pr[T], f[T], g[T];
  A npc_im[T], npr_re[T];
#pragma unroll
  for (int q = 0; q < T; ++q) {
    pc[q] = mk(A(0), A(0));
    pr[q] = mk(A(0), A(0));
    if (DOF) {
      const int col = lc * T + q;
      if (FULL || col < n) {
        const cx<VR> z = v[col];
        pc[q] = ((g5 & 1) && col >= (n >> 1)) ? mk(A(-z.re), A(-z.im)) : mk(A(z.re), A(z.im));
      }
    }
    if (DOG) {
      const int row = lr * T + q;
      if (FULL || row < n) {
        const cx<VR> z = v[row];
        pr[q] = ((g5 & 1) || row < (n >> 1)) ? mk(A(z.re), A(z.im)) : mk(A(-z.re), A(-z.im));
      }
    }
    npc_im[q] = -pc[q].im;
    npr_re[q] = -pr[q].re;
    f[q] = mk(A(0), A(0));
    g[q] = mk(A(0), A(0));
  }
  tile_products<T, P, DOF, DOG>(R, pc, npc_im, pr, npr_re, f, g);
  if constexpr (DOF) {
#pragma unroll
    for (int q = 0; q < T; ++q) {
      f[q].re = sum_row8(f[q].re) * s;
      f[q].im = sum_row8(f[q].im) * s;
    }
    if (lc == 0) {
#pragma unroll
      for (int q = 0; q < T; ++q) {
        const int row = lr * T + q;
        if (FULL || row < n) {
          const bool low = row >= (n >> 1);
          cx<A> w = f[q];
          if ((g5 & 2) && low) w = mk(-w.re, -w.im);
          if (DIR == 0 && tm != 0.0) {  // i * tm * Gamma5 v in the accumulation precision
            const bool neg = low && (g5 & 1) == (g5 >> 1);
            const A t = A(neg ? -tm : tm);
            const cx<VR> z = v[row];
            w.re -= t * A(z.im);
            w.im += t * A(z.re);
          }
          dst[row] = mk(VR(w.re), VR(w.im));
        }
      }
    }
  } else {
#pragma unroll
    for (int q = 0; q < T; ++q) {
      g[q].re = sum_col8(g[q].re) * s;
      g[q].im = sum_col8(g[q].im) * s;
    }
    if (lr == 0) {
#pragma unroll
      for (int q = 0; q < T; ++q) {
        const int col = lc * T + q;
        if (FULL || col < n) {
          const A gg = ((g5 & 2) || col < (n >> 1)) ? A(1) : A(-1);
          dst[col] = mk(VR(gg * g[q].re), VR(gg * g[q].im));
        }
      }
    }
  }
}

constexpr int kRedWaves = 9;   // waves per workgroup of the reduced kernels

template <int T, int P>
__device__ __forceinline__ const uint4* block_ptr(const void* blocks, size_t item) {
  return static_cast<const uint4*>(blocks) + item * (size_t(Tile<T, P>::UNITS) * 64);
}

// Tile `item` into R; non-temporally if `stream` says so, FP16 tiles always.
template <int T, int P>
__device__ __forceinline__ void load_block_tile(TileRegs<T, P>& R, const void* blocks, size_t item,
                                                int lane, int stream) {
  if (P == P16S || stream) R.load_stream(block_ptr<T, P>(blocks, item), lane);
  else R.load(block_ptr<T, P>(blocks, item), lane);
}

// The full-lattice apply in one launch, for operators whose blocks stay in the caches:
// workgroup per site, wave 0 the self block, waves 1-4 the forward hops, 5-8 the
// backward hops, summed in the order of the two-kernel form (equal bit for bit).
// Every hop block is read twice, but there is no second launch and nothing goes
// through memory between the two: 4^4, n = 16, FP64: 6.2 us in two kernels -> 3.4.
template <int T, int P, bool FULL>
__global__ __launch_bounds__(64 * kRedWaves) void k_apply_site(
    const void* __restrict__ blocks, const float* __restrict__ scales,
    const cx<typename VecOf<P>::R>* __restrict__ psi, cx<typename VecOf<P>::R>* __restrict__ out,
    const int* __restrict__ nbr, int V, int n, int chunk, double tm, int g5,
    const int* __restrict__ done) {
  using A = typename Tile<T, P>::A;
  using VR = typename VecOf<P>::R;
  __shared__ cx<VR> part[kRedWaves][64];
  if (done && *done) return;
  const int b = blockIdx.x;
  const int x = (b & 7) * chunk + (b >> 3);   // contiguous sites per XCD
  if (x >= V) return;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  TileRegs<T, P> R;
  if (w < 5) {
    const int item = 5 * x + w;
    R.load(block_ptr<T, P>(blocks, size_t(item)), lane);
    const A s = (P == P16S) ? A(scales[item]) : A(1);
    if (w == 0) {
      wave_product<T, P, FULL, 0>(R, s, psi + size_t(x) * n, part[0], n, tm, lane, g5);
    } else {
      const int src = nbr[(w - 1) * V + x];
      wave_product<T, P, FULL, 1>(R, s, psi + size_t(src) * n, part[w], n, 0.0, lane, g5);
    }
  } else {
    const int src = nbr[(w - 1) * V + x];
    const int item = 5 * src + w - 4;
    R.load(block_ptr<T, P>(blocks, size_t(item)), lane);
    const A s = (P == P16S) ? A(scales[item]) : A(1);
    wave_product<T, P, FULL, 2>(R, s, psi + size_t(src) * n, part[w], n, 0.0, lane, g5);
  }
  __syncthreads();
  if (w != 0 || lane >= n) return;
  cx<VR> t = part[0][lane];
#pragma unroll
  for (int k = 1; k < kRedWaves; ++k) {
    t.re += part[k][lane].re;
    t.im += part[k][lane].im;
  }
  out[size_t(x) * n + lane] = t;
}

// t_o = A_o^{-1} D_oe x_e.  Workgroup per odd row r (site x = osite[r]):
// waves 0-3 the forward hops B[x,mu] x_e(x+mu), waves 4-7 the backward hops
// Gamma5 B[x-mu,mu]^H Gamma5 x_e(x-mu), then wave 8 applies the inverse of
// x's self block to the sum of the eight products.
// Rows are ordered XCD-aware as in k_apply_blocks (contiguous rows per XCD).
template <int T, int P, bool FULL, bool G5>
__global__ __launch_bounds__(64 * kRedWaves) void k_reduced_oe(
    const void* __restrict__ blocks, const float* __restrict__ scales,
    const void* __restrict__ inv, const float* __restrict__ invsc,
    const cx<typename VecOf<P>::R>* __restrict__ x_e, cx<typename VecOf<P>::R>* __restrict__ t_o,
    const int* __restrict__ nbr, const int* __restrict__ osite, int V, int n, int chunk,
    const int* __restrict__ done) {
  using A = typename Tile<T, P>::A;
  using VR = typename VecOf<P>::R;
  __shared__ cx<VR> part[8][64];
  if (done && *done) return;
  const int b = blockIdx.x;
  const int r = (b & 7) * chunk + (b >> 3);
  if (r >= (V >> 1)) return;
  const int x = osite[r];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  TileRegs<T, P> R;
  if (w < 4) {
    const int item = 5 * x + 1 + w;
    R.load(block_ptr<T, P>(blocks, size_t(item)), lane);
    const A s = (P == P16S) ? A(scales[item]) : A(1);
    const int src = nbr[w * V + x];
    wave_product<T, P, FULL, 1>(R, s, x_e + size_t(src >> 1) * n, part[w], n, 0.0, lane, G5 ? 1 : 0);
  } else if (w < 8) {
    const int mu = w - 4;
    const int y = nbr[(4 + mu) * V + x];
    const int item = 5 * y + 1 + mu;
    R.load(block_ptr<T, P>(blocks, size_t(item)), lane);
    const A s = (P == P16S) ? A(scales[item]) : A(1);
    wave_product<T, P, FULL, 2>(R, s, x_e + size_t(y >> 1) * n, part[w], n, 0.0, lane, G5 ? 1 : 0);
  }
  __syncthreads();
  if (w != 8) return;
  // loaded after the barrier: holding the tile across it would raise the
  // kernel's register count past what three 9-wave workgroups per CU allow
  // (staging it in LDS before the barrier measured no faster)
  R.load(block_ptr<T, P>(inv, size_t(x)), lane);
  const int lr = lane >> 3, lc = lane & 7;
  cx<A> pc[T], pr[T], f[T], g[T];
  A npc_im[T], npr_re[T];
#pragma unroll
  for (int q = 0; q < T; ++q) {
    const int col = lc * T + q;
    cx<VR> t = mk(VR(0), VR(0));
    if (FULL || col < n) {
      t = part[0][col];
#pragma unroll
      for (int k = 1; k < 8; ++k) {
        t.re += part[k][col].re;
        t.im += part[k][col].im;
      }
    }
    pc[q] = mk(A(t.re), A(t.im));
    npc_im[q] = -pc[q].im;
    pr[q] = mk(A(0), A(0));
    npr_re[q] = A(0);
    f[q] = mk(A(0), A(0));
    g[q] = mk(A(0), A(0));
  }
  tile_products<T, P, true, false>(R, pc, npc_im, pr, npr_re, f, g);
  const A s = (P == P16S) ? A(invsc[x]) : A(1);
#pragma unroll
  for (int q = 0; q < T; ++q) {
    f[q].re = sum_row8(f[q].re) * s;
    f[q].im = sum_row8(f[q].im) * s;
  }
  if (lc != 0) return;
#pragma unroll
  for (int q = 0; q < T; ++q) {
    const int row = lr * T + q;
    if (FULL || row < n) t_o[size_t(r) * n + row] = mk(VR(f[q].re), VR(f[q].im));
  }
}

// Epilogue of the reduced operator on one entry i of its output (t = the
// operator applied to the input at i; e = v, the apply's chain input, where
// it is read):
//   EPI 0: out = t
//   EPI 1: p = e - ca t; out = p; y = c0 e + cb p       (first chain step)
//   EPI 2: p = out - ca t; out = p; y += cb p            (later chain steps)
//   EPI 3: out = e - t                                    (residual, e = b)
template <int EPI, typename VR>
__device__ __forceinline__ void reduced_epilogue(size_t i, cx<VR> t, cx<VR>* out,
                                                 const cx<VR>* e, cx<VR>* y, z64 c0, z64 ca,
                                                 z64 cb) {
  if (EPI == 0) {
    out[i] = t;
  } else if (EPI == 3) {
    const cx<VR> bb = e[i];
    out[i] = mk(VR(bb.re - t.re), VR(bb.im - t.im));
  } else {
    const VR ar = VR(ca.re), ai = VR(ca.im), br = VR(cb.re), bi = VR(cb.im);
    const cx<VR> base = (EPI == 1) ? e[i] : out[i];
    cx<VR> p = base;
    p.re -= ar * t.re - ai * t.im;
    p.im -= ar * t.im + ai * t.re;
    out[i] = p;
    cx<VR> yv;
    if (EPI == 1) {
      const VR zr = VR(c0.re), zi = VR(c0.im);
      yv.re = zr * base.re - zi * base.im + (br * p.re - bi * p.im);
      yv.im = zr * base.im + zi * base.re + (br * p.im + bi * p.re);
    } else {
      yv = y[i];
      yv.re += br * p.re - bi * p.im;
      yv.im += br * p.im + bi * p.re;
    }
    y[i] = yv;
  }
}

// s = A_e x_e - D_eo t_o (A_e x_e omitted when x_e is null), workgroup per
// even row r (site x = esite[r]): wave 0 the self block, waves 1-4 the forward
// hops B[x,mu] t_o(x+mu), waves 5-8 the backward hops Gamma5 B[x-mu,mu]^H
// Gamma5 t_o(x-mu), both negated; summed in that order.
// BJ (left block Jacobi with B = D_ee, Sec. 3.2): s = x_e - A_e^{-1} D_eo t_o
// = B^{-1} (A_e x_e - D_eo t_o); wave 0 loads the inverse of x's self block
// (einv, same tiled layout, indexed by site) before the barrier, in place of
// the self block, and applies it to the sum of the eight hop products.
// Epilogue on row r: reduced_epilogue<EPI> (EPI 3 only without BJ).
template <int T, int P, bool FULL, int EPI, bool BJ, bool G5>
__global__ __launch_bounds__(64 * kRedWaves) void k_reduced_eo(
    const void* __restrict__ blocks, const float* __restrict__ scales,
    const void* __restrict__ einv, const float* __restrict__ einvsc,
    const cx<typename VecOf<P>::R>* x_e, const cx<typename VecOf<P>::R>* __restrict__ t_o,
    const int* __restrict__ nbr, const int* __restrict__ esite, int V, int n, int chunk, double tm,
    cx<typename VecOf<P>::R>* out, const cx<typename VecOf<P>::R>* e, cx<typename VecOf<P>::R>* y,
    z64 c0, z64 ca, z64 cb, const int* __restrict__ done) {
  using A = typename Tile<T, P>::A;
  using VR = typename VecOf<P>::R;
  __shared__ cx<VR> part[kRedWaves][64];
  // BJ with FP32 / FP16 tiles: wave 0 stages the inverse in LDS before the
  // barrier (18 / 9 KB at n = 48); holding it in registers across the barrier
  // would cost a third of the resident workgroups.  FP64 tiles (37 KB) are
  // loaded after the barrier instead.
  constexpr bool STAGE = BJ && P != P64;
  constexpr int SU = STAGE ? Tile<T, P>::UNITS * 64 : 1;
  __shared__ uint4 inv_lds[SU];
  if (done && *done) return;
  const int b = blockIdx.x;
  const int r = (b & 7) * chunk + (b >> 3);
  if (r >= (V >> 1)) return;
  const int x = esite[r];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  TileRegs<T, P> R;
  if (w == 0) {
    if (STAGE) {
      const uint4* src = block_ptr<T, P>(einv, size_t(x));
#pragma unroll
      for (int u = 0; u < Tile<T, P>::UNITS; ++u) inv_lds[u * 64 + lane] = src[u * 64 + lane];
    } else if (BJ) {
      // FP64: loaded after the barrier
    } else if (x_e) {
      const int item = 5 * x;
      R.load(block_ptr<T, P>(blocks, size_t(item)), lane);
      const A s = (P == P16S) ? A(scales[item]) : A(1);
      wave_product<T, P, FULL, 0>(R, s, x_e + size_t(r) * n, part[0], n, tm, lane, G5 ? 1 : 0);
    } else {
      for (int i = lane; i < n; i += 64) part[0][i] = mk(VR(0), VR(0));
    }
  } else if (w < 5) {
    const int mu = w - 1;
    const int item = 5 * x + 1 + mu;
    R.load(block_ptr<T, P>(blocks, size_t(item)), lane);
    const A s = (P == P16S) ? A(scales[item]) : A(1);
    const int src = nbr[mu * V + x];
    wave_product<T, P, FULL, 1>(R, -s, t_o + size_t(src >> 1) * n, part[w], n, 0.0, lane);
  } else {
    const int mu = w - 5;
    const int yy = nbr[(4 + mu) * V + x];
    const int item = 5 * yy + 1 + mu;
    R.load(block_ptr<T, P>(blocks, size_t(item)), lane);
    const A s = (P == P16S) ? A(scales[item]) : A(1);
    wave_product<T, P, FULL, 2>(R, -s, t_o + size_t(yy >> 1) * n, part[w], n, 0.0, lane);
  }
  __syncthreads();
  if (w != 0) return;
  if constexpr (BJ) {
    if (STAGE) R.load(inv_lds, lane);
    else R.load(block_ptr<T, P>(einv, size_t(x)), lane);
    const int lr = lane >> 3, lc = lane & 7;
    cx<A> pc[T], pr[T], f[T], g[T];
    A npc_im[T], npr_re[T];
#pragma unroll
    for (int q = 0; q < T; ++q) {
      const int col = lc * T + q;
      cx<VR> t = mk(VR(0), VR(0));
      if (FULL || col < n) {
        t = part[1][col];
#pragma unroll
        for (int k = 2; k < kRedWaves; ++k) {
          t.re += part[k][col].re;
          t.im += part[k][col].im;
        }
      }
      pc[q] = mk(A(t.re), A(t.im));
      npc_im[q] = -pc[q].im;
      pr[q] = mk(A(0), A(0));
      npr_re[q] = A(0);
      f[q] = mk(A(0), A(0));
      g[q] = mk(A(0), A(0));
    }
    tile_products<T, P, true, false>(R, pc, npc_im, pr, npr_re, f, g);
    const A s = (P == P16S) ? A(einvsc[x]) : A(1);
    // the row sums leave row lr*T + q's value in all eight lanes of row group
    // lr; lane lc takes row lr*T + lc
    cx<A> mine = mk(A(0), A(0));
#pragma unroll
    for (int q = 0; q < T; ++q) {
      const A fr = sum_row8(f[q].re) * s, fi = sum_row8(f[q].im) * s;
      if (q == lc) mine = mk(fr, fi);
    }
    const int row = lr * T + lc;
    if (lc >= T || !(FULL || row < n)) return;
    const size_t i = size_t(r) * n + row;
    cx<VR> t = mk(VR(mine.re), VR(mine.im));
    if (x_e) {
      const cx<VR> xv = x_e[i];
      const VR sx = VR((G5 && row >= (n >> 1)) ? -1 : 1);
      t.re += sx * xv.re;
      t.im += sx * xv.im;
    }
    if (G5 && row >= (n >> 1)) t = mk(-t.re, -t.im);
    reduced_epilogue<EPI>(i, t, out, e, y, c0, ca, cb);
  } else {
    for (int c = lane; c < n; c += 64) {
      cx<VR> t = part[0][c];
#pragma unroll
      for (int k = 1; k < kRedWaves; ++k) {
        t.re += part[k][c].re;
        t.im += part[k][c].im;
      }
      if (G5 && c >= (n >> 1)) t = mk(-t.re, -t.im);
      reduced_epilogue<EPI>(size_t(r) * n + c, t, out, e, y, c0, ca, cb);
    }
  }
}

// Single-read form of the same operator.  Each hop block couples exactly one
// odd and one even site, so the odd row's workgroup can apply it in both
// directions while it holds it: k_reduced_scatter forms t_o(x) as k_reduced_oe
// does (same products, same order), keeps the eight hop tiles in registers
// across the barriers, and then applies each of them the other way to t_o(x),
// which gives one of the eight D_eo products of the even neighbour it couples
// to.  Those go to hp[row][slot][n] of that even row: slots 0-3 its forward hops
// B[e,mu] t_o(e+mu), 4-7 its backward hops Gamma5 B[e-mu,mu]^H Gamma5 t_o(e-mu);
// every (row, slot) has exactly one writer.  k_reduced_gather then sums the
// eight slots in that order and finishes the row with A_e (or A_e^{-1} for
// block Jacobi) and the epilogue.  Per site pair ten blocks are read instead
// of eighteen; the sums and signs are those of the two-kernel form, so the
// results agree with it bit for bit.
//
// Eight waves per workgroup, one per hop tile; the inverse, and the tiles of operators
// beyond the last-level cache (FP16 ones of any), are loaded non-temporally (one
// launch reads each once).  The odd site's inverse tile is
// staged in LDS and its product with the summed hop products is split over the
// eight waves: wave w takes rows w T .. w T + T - 1, which lane group lr = w
// holds in the one-wave tile layout; its lane (a, lc) forms the partial sum
// that lane (w, lc) forms for row a there, and the same row reduction over lc
// finishes it.  FP16 tiles up to n = 48 fit three workgroups per CU (7 waves
// per SIMD, 70 registers, no spill); at 8 waves per SIMD the registers spill
// and the kernel runs slower.  FP64 tiles of n = 48 take 202 registers, one
// workgroup per CU: its 330 KB of loads are all in flight at once, so the CUs
// that wait on loads keep HBM busy while others multiply.  HBM bound: 12^4,
// n = 48, one apply with the gather: FP64 1179 us (two-kernel form) -> 752 us,
// 5.1 TB/s of algorithmic bytes; FP32 580 -> 340 us, 5.6 TB/s; ragged n = 42,
// FP64: 1605 -> 762 us.
template <int T, int P>
constexpr int scatter_min_waves() { return (P == P16S && T <= 6) ? 7 : 1; }

template <int T, int P, bool FULL, bool G5, bool NT>
__global__ __launch_bounds__(512, (scatter_min_waves<T, P>())) void k_reduced_scatter(
    const void* __restrict__ blocks, const float* __restrict__ scales,
    const void* __restrict__ inv, const float* __restrict__ invsc,
    const cx<typename VecOf<P>::R>* __restrict__ x_e, cx<typename VecOf<P>::R>* __restrict__ hp,
    const int* __restrict__ nbr, const int* __restrict__ osite, int V, int n, int chunk,
    const int* __restrict__ done) {
  using A = typename Tile<T, P>::A;
  using VR = typename VecOf<P>::R;
  constexpr int UNITS = Tile<T, P>::UNITS;
  __shared__ cx<VR> part[8][64];
  __shared__ cx<VR> tsum[64];
  __shared__ cx<VR> tx[64];
  __shared__ uint4 inv_lds[UNITS * 64];
  if (done && *done) return;
  const int b = blockIdx.x;
  const int r = (b & 7) * chunk + (b >> 3);
  if (r >= (V >> 1)) return;   // uniform per workgroup: no barrier is skipped by part of it
  const int x = osite[r];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  {
    const uint4* ip = block_ptr<T, P>(inv, size_t(x));
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    for (int u = w; u < UNITS; u += 8) {   // read once per launch: non-temporal
      const u32x4 q = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(ip) + u * 64 + lane);
      inv_lds[u * 64 + lane] = make_uint4(q.x, q.y, q.z, q.w);
    }
  }
  TileRegs<T, P> R;
  A s = A(1);
  size_t dst = 0;   // element offset of this wave's D_eo product in hp
  if (w < 4) {
    const int item = 5 * x + 1 + w;
    load_block_tile<T, P>(R, blocks, size_t(item), lane, NT);
    if (P == P16S) s = A(scales[item]);
    const int src = nbr[w * V + x];
    wave_product<T, P, FULL, 1>(R, s, x_e + size_t(src >> 1) * n, part[w], n, 0.0, lane, G5 ? 1 : 0);
    dst = (size_t(src >> 1) * 8 + 4 + w) * n;        // backward hop mu = w of even x + mu
  } else {
    const int mu = w - 4;
    const int y = nbr[(4 + mu) * V + x];
    const int item = 5 * y + 1 + mu;
    load_block_tile<T, P>(R, blocks, size_t(item), lane, NT);
    if (P == P16S) s = A(scales[item]);
    wave_product<T, P, FULL, 2>(R, s, x_e + size_t(y >> 1) * n, part[w], n, 0.0, lane, G5 ? 1 : 0);
    dst = (size_t(y >> 1) * 8 + mu) * n;             // forward hop mu of even x - mu
  }
  __syncthreads();
  if (w == 0) {   // the eight products summed in a fixed order
    cx<VR> t = mk(VR(0), VR(0));
    if (lane < n) {
      t = part[0][lane];
#pragma unroll
      for (int k = 1; k < 8; ++k) {
        t.re += part[k][lane].re;
        t.im += part[k][lane].im;
      }
    }
    tsum[lane] = t;
  }
  __syncthreads();
  {
    // rows w T + a of A_o^{-1} tsum: lane (a, lc) forms sum_c z[wT+a][lc T+c]
    // tsum[lc T + c] over its T columns (the tile element a T + c of layout
    // lane w*8 + lc), the row reduction adds the eight lanes of a row
    const int a = lane >> 3, lc = lane & 7;
    const int src_lane = w * 8 + lc;
    cx<A> f = mk(A(0), A(0));
    if (a < T) {
#pragma unroll
      for (int c = 0; c < T; ++c) {
        const int e = a * T + c;
        const cx<VR> t = tsum[lc * T + c];
        const A pr_ = A(t.re), pi_ = A(t.im);
        A zr, zi;
        if constexpr (P == P16S) {
          const uint4 q = inv_lds[(e >> 2) * 64 + src_lane];
          const uint32_t word = (e & 3) == 0 ? q.x : (e & 3) == 1 ? q.y : (e & 3) == 2 ? q.z : q.w;
          zr = lo_h(word);
          zi = hi_h(word);
        } else if constexpr (P == P64) {
          const double2 q = reinterpret_cast<const double2*>(inv_lds)[e * 64 + src_lane];
          zr = q.x;
          zi = q.y;
        } else {
          const float4 q = reinterpret_cast<const float4*>(inv_lds)[(e >> 1) * 64 + src_lane];
          zr = (e & 1) ? q.z : q.x;
          zi = (e & 1) ? q.w : q.y;
        }
        f.re = fma(zr, pr_, f.re);
        f.re = fma(zi, -pi_, f.re);
        f.im = fma(zr, pi_, f.im);
        f.im = fma(zi, pr_, f.im);
      }
    }
    const A si = (P == P16S) ? A(invsc[x]) : A(1);
    f.re = sum_row8(f.re) * si;
    f.im = sum_row8(f.im) * si;
    if (lc == 0 && a < T) tx[w * T + a] = mk(VR(f.re), VR(f.im));
  }
  __syncthreads();
  if (w < 4)
    wave_product<T, P, FULL, 2>(R, s, tx, hp + dst, n, 0.0, lane);
  else
    wave_product<T, P, FULL, 1>(R, s, tx, hp + dst, n, 0.0, lane);
}

// Second kernel of the single-read form: one wave per even row r (site
// x = esite[r]); its block is loaded non-temporally (read once per launch).  The eight slots of hp[r], negated and summed in slot order,
// are the hop terms k_reduced_eo sums from its own products; the row is then
// finished as there: BJ x_e + A_e^{-1} (sum), else A_e x_e (+ i tm Gamma5 x_e)
// with the terms added one by one, and the epilogue.
template <int T, int P, bool FULL, int EPI, bool BJ, bool G5>
__global__ __launch_bounds__(64) void k_reduced_gather(
    const void* __restrict__ blocks, const float* __restrict__ scales,
    const void* __restrict__ einv, const float* __restrict__ einvsc,
    const cx<typename VecOf<P>::R>* x_e, const cx<typename VecOf<P>::R>* __restrict__ hp,
    const int* __restrict__ esite, int V, int n, int chunk, double tm,
    cx<typename VecOf<P>::R>* out, const cx<typename VecOf<P>::R>* e, cx<typename VecOf<P>::R>* y,
    z64 c0, z64 ca, z64 cb, int stream, const int* __restrict__ done) {
  using A = typename Tile<T, P>::A;
  using VR = typename VecOf<P>::R;
  __shared__ cx<VR> self_part[64];
  __shared__ cx<VR> tsum[64];
  if (done && *done) return;
  const int b = blockIdx.x;
  const int r = (b & 7) * chunk + (b >> 3);
  if (r >= (V >> 1)) return;
  const int x = esite[r];
  const int lane = threadIdx.x;
  TileRegs<T, P> R;
  if (BJ) load_block_tile<T, P>(R, einv, size_t(x), lane, stream);
  cx<VR> h[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    h[k] = mk(VR(0), VR(0));
    if (lane < n) h[k] = hp[(size_t(r) * 8 + k) * n + lane];
  }
  if constexpr (BJ) {
    cx<VR> t = mk(-h[0].re, -h[0].im);
#pragma unroll
    for (int k = 1; k < 8; ++k) {
      t.re += -h[k].re;
      t.im += -h[k].im;
    }
    tsum[lane] = t;
    __syncthreads();
    const int lr = lane >> 3, lc = lane & 7;
    cx<A> pc[T], pr[T], f[T], g[T];
    A npc_im[T], npr_re[T];
#pragma unroll
    for (int q = 0; q < T; ++q) {
      const cx<VR> u = tsum[lc * T + q];
      pc[q] = mk(A(u.re), A(u.im));
      npc_im[q] = -pc[q].im;
      pr[q] = mk(A(0), A(0));
      npr_re[q] = A(0);
      f[q] = mk(A(0), A(0));
      g[q] = mk(A(0), A(0));
    }
    tile_products<T, P, true, false>(R, pc, npc_im, pr, npr_re, f, g);
    const A s = (P == P16S) ? A(einvsc[x]) : A(1);
    cx<A> mine = mk(A(0), A(0));
#pragma unroll
    for (int q = 0; q < T; ++q) {
      const A fr = sum_row8(f[q].re) * s, fi = sum_row8(f[q].im) * s;
      if (q == lc) mine = mk(fr, fi);
    }
    const int row = lr * T + lc;
    if (lc >= T || !(FULL || row < n)) return;
    const size_t i = size_t(r) * n + row;
    cx<VR> o = mk(VR(mine.re), VR(mine.im));
    if (x_e) {
      const cx<VR> xv = x_e[i];
      const VR sx = VR((G5 && row >= (n >> 1)) ? -1 : 1);
      o.re += sx * xv.re;
      o.im += sx * xv.im;
    }
    if (G5 && row >= (n >> 1)) o = mk(-o.re, -o.im);
    reduced_epilogue<EPI>(i, o, out, e, y, c0, ca, cb);
  } else {
    if (x_e) {
      const int item = 5 * x;
      load_block_tile<T, P>(R, blocks, size_t(item), lane, stream);
      const A s = (P == P16S) ? A(scales[item]) : A(1);
      wave_product<T, P, FULL, 0>(R, s, x_e + size_t(r) * n, self_part, n, tm, lane, G5 ? 1 : 0);
    } else {
      self_part[lane] = mk(VR(0), VR(0));
    }
    __syncthreads();
    if (lane >= n) return;
    cx<VR> o = self_part[lane];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      o.re += -h[k].re;
      o.im += -h[k].im;
    }
    if (G5 && lane >= (n >> 1)) o = mk(-o.re, -o.im);
    reduced_epilogue<EPI>(size_t(r) * n + lane, o, out, e, y, c0, ca, cb);
  }
}

// Sum of the 9 slots in a fixed order: self, forward hops, backward hops.
template <typename VR>
__device__ inline cx<VR> gather5(const cx<VR>* __restrict__ gbuf, size_t i, int n) {
  const size_t site = i / n, c = i - site * n;
  const size_t base = site * kSlots * n + c;
  cx<VR> s = gbuf[base + 4 * size_t(n)];
#pragma unroll
  for (int w = 5; w < 9; ++w) {
    const cx<VR> t = gbuf[base + size_t(w) * n];
    s.re += t.re;
    s.im += t.im;
  }
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const cx<VR> t = gbuf[base + size_t(w) * n];
    s.re += t.re;
    s.im += t.im;
  }
  return s;
}

// ------------------------------------------------------------------ block Jacobi
// out_x = M_x t_x with M_x the stored inverse and t either the sum of the 9
// gbuf slots (t = D psi) or a plain vector; one wave per site; epilogue as in
// the gather kernels (0 store, 1 poly_first, 2 poly).
template <int T, int P, bool FULL, bool FROMBUF, int EPI>
__global__ __launch_bounds__(64) void k_block_jacobi(
    const void* __restrict__ blocks, const float* __restrict__ scales,
    const cx<typename VecOf<P>::R>* __restrict__ tin, cx<typename VecOf<P>::R>* out,
    const cx<typename VecOf<P>::R>* vin, cx<typename VecOf<P>::R>* y, int V, int n, int chunk,
    z64 c0, z64 ca, z64 cb, const int* __restrict__ done, const int* __restrict__ rowsite) {
  using A = typename Tile<T, P>::A;
  using VR = typename VecOf<P>::R;
  if (done && *done) return;
  const int b = blockIdx.x;
  const int site = (b & 7) * chunk + (b >> 3);   // row of the vectors
  if (site >= V) return;
  const int blk = rowsite ? rowsite[site] : site;  // block of that row's lattice site
  const int lane = threadIdx.x, lr = lane >> 3, lc = lane & 7;
  const size_t blk_units = size_t(Tile<T, P>::UNITS) * 64;
  TileRegs<T, P> R;
  R.load(static_cast<const uint4*>(blocks) + size_t(blk) * blk_units, lane);
  cx<A> pc[T], pr[T], f[T], g[T];
  A npc_im[T], npr_re[T];
#pragma unroll
  for (int q = 0; q < T; ++q) {
    const int col = lc * T + q;
    cx<A> t = mk(A(0), A(0));
    if (FULL || col < n) {
      if (FROMBUF) {
        const cx<VR> z = gather5(tin, size_t(site) * n + col, n);
        t = mk(A(z.re), A(z.im));
      } else {
        const cx<VR> z = tin[size_t(site) * n + col];
        t = mk(A(z.re), A(z.im));
      }
    }
    pc[q] = t;
    npc_im[q] = -t.im;
    pr[q] = mk(A(0), A(0));
    npr_re[q] = A(0);
    f[q] = mk(A(0), A(0));
    g[q] = mk(A(0), A(0));
  }
  tile_products<T, P, true, false>(R, pc, npc_im, pr, npr_re, f, g);
  A s = A(1);
  if (P == P16S) s = A(scales[blk]);
#pragma unroll
  for (int q = 0; q < T; ++q) {
    f[q].re = sum_row8(f[q].re) * s;
    f[q].im = sum_row8(f[q].im) * s;
  }
  if (lc != 0) return;
#pragma unroll
  for (int q = 0; q < T; ++q) {
    const int row = lr * T + q;
    if (!(FULL || row < n)) continue;
    const size_t i = size_t(site) * n + row;
    const VR sr = VR(f[q].re), si = VR(f[q].im);
    if (EPI == 0) {
      out[i] = mk(sr, si);
    } else {
      const cx<VR> base = (EPI == 1) ? vin[i] : out[i];
      cx<VR> p = base;
      p.re -= VR(ca.re) * sr - VR(ca.im) * si;
      p.im -= VR(ca.re) * si + VR(ca.im) * sr;
      out[i] = p;
      cx<VR> yy = (EPI == 1) ? mk(VR(VR(c0.re) * base.re - VR(c0.im) * base.im),
                                  VR(VR(c0.re) * base.im + VR(c0.im) * base.re))
                             : y[i];
      yy.re += VR(cb.re) * p.re - VR(cb.im) * p.im;
      yy.im += VR(cb.re) * p.im + VR(cb.im) * p.re;
      y[i] = yy;
    }
  }
}

// ------------------------------------------------------------------ batched chain step
// For r < R (device pointer arrays): first step (first != 0):
//   prod_r = v_r - ca t_r;  y_r = c0 v_r + cb prod_r,
// later steps: prod_r -= ca t_r;  y_r += cb prod_r  (t_r = A~ of the chain input).
template <typename VR>
__device__ __forceinline__ void chain_multi_body(const cx<VR>* const* __restrict__ t,
                                                 const cx<VR>* const* __restrict__ v,
                                                 cx<VR>* const* __restrict__ prod,
                                                 cx<VR>* const* __restrict__ y, size_t N, z64 c0,
                                                 z64 ca, z64 cb, int first, int r) {
  const cx<VR>* tr = t[r];
  cx<VR>* pr = prod[r];
  cx<VR>* yr = y[r];
  const VR ar = VR(ca.re), ai = VR(ca.im), br = VR(cb.re), bi = VR(cb.im);
  const VR zr = VR(c0.re), zi = VR(c0.im);
  const size_t stride = size_t(gridDim.x) * blockDim.x;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < N; i += stride) {
    const cx<VR> s = tr[i];
    const cx<VR> base = first ? v[r][i] : pr[i];
    cx<VR> p = base;
    p.re -= ar * s.re - ai * s.im;
    p.im -= ar * s.im + ai * s.re;
    pr[i] = p;
    cx<VR> yy = first ? mk(VR(zr * base.re - zi * base.im), VR(zr * base.im + zi * base.re)) : yr[i];
    yy.re += br * p.re - bi * p.im;
    yy.im += br * p.im + bi * p.re;
    yr[i] = yy;
  }
}

template <typename VR>
__global__ void k_chain_multi(const cx<VR>* const* __restrict__ t, const cx<VR>* const* __restrict__ v,
                              cx<VR>* const* __restrict__ prod, cx<VR>* const* __restrict__ y,
                              size_t N, z64 c0, z64 ca, z64 cb, int first) {
  chain_multi_body<VR>(t, v, prod, y, N, c0, ca, cb, first, blockIdx.y);
}

// The chain step of several operators' column sets in one launch: blockIdx.z
// is the operator, blockIdx.y its column (elementwise, so any grid gives the
// per-operator launches' results).
template <typename VR>
__global__ void k_chain_groups(ChainGroups g, int first) {
  const int gi = int(blockIdx.z), r = int(blockIdx.y);
  if (gi >= g.count || r >= g.R[gi]) return;
  chain_multi_body<VR>(static_cast<const cx<VR>* const*>(g.t[gi]),
                       static_cast<const cx<VR>* const*>(g.v[gi]),
                       static_cast<cx<VR>* const*>(g.prod[gi]), static_cast<cx<VR>* const*>(g.y[gi]),
                       g.N[gi], g.c0[gi], g.ca[gi], g.cb[gi], first, r);
}

template <typename VR>
__global__ void k_gather_store(const cx<VR>* __restrict__ gbuf, cx<VR>* __restrict__ out,
                               size_t N, int n, const int* __restrict__ done) {
  if (done && *done) return;
  const size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= N) return;
  out[i] = gather5(gbuf, i, n);
}

template <typename VR>
__global__ void k_gather_poly(const cx<VR>* __restrict__ gbuf, cx<VR>* __restrict__ prod,
                              cx<VR>* __restrict__ y, size_t N, int n, z64 ca, z64 cb,
                              const int* __restrict__ done) {
  if (done && *done) return;
  const size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= N) return;
  const cx<VR> s = gather5(gbuf, i, n);
  cx<VR> p = prod[i];
  const VR ar = VR(ca.re), ai = VR(ca.im), br = VR(cb.re), bi = VR(cb.im);
  p.re -= ar * s.re - ai * s.im;
  p.im -= ar * s.im + ai * s.re;
  prod[i] = p;
  cx<VR> yy = y[i];
  yy.re += br * p.re - bi * p.im;
  yy.im += br * p.im + bi * p.re;
  y[i] = yy;
}

template <typename VR>
__global__ void k_gather_poly_first(const cx<VR>* __restrict__ gbuf, const cx<VR>* __restrict__ v,
                                    cx<VR>* __restrict__ prod, cx<VR>* __restrict__ y, size_t N,
                                    int n, z64 c0, z64 ca, z64 cb, const int* __restrict__ done) {
  if (done && *done) return;
  const size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= N) return;
  const cx<VR> s = gather5(gbuf, i, n);
  const cx<VR> vv = v[i];
  cx<VR> p = vv;
  const VR ar = VR(ca.re), ai = VR(ca.im), br = VR(cb.re), bi = VR(cb.im);
  const VR zr = VR(c0.re), zi = VR(c0.im);
  p.re -= ar * s.re - ai * s.im;
  p.im -= ar * s.im + ai * s.re;
  prod[i] = p;
  cx<VR> yy;
  yy.re = zr * vv.re - zi * vv.im + (br * p.re - bi * p.im);
  yy.im = zr * vv.im + zi * vv.re + (br * p.im + bi * p.re);
  y[i] = yy;
}

template <typename VR>
__global__ void k_gather_resid(const cx<VR>* __restrict__ gbuf, const cx<VR>* __restrict__ b,
                               cx<VR>* __restrict__ out, size_t N, int n, Reducer red,
                               double* result) {
  double acc[1] = {0.0};
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < N;
       i += size_t(gridDim.x) * blockDim.x) {
    const cx<VR> s = gather5(gbuf, i, n);
    const cx<VR> bb = b[i];
    const cx<VR> r = mk(VR(bb.re - s.re), VR(bb.im - s.im));
    out[i] = r;
    acc[0] += double(r.re) * double(r.re) + double(r.im) * double(r.im);
  }
  block_partials<1>(acc, red.partials);
}

// ------------------------------------------------------------------ odd-even split
template <typename VR>
__global__ void k_oddeven_split(int n, int H, const int* __restrict__ esite,
                                const int* __restrict__ osite, cx<VR>* full, cx<VR>* ve,
                                cx<VR>* vo, int dir) {
  const size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= size_t(H) * n) return;
  const int r = int(i / n), c = int(i % n);
  const size_t fe = size_t(esite[r]) * n + c, fo = size_t(osite[r]) * n + c;
  if (dir == 0) {
    if (ve) ve[i] = full[fe];
    if (vo) vo[i] = full[fo];
  } else {
    full[fe] = ve ? ve[i] : mk(VR(0), VR(0));
    full[fo] = vo ? vo[i] : mk(VR(0), VR(0));
  }
}

// ------------------------------------------------------------------ gradient
// d S / d B[x, dir]: the n x n outer products of a site and its neighbour, bound by the
// writes.  Thread (i, j), i < rows = min(256 / n, n), keeps column j for every rows-th row,
// so its neighbour entries are read once and nothing is divided in the loop; threads
// past the rows end at once.  inv = 65536 / n + 1 divides a thread number by n exactly.
// Measured, us, with a division per entry / now: 8^4 tied n = 32 (268 MB) 50.6 / 48.3
// in the kernel (5.6 TB/s; non-temporal stores: 51); calls of 1,800 sites tied n = 20 12.0 /
// 10.8, n = 26 17.1 / 15.0, 4,096 sites untied n = 10 13.7 / 14.0 (18.0 with threads past the rows
// loading, and the rows' entries loaded after the neighbour's).
__global__ __launch_bounds__(256) void k_grad_hops(const z64* __restrict__ lam,
                                                   const z64* __restrict__ x,
                                                   z64* __restrict__ grad,
                                                   const int* __restrict__ nbr, int V, int n,
                                                   int tied, int rows, unsigned inv) {
  typedef double d2 __attribute__((ext_vector_type(2)));
  const int site = blockIdx.x;
  const int dir = blockIdx.y;  // 0..7 untied, 0..3 tied
  const int i0 = int(threadIdx.x * inv) >> 16, j = int(threadIdx.x) - i0 * n;
  if (i0 >= rows) return;
  // the rows' own entries are loaded a row ahead, the first ones beside the neighbour's
  const z64 *ls = lam + size_t(site) * n, *xs = x + size_t(site) * n;
  z64 l = ls[i0], xx = tied ? xs[i0] : mk(0.0, 0.0);
  const int y = nbr[dir * V + site];
  d2* out = reinterpret_cast<d2*>(grad) + (size_t(site) * (tied ? 4 : 8) + dir) * (size_t(n) * n) + j;
  const z64 xv = x[size_t(y) * n + j];
  const z64 ly = tied ? lam[size_t(y) * n + j] : mk(0.0, 0.0);
  const double gj = gam(j, n);
  for (int i = i0; i < n; i += rows) {
    const z64 li = l, xi = xx;
    if (i + rows < n) {
      l = ls[i + rows];
      if (tied) xx = xs[i + rows];
    }
    // -lambda_x,i * conj(x_y,j)
    double gr = -(li.re * xv.re + li.im * xv.im);
    double gi = -(li.im * xv.re - li.re * xv.im);
    if (tied) {
      // - g5_i x_x,i conj(lambda_y,j) g5_j
      const double s = gam(i, n) * gj;
      gr -= s * (xi.re * ly.re + xi.im * ly.im);
      gi -= s * (xi.im * ly.re - xi.re * ly.im);
    }
    out[size_t(i) * n] = d2{gr, gi};
  }
}

}  // namespace

// ====================================================================== launchers

void launch_neighbours(int* nbr, int L0, int L1, int L2, int L3, hipStream_t st) {
  const int V = L0 * L1 * L2 * L3;
  hipLaunchKernelGGL(k_neighbours, dim3((V + 255) / 256), dim3(256), 0, st, nbr, L0, L1, L2, L3);
  DC_HIP(hipGetLastError());
}

// bytes per complex block entry
constexpr size_t block_entry(int p) { return p == P64 ? 16 : p == P32 ? 8 : 4; }

// Blocks beyond the 256 MB last-level cache are loaded non-temporally: a pass
// evicts them before the next one comes, and past the caches they leave those to the
// slots.  Within it a repeated apply finds them there, unless the loads say that
// they are not reused (one apply, cached / non-temporal, us; n = 48 but for the first):
// 80 MB FP64 n = 16 18.9 / 21.1, 180 MB FP16 36.2 / 42.5, 360 MB FP32 78.5 / 68.4,
// 720 MB FP64 157 / 141, 2.9 GB FP16 659 / 626, 5.8 GB FP32 1202 / 1084.  At 270 MB what a pass
// leaves there still helps FP64 (n = 24 53.5 / 57.1, n = 16 57.0 / 59.3), not FP32 (n = 16 64.1 /
// 60.7) or FP16 (n = 32 63.2 / 61.8): FP64's line is 288 MB.
constexpr size_t kCacheBytes = size_t(256) << 20;

template <int P>
static void apply_T(int n, int V, const void* blocks, const float* scales, const void* in,
                    void* gbuf, const int* nbr, double tm, const int* done, hipStream_t st,
                    hipEvent_t ev0, hipEvent_t ev1, int g5) {
  using VR = typename VecOf<P>::R;
  const int chunk = (5 * V + 7) / 8;
  const dim3 grid(unsigned(chunk) * 8u), block(64);
  const auto* pin = static_cast<const cx<VR>*>(in);
  auto* pg = static_cast<cx<VR>*>(gbuf);
  const size_t fits = P == P64 ? kCacheBytes + kCacheBytes / 8 : kCacheBytes;
  const int stream = size_t(V) * 5 * n * n * block_entry(P) > fits;
  const bool full = (n % 8) == 0;
  switch (tile_T(n)) {
  // with events: the dispatch itself records its start and end (no marker packets)
#define DC_CASE(TV)                                                                            \
  case TV: {                                                                                   \
    const auto k = full ? (g5 ? k_apply_blocks<TV, P, true, true> : k_apply_blocks<TV, P, true, false>)\
                        : (g5 ? k_apply_blocks<TV, P, false, true> : k_apply_blocks<TV, P, false, false>);\
    hipExtLaunchKernelGGL(k, grid, block, 0, st, ev0, ev1, 0, blocks, scales, pin, pg, nbr, V, \
                          n, chunk, tm, stream, done);                                         \
    break;                                                                                     \
  }
    DC_CASE(1) DC_CASE(2) DC_CASE(3) DC_CASE(4) DC_CASE(5) DC_CASE(6) DC_CASE(7) DC_CASE(8)
#undef DC_CASE
    default:
      throw InvalidArg("block size n > 64 is not supported");
  }
  DC_HIP(hipGetLastError());
}

void launch_apply_blocks(Prec p, int n, int V, const void* blocks, const float* scales,
                         const void* in, void* gbuf, const int* nbr, double tm, const int* done,
                         hipStream_t st, hipEvent_t ev0, hipEvent_t ev1, int g5) {
  if (p == P64) apply_T<P64>(n, V, blocks, scales, in, gbuf, nbr, tm, done, st, ev0, ev1, g5);
  else if (p == P32) apply_T<P32>(n, V, blocks, scales, in, gbuf, nbr, tm, done, st, ev0, ev1, g5);
  else apply_T<P16S>(n, V, blocks, scales, in, gbuf, nbr, tm, done, st, ev0, ev1, g5);
}

// The one-launch form reads every hop block twice and takes nine waves a site: it is the
// faster one while that costs less than a second launch and the slots' way through the
// caches, so up to the eight 4 MB L2s of tiled blocks (one apply, two launches / one, us):
// 5 MB FP64 11.1 / 8.6, 20 MB FP16 11.1 / 8.7, 28 MB FP32 11.0 / 8.5; 40 MB FP64 11.7 / 12.4, 42
// MB FP64 n = 12 (22 MB of entries) 11.7 / 13.7; and up to 16 workgroups per CU, beyond
// which their number is what it waits for: 4,096 sites FP64 n = 8 11.2 / 10.4, FP32 n = 8
// 11.0 / 8.7; 6,144 sites 12.4 / 18.2 and 11.4 / 11.6, 16,384 sites n = 2 22 / 46 and 22 / 28.
constexpr size_t kSiteBytes = size_t(32) << 20;
constexpr int kSiteMax = 4096;

// Tiles it takes: FP64 tiles of T >= 6 would spill (nine waves: 168 registers each).
template <int P>
constexpr bool site_tile(int T) { return T >= 1 && T <= (P == P64 ? 5 : 8); }

bool apply_one_launch(Prec p, int n, int V) {
  if ((p == P64 && !site_tile<P64>(tile_T(n))) || V > kSiteMax) return false;
  const size_t edge = size_t(tile_T(n)) * 8;
  return size_t(V) * 5 * edge * edge * block_entry(p) <= kSiteBytes;
}

template <int P>
static void site_T(int n, int V, const void* blocks, const float* scales, const void* in, void* out,
                   const int* nbr, double tm, const int* done, hipStream_t st, hipEvent_t ev0,
                   hipEvent_t ev1, int g5) {
  using VR = typename VecOf<P>::R;
  const int chunk = (V + 7) / 8;
  const dim3 grid(unsigned(chunk) * 8u), block(64 * kRedWaves);
  const auto* pin = static_cast<const cx<VR>*>(in);
  auto* po = static_cast<cx<VR>*>(out);
  const bool full = (n % 8) == 0;
  const int g = g5 ? 3 : 0;
  switch (tile_T(n)) {
#define DC_CASE(TV)                                                                          \
  case TV:                                                                                   \
    if constexpr (site_tile<P>(TV)) {                                                        \
      if (full)                                                                              \
        hipExtLaunchKernelGGL((k_apply_site<TV, P, true>), grid, block, 0, st, ev0, ev1, 0,  \
                              blocks, scales, pin, po, nbr, V, n, chunk, tm, g, done);       \
      else                                                                                   \
        hipExtLaunchKernelGGL((k_apply_site<TV, P, false>), grid, block, 0, st, ev0, ev1, 0, \
                              blocks, scales, pin, po, nbr, V, n, chunk, tm, g, done);       \
    }                                                                                        \
    break;
    DC_CASE(1) DC_CASE(2) DC_CASE(3) DC_CASE(4) DC_CASE(5) DC_CASE(6) DC_CASE(7) DC_CASE(8)
#undef DC_CASE
    default:
      throw InvalidArg("block size n > 64 is not supported");
  }
  DC_HIP(hipGetLastError());
}

void launch_apply_site(Prec p, int n, int V, const void* blocks, const float* scales, const void* in,
                       void* out, const int* nbr, double tm, const int* done, hipStream_t st,
                       hipEvent_t ev0, hipEvent_t ev1, int g5) {
  if (p == P64 && !site_tile<P64>(tile_T(n)))
    throw InvalidArg("the one-launch apply does not take this block size in FP64");
  if (p == P64) site_T<P64>(n, V, blocks, scales, in, out, nbr, tm, done, st, ev0, ev1, g5);
  else if (p == P32) site_T<P32>(n, V, blocks, scales, in, out, nbr, tm, done, st, ev0, ev1, g5);
  else site_T<P16S>(n, V, blocks, scales, in, out, nbr, tm, done, st, ev0, ev1, g5);
}

template <int P, bool FROMBUF, int EPI>
static void bj_T(int n, int V, const void* blocks, const float* scales, const void* tin, void* out,
                 const void* vin, void* y, z64 c0, z64 ca, z64 cb, const int* done,
                 hipStream_t st, const int* rowsite = nullptr) {
  using VR = typename VecOf<P>::R;
  const int chunk = (V + 7) / 8;
  const dim3 grid(unsigned(chunk) * 8u), block(64);
  const auto* ti = static_cast<const cx<VR>*>(tin);
  auto* o = static_cast<cx<VR>*>(out);
  const auto* vi = static_cast<const cx<VR>*>(vin);
  auto* yy = static_cast<cx<VR>*>(y);
  const bool full = (n % 8) == 0;
  switch (tile_T(n)) {
#define DC_CASE(TV)                                                                              \
  case TV:                                                                                       \
    if (full)                                                                                    \
      hipLaunchKernelGGL((k_block_jacobi<TV, P, true, FROMBUF, EPI>), grid, block, 0, st, blocks, \
                         scales, ti, o, vi, yy, V, n, chunk, c0, ca, cb, done, rowsite);         \
    else                                                                                         \
      hipLaunchKernelGGL((k_block_jacobi<TV, P, false, FROMBUF, EPI>), grid, block, 0, st,       \
                         blocks, scales, ti, o, vi, yy, V, n, chunk, c0, ca, cb, done, rowsite); \
    break;
    DC_CASE(1) DC_CASE(2) DC_CASE(3) DC_CASE(4) DC_CASE(5) DC_CASE(6) DC_CASE(7) DC_CASE(8)
#undef DC_CASE
    default:
      throw InvalidArg("block size n > 64 is not supported");
  }
  DC_HIP(hipGetLastError());
}

template <bool FROMBUF, int EPI>
static void bj_P(Prec p, int n, int V, const void* blocks, const float* scales, const void* tin,
                 void* out, const void* vin, void* y, z64 c0, z64 ca, z64 cb, const int* done,
                 hipStream_t st, const int* rowsite = nullptr) {
  if (p == P64) bj_T<P64, FROMBUF, EPI>(n, V, blocks, scales, tin, out, vin, y, c0, ca, cb, done, st, rowsite);
  else if (p == P32) bj_T<P32, FROMBUF, EPI>(n, V, blocks, scales, tin, out, vin, y, c0, ca, cb, done, st, rowsite);
  else bj_T<P16S, FROMBUF, EPI>(n, V, blocks, scales, tin, out, vin, y, c0, ca, cb, done, st, rowsite);
}

void launch_bj_vec(Prec p, int n, int V, const void* inv, const float* scales, const void* in,
                   void* out, hipStream_t st) {
  const z64 z = mk(0.0, 0.0);
  bj_P<false, 0>(p, n, V, inv, scales, in, out, nullptr, nullptr, z, z, z, nullptr, st);
}

void launch_bj_gather_store(Prec p, int n, int V, const void* inv, const float* scales,
                            const void* gbuf, void* out, const int* done, hipStream_t st) {
  const z64 z = mk(0.0, 0.0);
  bj_P<true, 0>(p, n, V, inv, scales, gbuf, out, nullptr, nullptr, z, z, z, done, st);
}

void launch_bj_rows(Prec p, int n, int rows, const int* rowsite, const void* inv,
                    const float* scales, const void* in, void* out, hipStream_t st) {
  const z64 z = mk(0.0, 0.0);
  bj_P<false, 0>(p, n, rows, inv, scales, in, out, nullptr, nullptr, z, z, z, nullptr, st, rowsite);
}

template <int P>
static void reduced_oe_T(int n, int V, const void* blocks, const float* scales, const void* inv,
                         const float* invsc, const void* x_e, void* t_o, const int* nbr,
                         const int* osite, const int* done, hipStream_t st, hipEvent_t ev0,
                         hipEvent_t ev1, int g5) {
  using VR = typename VecOf<P>::R;
  const int rows = V / 2;
  const int chunk = (rows + 7) / 8;
  const dim3 grid(unsigned(chunk) * 8u), block(64 * kRedWaves);
  const auto* xe = static_cast<const cx<VR>*>(x_e);
  auto* to = static_cast<cx<VR>*>(t_o);
  const bool full = (n % 8) == 0;
  switch (tile_T(n)) {
#define DC_CASE(TV)                                                                            \
  case TV: {                                                                                   \
    const auto k = full ? (g5 ? k_reduced_oe<TV, P, true, true> : k_reduced_oe<TV, P, true, false>)\
                        : (g5 ? k_reduced_oe<TV, P, false, true> : k_reduced_oe<TV, P, false, false>);\
    hipExtLaunchKernelGGL(k, grid, block, 0, st, ev0, ev1, 0, blocks, scales, inv, invsc, xe,  \
                          to, nbr, osite, V, n, chunk, done);                                  \
    break;                                                                                     \
  }
    DC_CASE(1) DC_CASE(2) DC_CASE(3) DC_CASE(4) DC_CASE(5) DC_CASE(6) DC_CASE(7) DC_CASE(8)
#undef DC_CASE
    default:
      throw InvalidArg("block size n > 64 is not supported");
  }
  DC_HIP(hipGetLastError());
}

void launch_reduced_oe(Prec p, int n, int V, const void* blocks, const float* scales,
                       const void* inv, const float* invsc, const void* x_e, void* t_o,
                       const int* nbr, const int* osite, const int* done, hipStream_t st,
                       hipEvent_t ev0, hipEvent_t ev1, int g5) {
  if (V < 2 || V % 2) throw InvalidArg("the reduced operator needs an even number of sites");
  if (p == P64) reduced_oe_T<P64>(n, V, blocks, scales, inv, invsc, x_e, t_o, nbr, osite, done, st, ev0, ev1, g5);
  else if (p == P32) reduced_oe_T<P32>(n, V, blocks, scales, inv, invsc, x_e, t_o, nbr, osite, done, st, ev0, ev1, g5);
  else reduced_oe_T<P16S>(n, V, blocks, scales, inv, invsc, x_e, t_o, nbr, osite, done, st, ev0, ev1, g5);
}

template <int P, int EPI, bool BJ>
static void reduced_eo_T(int n, int V, const void* blocks, const float* scales, const void* einv,
                         const float* einvsc, const void* x_e, const void* t_o, const int* nbr,
                         const int* esite, double tm, void* out, const void* e, void* y, z64 c0,
                         z64 ca, z64 cb, const int* done, hipStream_t st, hipEvent_t ev0,
                         hipEvent_t ev1, int g5) {
  using VR = typename VecOf<P>::R;
  const int rows = V / 2;
  const int chunk = (rows + 7) / 8;
  const dim3 grid(unsigned(chunk) * 8u), block(64 * kRedWaves);
  const auto* xe = static_cast<const cx<VR>*>(x_e);
  const auto* to = static_cast<const cx<VR>*>(t_o);
  auto* o = static_cast<cx<VR>*>(out);
  const auto* ee = static_cast<const cx<VR>*>(e);
  auto* yy = static_cast<cx<VR>*>(y);
  const bool full = (n % 8) == 0;
  constexpr bool E0 = EPI == 0;   // Gamma5 comes with the plain store only
  switch (tile_T(n)) {
#define DC_CASE(TV)                                                                       \
  case TV: {                                                                              \
    const auto k = full ? (E0 && g5 ? k_reduced_eo<TV, P, true, EPI, BJ, E0>              \
                                    : k_reduced_eo<TV, P, true, EPI, BJ, false>)          \
                        : (E0 && g5 ? k_reduced_eo<TV, P, false, EPI, BJ, E0>             \
                                    : k_reduced_eo<TV, P, false, EPI, BJ, false>);        \
    hipExtLaunchKernelGGL(k, grid, block, 0, st, ev0, ev1, 0, blocks, scales, einv,       \
                          einvsc, xe, to, nbr, esite, V, n, chunk, tm, o,                 \
                          ee, yy, c0, ca, cb, done);                                      \
    break;                                                                                \
  }
    DC_CASE(1) DC_CASE(2) DC_CASE(3) DC_CASE(4) DC_CASE(5) DC_CASE(6) DC_CASE(7) DC_CASE(8)
#undef DC_CASE
    default:
      throw InvalidArg("block size n > 64 is not supported");
  }
  DC_HIP(hipGetLastError());
}

template <int P>
static void reduced_eo_P(int epi, int n, int V, const void* blocks, const float* scales,
                         const void* einv, const float* einvsc, const void* x_e, const void* t_o,
                         const int* nbr, const int* esite, double tm, void* out, const void* e,
                         void* y, z64 c0, z64 ca, z64 cb, const int* done, hipStream_t st,
                         hipEvent_t ev0, hipEvent_t ev1, int g5) {
#define DC_ARGS n, V, blocks, scales, einv, einvsc, x_e, t_o, nbr, esite, tm, out, e, y, c0, ca, cb, done, st, ev0, ev1, g5
  if (einv) {
    switch (epi) {
      case 0: reduced_eo_T<P, 0, true>(DC_ARGS); break;
      case 1: reduced_eo_T<P, 1, true>(DC_ARGS); break;
      default: reduced_eo_T<P, 2, true>(DC_ARGS); break;
    }
    return;
  }
  switch (epi) {
    case 0: reduced_eo_T<P, 0, false>(DC_ARGS); break;
    case 1: reduced_eo_T<P, 1, false>(DC_ARGS); break;
    case 2: reduced_eo_T<P, 2, false>(DC_ARGS); break;
    default: reduced_eo_T<P, 3, false>(DC_ARGS); break;
  }
#undef DC_ARGS
}

void launch_reduced_eo(Prec p, int epi, int n, int V, const void* blocks, const float* scales,
                       const void* einv, const float* einvsc, const void* x_e, const void* t_o,
                       const int* nbr, const int* esite, double tm, void* out, const void* e,
                       void* y, z64 c0, z64 ca, z64 cb, const int* done, hipStream_t st,
                       hipEvent_t ev0, hipEvent_t ev1, int g5) {
  if (epi < 0 || epi > 3) throw InvalidArg("reduced epilogue must be 0..3");
  if (g5 && epi != 0) throw InvalidArg("Gamma5 comes with the plain store only");
  if (einv && epi == 3) throw InvalidArg("the residual epilogue takes the unpreconditioned operator");
  if (einv && p == P16S && !einvsc) throw InvalidArg("FP16 inverses need their scales");
  if (V < 2 || V % 2) throw InvalidArg("the reduced operator needs an even number of sites");
  if (!t_o || !out) throw InvalidArg("null vector pointer");
  if ((epi == 1 || epi == 3) && !e) throw InvalidArg("null epilogue input");
  if ((epi == 1 || epi == 2) && !y) throw InvalidArg("null chain output");
#define DC_ARGS epi, n, V, blocks, scales, einv, einvsc, x_e, t_o, nbr, esite, tm, out, e, y, c0, ca, cb, done, st, ev0, ev1, g5
  if (p == P64) reduced_eo_P<P64>(DC_ARGS);
  else if (p == P32) reduced_eo_P<P32>(DC_ARGS);
  else reduced_eo_P<P16S>(DC_ARGS);
#undef DC_ARGS
}

namespace {
int g_reduced_mode = 0;
}

void set_reduced_mode(int mode) {
  if (mode < 0 || mode > 1) throw InvalidArg("reduced kernel mode must be 0 or 1");
  g_reduced_mode = mode;
}

int reduced_mode() { return g_reduced_mode; }

// Tiles the single-read form takes: an FP64 tile of T >= 7 (n > 48) would not
// fit the registers of its wave (2 T^2 doubles of 256 VGPRs at eight waves).
template <int P>
constexpr bool single_read_tile(int T) { return T >= 1 && T <= (P == P64 ? 6 : 8); }

static bool single_read_fits(Prec p, int n) {
  const int T = tile_T(n);
  return p == P64 ? single_read_tile<P64>(T) : single_read_tile<P32>(T);
}

// FP64 operators whose blocks stay in the XCDs' L2 (8 x 4 MB) keep the
// two-kernel form: its second read of a hop block is an L2 hit there and its
// workgroups have one barrier instead of three.  Measured (whole FP64 solves,
// two-kernel / single-read): 21 MB of blocks 9.47 / 9.72 ms, 26 MB 13.1 / 12.2,
// 47 MB 14.1 / 12.6; one apply at 12^4, n = 48 (3.8 GB): 1179 / 752 us.
constexpr size_t kSingleReadF64Bytes = size_t(24) << 20;

// FP32 and FP64 tiles are loaded non-temporally where the blocks of an apply do not fit
// the 256 MB last-level cache (a pass leaves enough of them there up to somewhat more).
// Cached / non-temporal, one apply, us: FP32 51 MB n = 8 32.7 / 35.6, 202 MB n = 16 41.9 /
// 49.4, 270 MB n = 16 59.3 / 65.7, 304 MB n = 24 67.1 / 65.6, 506 MB n = 48 99.9 / 93.2; FP64
// 135 MB n = 8 44.0 / 50.0, 270 MB n = 24 48.8 / 52.9, 405 MB n = 24 85.4 / 78.5.  FP16 tiles
// always are: cached they gained between 100 and 200 MB only (190 MB, n = 48: 36.5 / 38.1)
// and lost on either side (60 MB 19.7 / 16.8, 430 MB 90.6 / 81.7).
static int reduced_stream(int p, int n, int V) {
  const size_t edge = size_t(tile_T(n)) * 8;
  return size_t(V) * 5 * edge * edge * block_entry(p) > kCacheBytes + kCacheBytes / 8;
}

bool reduced_single_read(Prec p, int n, int V) {
  if (g_reduced_mode == 1 || !single_read_fits(p, n)) return false;
  return p != P64 || size_t(V) * 5 * n * n * sizeof(z64) > kSingleReadF64Bytes;
}

template <int T, int P, bool FULL, bool G5>
static auto scatter_kernel(int stream) {
  if constexpr (P == P16S) return k_reduced_scatter<T, P, FULL, G5, true>;
  else return stream ? k_reduced_scatter<T, P, FULL, G5, true> : k_reduced_scatter<T, P, FULL, G5, false>;
}

template <int P>
static void reduced_scatter_T(int n, int V, const void* blocks, const float* scales,
                              const void* inv, const float* invsc, const void* x_e, void* hp,
                              const int* nbr, const int* osite, const int* done, hipStream_t st,
                              hipEvent_t ev0, hipEvent_t ev1, int g5) {
  using VR = typename VecOf<P>::R;
  const int rows = V / 2;
  const int chunk = (rows + 7) / 8;
  const dim3 grid(unsigned(chunk) * 8u), block(512);
  const auto* xe = static_cast<const cx<VR>*>(x_e);
  auto* h = static_cast<cx<VR>*>(hp);
  const bool full = (n % 8) == 0;
  const int stream = reduced_stream(P, n, V);
  switch (tile_T(n)) {
#define DC_CASE(TV)                                                                                    \
  case TV:                                                                                             \
    if constexpr (single_read_tile<P>(TV)) {                                                           \
      const auto k =                                                                                   \
          full ? (g5 ? scatter_kernel<TV, P, true, true>(stream) : scatter_kernel<TV, P, true, false>(stream))   \
               : (g5 ? scatter_kernel<TV, P, false, true>(stream) : scatter_kernel<TV, P, false, false>(stream));\
      hipExtLaunchKernelGGL(k, grid, block, 0, st, ev0, ev1, 0, blocks, scales, inv, invsc, xe,        \
                            h, nbr, osite, V, n, chunk, done);                                         \
    }                                                                                                  \
    break;
    DC_CASE(1) DC_CASE(2) DC_CASE(3) DC_CASE(4) DC_CASE(5) DC_CASE(6) DC_CASE(7) DC_CASE(8)
#undef DC_CASE
    default:
      throw InvalidArg("block size n > 64 is not supported");
  }
  DC_HIP(hipGetLastError());
}

void launch_reduced_scatter(Prec p, int n, int V, const void* blocks, const float* scales,
                            const void* inv, const float* invsc, const void* x_e, void* hp,
                            const int* nbr, const int* osite, const int* done, hipStream_t st,
                            hipEvent_t ev0, hipEvent_t ev1, int g5) {
  if (V < 2 || V % 2) throw InvalidArg("the reduced operator needs an even number of sites");
  if (!single_read_fits(p, n))
    throw InvalidArg("the single-read reduced kernels do not take this precision and block size");
  if (p == P16S && (!scales || !invsc)) throw InvalidArg("FP16 blocks need their scales");
  if (!x_e || !hp || !inv) throw InvalidArg("null pointer");
  if (p == P64) reduced_scatter_T<P64>(n, V, blocks, scales, inv, invsc, x_e, hp, nbr, osite, done, st, ev0, ev1, g5);
  else if (p == P32) reduced_scatter_T<P32>(n, V, blocks, scales, inv, invsc, x_e, hp, nbr, osite, done, st, ev0, ev1, g5);
  else reduced_scatter_T<P16S>(n, V, blocks, scales, inv, invsc, x_e, hp, nbr, osite, done, st, ev0, ev1, g5);
}

template <int P, int EPI, bool BJ>
static void reduced_gather_T(int n, int V, const void* blocks, const float* scales,
                             const void* einv, const float* einvsc, const void* x_e,
                             const void* hp, const int* esite, double tm, void* out,
                             const void* e, void* y, z64 c0, z64 ca, z64 cb, const int* done,
                             hipStream_t st, hipEvent_t ev0, hipEvent_t ev1, int g5) {
  using VR = typename VecOf<P>::R;
  const int rows = V / 2;
  const int chunk = (rows + 7) / 8;
  const dim3 grid(unsigned(chunk) * 8u), block(64);
  const auto* xe = static_cast<const cx<VR>*>(x_e);
  const auto* h = static_cast<const cx<VR>*>(hp);
  auto* o = static_cast<cx<VR>*>(out);
  const auto* ee = static_cast<const cx<VR>*>(e);
  auto* yy = static_cast<cx<VR>*>(y);
  const bool full = (n % 8) == 0;
  constexpr bool E0 = EPI == 0;   // Gamma5 comes with the plain store only
  const int stream = reduced_stream(P, n, V);
  switch (tile_T(n)) {
#define DC_CASE(TV)                                                                       \
  case TV:                                                                                \
    if constexpr (single_read_tile<P>(TV)) {                                              \
      const auto k = full ? (E0 && g5 ? k_reduced_gather<TV, P, true, EPI, BJ, E0>        \
                                      : k_reduced_gather<TV, P, true, EPI, BJ, false>)    \
                          : (E0 && g5 ? k_reduced_gather<TV, P, false, EPI, BJ, E0>       \
                                      : k_reduced_gather<TV, P, false, EPI, BJ, false>);  \
      hipExtLaunchKernelGGL(k, grid, block, 0, st, ev0, ev1, 0, blocks, scales, einv,     \
                            einvsc, xe, h, esite, V, n, chunk, tm, o, ee, yy,             \
                            c0, ca, cb, stream, done);                                    \
    }                                                                                     \
    break;
    DC_CASE(1) DC_CASE(2) DC_CASE(3) DC_CASE(4) DC_CASE(5) DC_CASE(6) DC_CASE(7) DC_CASE(8)
#undef DC_CASE
    default:
      throw InvalidArg("block size n > 64 is not supported");
  }
  DC_HIP(hipGetLastError());
}

template <int P>
static void reduced_gather_P(int epi, int n, int V, const void* blocks, const float* scales,
                             const void* einv, const float* einvsc, const void* x_e,
                             const void* hp, const int* esite, double tm, void* out,
                             const void* e, void* y, z64 c0, z64 ca, z64 cb, const int* done,
                             hipStream_t st, hipEvent_t ev0, hipEvent_t ev1, int g5) {
#define DC_ARGS n, V, blocks, scales, einv, einvsc, x_e, hp, esite, tm, out, e, y, c0, ca, cb, done, st, ev0, ev1, g5
  if (einv) {
    switch (epi) {
      case 0: reduced_gather_T<P, 0, true>(DC_ARGS); break;
      case 1: reduced_gather_T<P, 1, true>(DC_ARGS); break;
      default: reduced_gather_T<P, 2, true>(DC_ARGS); break;
    }
    return;
  }
  switch (epi) {
    case 0: reduced_gather_T<P, 0, false>(DC_ARGS); break;
    case 1: reduced_gather_T<P, 1, false>(DC_ARGS); break;
    case 2: reduced_gather_T<P, 2, false>(DC_ARGS); break;
    default: reduced_gather_T<P, 3, false>(DC_ARGS); break;
  }
#undef DC_ARGS
}

void launch_reduced_gather(Prec p, int epi, int n, int V, const void* blocks,
                           const float* scales, const void* einv, const float* einvsc,
                           const void* x_e, const void* hp, const int* esite, double tm,
                           void* out, const void* e, void* y, z64 c0, z64 ca, z64 cb,
                           const int* done, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1, int g5) {
  if (epi < 0 || epi > 3) throw InvalidArg("reduced epilogue must be 0..3");
  if (g5 && epi != 0) throw InvalidArg("Gamma5 comes with the plain store only");
  if (einv && epi == 3) throw InvalidArg("the residual epilogue takes the unpreconditioned operator");
  if (!single_read_fits(p, n))
    throw InvalidArg("the single-read reduced kernels do not take this precision and block size");
  if (p == P16S && ((einv && !einvsc) || (!einv && !scales)))
    throw InvalidArg("FP16 blocks need their scales");
  if (V < 2 || V % 2) throw InvalidArg("the reduced operator needs an even number of sites");
  if (!hp || !out) throw InvalidArg("null vector pointer");
  if (einv && !x_e) throw InvalidArg("block Jacobi needs x_e");
  if ((epi == 1 || epi == 3) && !e) throw InvalidArg("null epilogue input");
  if ((epi == 1 || epi == 2) && !y) throw InvalidArg("null chain output");
#define DC_ARGS epi, n, V, blocks, scales, einv, einvsc, x_e, hp, esite, tm, out, e, y, c0, ca, cb, done, st, ev0, ev1, g5
  if (p == P64) reduced_gather_P<P64>(DC_ARGS);
  else if (p == P32) reduced_gather_P<P32>(DC_ARGS);
  else reduced_gather_P<P16S>(DC_ARGS);
#undef DC_ARGS
}

void launch_oddeven_split(Prec p, int n, int half_sites, const int* esite, const int* osite,
                          void* full, void* ve, void* vo, int dir, hipStream_t st) {
  const size_t N = size_t(half_sites) * n;
  if (N == 0) return;
  const dim3 grid(unsigned((N + 255) / 256)), block(256);
  if (p == P64)
    hipLaunchKernelGGL(k_oddeven_split<double>, grid, block, 0, st, n, half_sites, esite, osite,
                       static_cast<z64*>(full), static_cast<z64*>(ve), static_cast<z64*>(vo), dir);
  else
    hipLaunchKernelGGL(k_oddeven_split<float>, grid, block, 0, st, n, half_sites, esite, osite,
                       static_cast<z32*>(full), static_cast<z32*>(ve), static_cast<z32*>(vo), dir);
  DC_HIP(hipGetLastError());
}

void launch_bj_gather_poly_first(Prec p, int n, int V, const void* inv, const float* scales,
                                 const void* gbuf, const void* v, void* prod, void* y, z64 c0,
                                 z64 ca, z64 cb, const int* done, hipStream_t st) {
  bj_P<true, 1>(p, n, V, inv, scales, gbuf, prod, v, y, c0, ca, cb, done, st);
}

void launch_bj_gather_poly(Prec p, int n, int V, const void* inv, const float* scales,
                           const void* gbuf, void* prod, void* y, z64 ca, z64 cb, const int* done,
                           hipStream_t st) {
  const z64 z = mk(0.0, 0.0);
  bj_P<true, 2>(p, n, V, inv, scales, gbuf, prod, nullptr, y, z, ca, cb, done, st);
}

void launch_chain_multi(Prec p, const void* const* t, const void* const* v, void* const* prod,
                        void* const* y, int R, size_t N, z64 c0, z64 ca, z64 cb, int first,
                        hipStream_t st) {
  if (R <= 0) return;
  const dim3 grid(grid_for(N, 256, 512), unsigned(R)), block(256);
  if (p == P64)
    hipLaunchKernelGGL(k_chain_multi<double>, grid, block, 0, st,
                       reinterpret_cast<const z64* const*>(t), reinterpret_cast<const z64* const*>(v),
                       reinterpret_cast<z64* const*>(prod), reinterpret_cast<z64* const*>(y), N, c0,
                       ca, cb, first);
  else
    hipLaunchKernelGGL(k_chain_multi<float>, grid, block, 0, st,
                       reinterpret_cast<const z32* const*>(t), reinterpret_cast<const z32* const*>(v),
                       reinterpret_cast<z32* const*>(prod), reinterpret_cast<z32* const*>(y), N, c0,
                       ca, cb, first);
  DC_HIP(hipGetLastError());
}

void launch_chain_groups(Prec p, const ChainGroups& g, int first, hipStream_t st) {
  if (g.count < 0 || g.count > kChainGroups) throw InvalidArg("chain table holds 0..8 operators");
  if (g.count == 0) return;
  size_t nmax = 1;
  int rmax = 0;
  for (int i = 0; i < g.count; ++i) {
    if (g.R[i] < 0) throw InvalidArg("negative column count");
    if (first && g.R[i] > 0 && !g.v[i]) throw InvalidArg("the first chain step needs v");
    nmax = std::max(nmax, g.N[i]);
    rmax = std::max(rmax, g.R[i]);
  }
  if (rmax == 0) return;
  const dim3 grid(grid_for(nmax, 256, 512), unsigned(rmax), unsigned(g.count)), block(256);
  if (p == P64) hipLaunchKernelGGL(k_chain_groups<double>, grid, block, 0, st, g, first);
  else hipLaunchKernelGGL(k_chain_groups<float>, grid, block, 0, st, g, first);
  DC_HIP(hipGetLastError());
}

void launch_gather_store(Prec p, int n, int V, const void* gbuf, void* out, const int* done,
                         hipStream_t st) {
  const size_t N = size_t(V) * n;
  const dim3 grid(unsigned((N + 255) / 256)), block(256);
  if (p == P64)
    hipLaunchKernelGGL(k_gather_store<double>, grid, block, 0, st,
                       static_cast<const z64*>(gbuf), static_cast<z64*>(out), N, n, done);
  else
    hipLaunchKernelGGL(k_gather_store<float>, grid, block, 0, st,
                       static_cast<const z32*>(gbuf), static_cast<z32*>(out), N, n, done);
  DC_HIP(hipGetLastError());
}

void launch_gather_poly(Prec p, int n, int V, const void* gbuf, void* prod, void* y, z64 ca,
                        z64 cb, const int* done, hipStream_t st) {
  const size_t N = size_t(V) * n;
  const dim3 grid(unsigned((N + 255) / 256)), block(256);
  if (p == P64)
    hipLaunchKernelGGL(k_gather_poly<double>, grid, block, 0, st, static_cast<const z64*>(gbuf),
                       static_cast<z64*>(prod), static_cast<z64*>(y), N, n, ca, cb, done);
  else
    hipLaunchKernelGGL(k_gather_poly<float>, grid, block, 0, st, static_cast<const z32*>(gbuf),
                       static_cast<z32*>(prod), static_cast<z32*>(y), N, n, ca, cb, done);
  DC_HIP(hipGetLastError());
}

void launch_gather_poly_first(Prec p, int n, int V, const void* gbuf, const void* v, void* prod,
                              void* y, z64 c0, z64 ca, z64 cb, const int* done, hipStream_t st) {
  const size_t N = size_t(V) * n;
  const dim3 grid(unsigned((N + 255) / 256)), block(256);
  if (p == P64)
    hipLaunchKernelGGL(k_gather_poly_first<double>, grid, block, 0, st,
                       static_cast<const z64*>(gbuf), static_cast<const z64*>(v),
                       static_cast<z64*>(prod), static_cast<z64*>(y), N, n, c0, ca, cb, done);
  else
    hipLaunchKernelGGL(k_gather_poly_first<float>, grid, block, 0, st,
                       static_cast<const z32*>(gbuf), static_cast<const z32*>(v),
                       static_cast<z32*>(prod), static_cast<z32*>(y), N, n, c0, ca, cb, done);
  DC_HIP(hipGetLastError());
}

void launch_gather_resid(Prec p, int n, int V, const void* gbuf, const void* b, void* out,
                         Reducer red, double* result, hipStream_t st) {
  const size_t N = size_t(V) * n;
  const unsigned nb = red_blocks(N);
  const dim3 grid(nb), block(256);
  if (p == P64)
    hipLaunchKernelGGL(k_gather_resid<double>, grid, block, 0, st, static_cast<const z64*>(gbuf),
                       static_cast<const z64*>(b), static_cast<z64*>(out), N, n, red, result);
  else
    hipLaunchKernelGGL(k_gather_resid<float>, grid, block, 0, st, static_cast<const z32*>(gbuf),
                       static_cast<const z32*>(b), static_cast<z32*>(out), N, n, red, result);
  DC_HIP(hipGetLastError());
  launch_finalize(red.partials, 1, int(nb), result, nullptr, st);
}

void launch_grad_hops(const z64* lam, const z64* x, z64* grad, const int* nbr, int V, int n,
                      int tied, hipStream_t st) {
  hipLaunchKernelGGL(k_grad_hops, dim3(unsigned(V), tied ? 4u : 8u), dim3(256), 0, st, lam, x,
                     grad, nbr, V, n, tied, std::min(256 / n, n), 65536u / unsigned(n) + 1u);
  DC_HIP(hipGetLastError());
}

}  // namespace dc
