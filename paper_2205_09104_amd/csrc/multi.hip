// Multi-right-hand-side apply on the matrix cores.
#include "kernels.hpp"
#include "device.hpp"

#include <algorithm>
#include <cfloat>
#include <map>
#include <mutex>
#include <tuple>

namespace dc {

namespace {

// ------------------------------------------------------------------ multi-RHS apply
// Y_r = D X_r for R right-hand sides at once: each of a site's nine couplings
// times the n x R panel at its source.  A workgroup of 4 waves takes one site (two or
// four where a small block leaves waves over) and a tile of RB right-hand sides, over a
// work list of the sites of up to kMaxMultiOps operators (a mixed batch of lattices
// with one block size n); grid.y tiles the right-hand sides of the operator with the
// most, tiles past an operator's own count do nothing.  Backward hops Gamma5 B^H Gamma5
// use the stored forward block transposed.  Every stored block is read once per site
// that uses it (9 block reads per site).

typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef __bf16 b2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

// Pointers into device memory (a pointer picked from the kernel arguments at run
// time would otherwise be accessed with flat instructions, whose waits cover
// LDS traffic too).
template <typename X>
using gptr = const X __attribute__((address_space(1)))*;
template <typename X>
using gptr_w = X __attribute__((address_space(1)))*;

// Site number `item` of an operator in brick order: columns of up to 4 x 4 x 4
// sites in the first three directions, walked along the fourth.  The workgroups
// that run at once on an XCD then cover about one brick: most of a site's
// neighbours are among them, and the next brick of the column follows.
__device__ inline int brick_site(const MultiOpDesc& op, unsigned item) {
  const unsigned L0 = unsigned(op.dims[0]), L1 = unsigned(op.dims[1]);
  const unsigned L2 = unsigned(op.dims[2]), L3 = unsigned(op.dims[3]);
  const unsigned plane = L0 * L1 * 4u * L3;
  const unsigned b2 = item / plane;
  item -= b2 * plane;
  const unsigned s2 = min(4u, L2 - 4u * b2), row = L0 * 4u * s2 * L3;
  const unsigned b1 = item / row;
  item -= b1 * row;
  const unsigned s1 = min(4u, L1 - 4u * b1), col = 4u * s1 * s2 * L3;
  const unsigned b0 = item / col;
  item -= b0 * col;
  const unsigned s0 = min(4u, L0 - 4u * b0), brick = s0 * s1 * s2;
  const unsigned x3 = item / brick;
  item -= x3 * brick;
  const unsigned t = item / s0, y0 = item - t * s0, y2 = t / s1, y1 = t - y2 * s1;
  return int(4u * b0 + y0 + L0 * (4u * b1 + y1 + L1 * (4u * b2 + y2 + L2 * x3)));
}

// Couplings (0 self, 1..4 forward hop mu = c - 1, 5..8 backward hop mu = c - 5)
// in the order they are taken: the forward block of one site is the backward
// block of its neighbour, so the two uses follow each other closely in the
// workgroups that run together (directions 0..2), or in this brick's last and
// the next brick's second coupling (direction 3); so do a panel's uses.
__device__ inline int coupling(int step) { return int((0x473625180ull >> (4 * step)) & 15u); }

// The operator of work item `item` (uniform; picked by selects, so the
// kernel-argument array is never indexed dynamically).
__device__ inline MultiOpDesc op_of(const MultiOps& ops, unsigned item) {
  int o = 0;
#pragma unroll
  for (int i = 1; i < kMaxMultiOps; ++i)
    if (i < ops.n_ops && int(item) >= ops.op[i].site0) o = i;
  MultiOpDesc op = ops.op[0];
#pragma unroll
  for (int i = 1; i < kMaxMultiOps; ++i)
    if (i == o) op = ops.op[i];
  return op;
}

// ---- FP64
// Three real products per complex one (Re C = Re A Re B - Im A Im B, Im C = (Re A + Im
// A)(Re B + Im B) - both) on 16x16x4 tiles.  Blocks go to LDS as they are stored, by
// direct loads (double buffered, one barrier per coupling): with the rows of a
// tile taken as two of the layout's unit rows (rows lr T + a, a = 2 rt or 2 rt + 1)
// and the four columns of a step as (4 h + lk) T + b, a lane's operand is one
// 16-byte entry, as it is or transposed.  Unit slots are permuted (lc ^ lr) so that
// both reads spread over the banks.  A lane's panel operand is one entry of its
// right-hand side, loaded to registers a coupling ahead.  The 2 T steps of a
// coupling go to the four waves in turn (equal work); the four partial panels are
// added in LDS at the end, in wave order whatever the tile, so results do not
// depend on RB.
// Measured (FP64; before: planes staged through registers, three of four waves
// multiplying): 8^4, n = 48, 12 right-hand sides 412 -> 237 us, 16^4, 64: 25.7 -> 14.2
// ms, 8^4, n = 16, 32: 84 -> 67 us.  Matrix cores 46% busy at 12 right-hand sides;
// operands loaded straight from the tiled block to registers cost one address
// per lane and ran at 312 us.

// Where a lane of k_apply_multi_f64 finds its entry of row tile rt in step t of its
// wave: byte offsets in the block's LDS buffer.
template <int T>
struct F64Entry {
  static constexpr int BYTES = T * T * 1024;              // a block: T x T units of 64 entries
  static constexpr int RT = (T + 1) / 2, NS = 2 * T, SPW = (NS + 3) / 4;
  __host__ __device__ static constexpr int unit(bool trans, int a, int c) {
    return (trans ? c * T + a : a * T + c) * 1024;
  }
  // the lane's part: row lr (lc) = sub of unit row par, column kk of unit column c0
  __host__ __device__ static constexpr int lane_part(bool trans, int wave, int lane) {
    const int sub = lane & 7, par = (lane >> 3) & 1, kk = 4 * (wave & 1) + (lane >> 4);
    return unit(trans, par, wave >> 1) + (trans ? kk * 8 + (sub ^ kk) : sub * 8 + (kk ^ sub)) * 16;
  }
  // an odd T has no second unit row in its last tile
  __host__ __device__ static constexpr bool missing(int rt, int lane) {
    return T % 2 != 0 && rt == RT - 1 && ((lane >> 3) & 1) != 0;
  }
  // the uniform part; lanes without a unit row read the one before it (and put zero)
  __host__ __device__ static constexpr int step_part(bool trans, int rt, int t, bool none) {
    return unit(trans, 2 * rt - (none ? 1 : 0), 2 * t);
  }
  static constexpr bool inside() {
    for (int trans = 0; trans < 2; ++trans)
      for (int wave = 0; wave < 4; ++wave)
        for (int lane = 0; lane < 64; ++lane)
          for (int t = 0; wave + 4 * t < NS; ++t)
            for (int rt = 0; rt < RT; ++rt) {
              const int at = lane_part(trans, wave, lane) + step_part(trans, rt, t, missing(rt, lane));
              if (at < 0 || at + 16 > BYTES) return false;
            }
    return true;
  }
};
static_assert(F64Entry<1>::inside() && F64Entry<2>::inside() && F64Entry<3>::inside() &&
                  F64Entry<4>::inside() && F64Entry<5>::inside() && F64Entry<6>::inside() &&
                  F64Entry<7>::inside() && F64Entry<8>::inside(),
              "every read stays in its block's buffer");

template <int T, int RB>
__global__ __launch_bounds__(256, T <= 6 ? 2 : 1) void k_apply_multi_f64(MultiOps ops, unsigned sites,
                                                                        int chunk) {
  using acc_t = typename Mfma<double>::acc_t;
  typedef double d2 __attribute__((ext_vector_type(2)));
  constexpr int TT = T * T;
  constexpr int RT = (T + 1) / 2, CT = RB / 16;   // row and column tiles
  constexpr int NS = 2 * T, SPW = (NS + 3) / 4;   // steps of a coupling, per wave
  constexpr int LD = 8 * T + 1;                   // row stride of the output planes
  constexpr int BUF = TT * 1024;                  // bytes of a block
  constexpr int PAN = 2 * RB * LD * 8;            // bytes of the output planes
  __shared__ __align__(1024) unsigned char lds[2 * BUF > PAN ? 2 * BUF : PAN];
  const unsigned item = (blockIdx.x & 7u) * unsigned(chunk) + (blockIdx.x >> 3);
  if (item >= sites) return;
  const MultiOpDesc op = op_of(ops, item);
  const int n = ops.n, half = n >> 1, R = op.R, V = op.V;
  const int r0 = int(blockIdx.y) * RB;
  if (r0 >= R) return;
  const int site = brick_site(op, item - unsigned(op.site0));
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int l16 = lane & 15, lk = lane >> 4;
  const bool g5in = (ops.g5io & 1) != 0, g5out = (ops.g5io & 2) != 0;
  const auto nbr = (gptr<int>)op.nbr;
  gptr<d2> xr[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c)   // lanes past R repeat the last right-hand side
    xr[c] = (gptr<d2>)(((gptr<const void*>)op.xin)[min(r0 + c * 16 + l16, R - 1)]);

  // step t of this wave: s = wave + 4 t = 2 c + h, columns (4 h + lk) T + c
  const int kk = 4 * (wave & 1) + lk, c0 = wave >> 1;
  const int sub = l16 & 7, par = l16 >> 3;   // row of a tile: (lr or lc) = sub, a (b) = 2 rt + par
  using At = F64Entry<T>;
  const int at_f = At::lane_part(false, wave, lane), at_t = At::lane_part(true, wave, lane);

  auto load_block = [&](int blk, int buf) {
    const int lr = lane >> 3, lc = lane & 7;
    const auto src = (gptr<d2>)op.blocks + size_t(blk) * (64 * TT) + (lr * 8 + (lc ^ lr));
#pragma unroll
    for (int i = 0; i < (TT + 3) / 4; ++i) {
      const int e = wave + 4 * i;
      if (TT % 4 != 0 && e >= TT) continue;
      __builtin_amdgcn_global_load_lds(
          (const void __attribute__((address_space(1)))*)(src + e * 64),
          (void __attribute__((address_space(3)))*)(lds + buf * BUF + e * 1024), 16, 0, 0);
    }
  };
  d2 B[SPW][CT];
  auto load_panel = [&](int src) {
#pragma unroll
    for (int t = 0; t < SPW; ++t) {
      // past n the blocks are zero
      const size_t j = size_t(src) * n + min(kk * T + c0 + 2 * t, n - 1);
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) B[t][ct] = xr[ct][j];
    }
  };
  auto flip = [](double v, uint32_t m) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    return __builtin_bit_cast(double, b ^ (uint64_t(m) << 32));
  };
  acc_t crr[RT][CT], cii[RT][CT], css[RT][CT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) crr[rt][ct] = cii[rt][ct] = css[rt][ct] = acc_t{0, 0, 0, 0};
  load_block(site * 5, 0);
  load_panel(site);
  // lane l holds the source site and the block of the l-th coupling
  const int lcoup = coupling(min(lane, 8));
  const int lsrc = lcoup == 0 ? site : nbr[(lcoup - 1) * V + site];
  const int lblk = lcoup < 5 ? site * 5 + lcoup : lsrc * 5 + (lcoup - 4);
#pragma unroll 1
  for (int c = 0; c < 9; ++c) {
    const bool trans = coupling(c) >= 5;
    // this coupling's block is in LDS, and the other buffer's products are done
    __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
    __syncthreads();
    // signs: Gamma5 B^H Gamma5 conjugates the block and flips rows and columns of
    // the lower half; Gamma5 on the input flips the columns once more
    const bool colsign = trans != g5in;
    double br[SPW][CT], bi[SPW][CT];
#pragma unroll
    for (int t = 0; t < SPW; ++t) {
      const uint32_t mj = colsign && kk * T + c0 + 2 * t >= half ? 0x80000000u : 0u;
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        br[t][ct] = flip(B[t][ct].x, mj);
        bi[t][ct] = flip(B[t][ct].y, mj);
      }
    }
    if (c < 8) {
      load_block(__builtin_amdgcn_readlane(lblk, c + 1), (c + 1) & 1);
      load_panel(__builtin_amdgcn_readlane(lsrc, c + 1));
    }
    const unsigned char* base = lds + (c & 1) * BUF + (trans ? at_t : at_f);
#pragma unroll
    for (int t = 0; t < SPW; ++t) {
      if (NS % 4 != 0 && wave + 4 * t >= NS) continue;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const bool none = At::missing(rt, lane);
        d2 z = *reinterpret_cast<const d2*>(base + At::step_part(trans, rt, t, none));
        if (none) z = d2{0.0, 0.0};
        const uint32_t mi = trans && sub * T + 2 * rt + par >= half ? 0x80000000u : 0u;
        const double ar = flip(z.x, mi), ai = flip(z.y, trans ? mi ^ 0x80000000u : 0u);
        const double as = ar + ai;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          crr[rt][ct] = Mfma<double>::mma(ar, br[t][ct], crr[rt][ct]);
          cii[rt][ct] = Mfma<double>::mma(ai, bi[t][ct], cii[rt][ct]);
          css[rt][ct] = Mfma<double>::mma(as, br[t][ct] + bi[t][ct], css[rt][ct]);
        }
      }
    }
  }
  __syncthreads();
  // partial panels added in wave order: planes [right-hand side][entry]
  double* pr = reinterpret_cast<double*>(lds);
  double* pi = pr + RB * LD;
#pragma unroll 1
  for (int w = 0; w < 4; ++w) {
    if (wave == w) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row = Mfma<double>::row(lk, q), a = 2 * rt + (row >> 3);
          if (T % 2 != 0 && a >= T) continue;
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) {
            const int at = (ct * 16 + l16) * LD + (row & 7) * T + a;
            const double re = crr[rt][ct][q] - cii[rt][ct][q];
            const double im = css[rt][ct][q] - crr[rt][ct][q] - cii[rt][ct][q];
            pr[at] = w == 0 ? re : pr[at] + re;
            pi[at] = w == 0 ? im : pi[at] + im;
          }
        }
    }
    __syncthreads();
  }
  const int Rc = min(RB, R - r0);
  const double tm = op.tm;
  for (int t = threadIdx.x; t < Rc * n; t += 256) {
    const int r = t / n, i = t - r * n;
    double re = pr[r * LD + i], im = pi[r * LD + i];
    const size_t at = size_t(site) * n + i;
    if (tm != 0.0) {   // g_i (i tm) (g_i x_i with Gamma5 on the input)
      const d2 x = ((gptr<d2>)(((gptr<const void*>)op.xin)[r0 + r]))[at];
      const double ti = (g5in || i < half) ? tm : -tm;
      re -= ti * x.y;
      im += ti * x.x;
    }
    if (g5out && i >= half) {
      re = -re;
      im = -im;
    }
    ((gptr_w<d2>)(((gptr<void*>)op.yout)[r0 + r]))[at] = d2{re, im};
  }
}

// ---- FP32 vectors: BF16 pieces on the BF16 matrix cores
// The FP32 matrix instructions run at 1/16 of the BF16 rate.  A BF16 number has the
// exponents of an FP32 one and 8 of its 24 significant bits, so an FP32 number is the
// sum of three, x = x1 + x2 + x3, x1 = bf16(x), x2 = bf16(x - x1), x3 the rest, exactly
// (|x2| <= 2^-8, |x3| <= 2^-17 of x's binade), and an entry keeps its own precision
// whatever the others' sizes are.  A product of two is six products of pieces, a1 x1 +
// (a1 x2 + a2 x1) + (a1 x3 + a2 x2 + a3 x1): what is dropped is at most 2^-24 of it, the
// bound of an FP32 rounding.  A code of an FP16-stored block (11 bits) is two pieces, and
// its products five.  The sums are in FP32, as the results are.
// Pieces below 2^-126 would lose bits, and products of an FP16 block's codes, which are
// without its scale, can overflow where the result does not.  So an FP32 block (by
// its largest entry, kept at build time) and a right-hand side's n entries at a source
// site are moved by 2^40 where their largest is below 2^-64, by 2^-40 where it is 2^64 or
// more, and the products are multiplied by what undoes both and an FP16 block's scale:
// only what overflows in the result overflows.  Next to a largest entry of 2^-64 or
// more, entries below 2^-110 are held to 2^-133.
// Layout: complex values stay interleaved, (re, im) pairs are two k entries:
// Re = (ar, ai) . (pr, -pi), Im = (ar, ai) . (pi, pr), on 16x16x32 tiles (16
// complex columns per step).  The four waves of a workgroup take the RB / 16 column
// tiles, and share the k steps of each where there are fewer.  The couplings' blocks
// go through LDS as BF16 pairs, a plane per piece (rows padded to an odd number of
// 16-byte units: conflict-free fragment reads); the panels go from memory to the wave
// that multiplies them, which holds its fragments in registers and splits them one k
// step at a time, between the products.  A step's products are summed small ones first,
// from zero, and then added.
// Measured (16^4, n = 48, 64 right-hand sides; FP32 matrix instructions, three real products
// per complex one, and planes in LDS before): FP32 6.70 -> 5.18 ms, FP16 blocks 6.87 -> 4.14
// ms; 12 right-hand sides: 2.29 -> 2.21 and 2.38 -> 1.61 ms.  At 64 in FP32, matrix cores 44%,
// vector ALU (the splits) 64%, LDS 43% busy, at a clock that falls to 1.9 GHz under it.
// Error, each entry against the sum of the magnitudes that enter it, n = 48: 4e-8 to
// 1.6e-7 over evenly sized and graded operands (2e-7 to 5e-7 before).  Two FP16 pieces with a
// scale per block and column take three products and 3.7 ms, but hold entries far
// below the largest to too few bits: they lost rows and columns of graded blocks.
// Three couplings in flight instead of one cost more occupancy than they gain
// (n = 16, 32: 10% slower).

// Power of two that brings a largest magnitude m towards 1 where it is near an end of
// the range of the exponents, and its inverse.
__device__ inline void pow2_scale(float m, float& up, float& down) {
  const uint32_t e = (__float_as_uint(m) >> 23) & 255u;   // biased exponent
  up = e < 63u ? 0x1p40f : e > 190u ? 0x1p-40f : 1.f;
  down = e < 63u ? 0x1p-40f : e > 190u ? 0x1p40f : 1.f;
}

// The leading N BF16 pieces of a complex value, each packed (re low, im high).
template <int N>
__device__ inline void split_pair(float re, float im, uint32_t (&p)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    p[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{re, im}, b2));
    re -= __uint_as_float(p[i] << 16);
    im -= __uint_as_float(p[i] & 0xffff0000u);
  }
}

// Waves per column tile: they share its k steps, every one over all row tiles, so
// no panel entry is split twice; small blocks that leave waves over put several
// sites into a workgroup.  (16^4, n = 48, 12 right-hand sides, against waves that
// share the row tiles and each split the whole panel, with two pieces per entry: FP32 2.43
// -> 1.82 ms, FP16 blocks 1.84 -> 1.19; n = 16, 32 on 8^4: 54 -> 39 us.)
template <int T, int P, int RB>
struct SplitShape {
  static constexpr int NP = (8 * T + 15) / 16 * 16;   // block edge padded to whole tiles
  static constexpr int RT = NP / 16, KS = NP / 16;    // row tiles, k steps of 16 complex columns
  static constexpr int CT = RB / 16;                  // column tiles
  static constexpr int KG = (KS == 1 || CT == 4) ? 1 : (KS == 2 || CT == 2) ? 2 : 4;
  static constexpr int KSW = (KS + KG - 1) / KG;      // k steps per wave
  static constexpr int WPS = CT * KG, SPB = 4 / WPS;  // waves per site, sites per workgroup
  // Panels of more than 16 columns come in 128-byte segments and turn into fragments
  // through LDS: a fragment's own loads touch 64 cache lines each, and their look-ups
  // bounded the kernel.  16 columns (bound by the blocks) are loaded as fragments.
  // 16^4, n = 48, fragments / segments: 64 columns FP32 5.40 / 5.18 ms, FP16 blocks 4.56 /
  // 4.14, 32 6.54 / 6.50, 16 2.21 / 2.23.
  static constexpr bool STRIP = CT > 1;
  // Block buffers: two write the next block beside the products (one barrier per
  // coupling), one leaves room for more workgroups.  Two buffers / one, 16^4, n = 48, 12
  // right-hand sides, ms: FP32 (three pieces) 3.06 / 2.24, FP16 blocks (two) 1.65 / 1.91;
  // 64: 5.43 / 5.25 and 4.26 / 4.39; 8^4, n = 64, 64 in FP32: 0.75 / 0.58.
  static constexpr int NBUF = P == P32 ? 1 : 2;
  // workgroups per CU that the registers are held to (three: 168, T = 6 at 64 columns
  // spills two to four; against two there: 5.26 / 5.48 ms, FP16 blocks 4.22 / 4.47; four at
  // 16 columns spill more: 2.64 / 2.24 ms)
  static constexpr int WAVES = T > 6 ? 2 : 3;
};

template <int T, int P, int RB>
__global__ __launch_bounds__(256, (SplitShape<T, P, RB>::WAVES)) void k_apply_multi_split(
    MultiOps ops, unsigned sites, int chunk) {
  using Sh = SplitShape<T, P, RB>;
  constexpr int NP = Sh::NP, RT = Sh::RT, KS = Sh::KS, CT = Sh::CT, KG = Sh::KG, KSW = Sh::KSW;
  constexpr int WPS = Sh::WPS, SPB = Sh::SPB;
  constexpr int PIECES = (P == P32) ? 3 : 2;      // BF16 pieces of a block entry
  constexpr int NBUF = Sh::NBUF;                  // buffers of a block
  constexpr int LDA = (NP + 4) * 4;               // bytes of an LDS row (NP pairs + padding)
  constexpr int PLANE = NP * LDA + 16;            // + a word that takes padding entries
  constexpr int SLDS = NBUF * PIECES * PLANE;     // bytes of a site
  constexpr int TT = T * T;
  constexpr int EPL = (P == P32) ? 2 : 4;         // block entries per 16-byte unit
  constexpr int UPL = (TT + EPL - 1) / EPL;       // units per lane of a block
  constexpr int MU = (UPL + WPS - 1) / WPS;       // units per thread
  __shared__ __align__(16) unsigned char lds_all[SPB * SLDS];
  __shared__ __align__(16) unsigned char strips[Sh::STRIP ? 4 * 2048 : 16];   // a panel strip per wave
  static_assert((KG - 1) * CT * RT * 2 * 64 * 16 <= SLDS, "partial panels fit");
  const int gwave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int slot = gwave / WPS, wave = gwave % WPS;
  unsigned char* const lds = lds_all + slot * SLDS;
  // XCD-aware order: each XCD takes a contiguous range of sites, so neighbouring
  // sites share blocks and panels through its L2
  const unsigned item0 = ((blockIdx.x & 7u) * unsigned(chunk) + (blockIdx.x >> 3)) * SPB;
  if (item0 >= sites) return;
  // a slot past the end repeats the last site and stores nothing
  const unsigned item = min(item0 + unsigned(slot), sites - 1u);
  const MultiOpDesc op = op_of(ops, item);
  const int n = ops.n, half = n >> 1, R = op.R, V = op.V;
  const int r0 = int(blockIdx.y) * RB;
  if (SPB == 1 && r0 >= R) return;
  const bool live = item == item0 + unsigned(slot) && r0 < R;
  const int site = brick_site(op, item - unsigned(op.site0));
  const int l16 = lane & 15, lk = lane >> 4;
  const int lr = lane >> 3, lc = lane & 7;
  const int ct = wave % CT, kg = wave / CT;
  const bool g5in = (ops.g5io & 1) != 0, g5out = (ops.g5io & 2) != 0;
  const auto blocks = (gptr<u4>)op.blocks;
  const auto scales = (gptr<float>)op.scales;   // FP16: block scales; FP32: largest magnitudes
  const auto nbr = (gptr<int>)op.nbr;

  // Unit k = wave + WPS s of the tiled block, entries e = k EPL + q = a T + b: lane
  // (lr, lc) holds (lr T + a, lc T + b).  Its LDS byte offset is a lane part plus
  // a wave-uniform one, as it is or transposed.  Entries past the n x n block but
  // inside the tiled layout are zeros there and land in the padding of the
  // plane; the slots of a unit past the tile go to the spare word.
  const int lbase = lr * T * LDA + lc * T * 4, lbase_t = lc * T * LDA + lr * T * 4;
  const int rc = min(r0 + ct * 16 + l16, R - 1);  // lanes past R repeat the last column
  const auto xr = (gptr<z32>)(((gptr<const void*>)op.xin)[rc]);
  // Panel loads of k step ks = kg + KG t, q = 0, 1.  As fragments: entries 16 ks + 4 lk
  // + 2 q and the next of column l16.  As segments (STRIP): eight lanes for entries 16 ks
  // .. 16 ks + 15 of each of columns 8 q .. 8 q + 7, and the wave's LDS strip hands them
  // on as fragments; a column's eight units are permuted by its number so that the
  // reads spread over the banks.  Past n the last pair is read again (the blocks are
  // zero there).
  constexpr bool STRIP = Sh::STRIP;
  gptr<z32> xq[2];
  int joff[KSW][2], spos[2], fpos[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int col = STRIP ? 8 * q + (lane >> 3) : l16, u = STRIP ? lane & 7 : 2 * lk + q;
    xq[q] = (gptr<z32>)(((gptr<const void*>)op.xin)[min(r0 + ct * 16 + col, R - 1)]);
    spos[q] = col * 8 + (u ^ ((col >> 1) & 7));
    fpos[q] = l16 * 8 + ((2 * lk + q) ^ ((l16 >> 1) & 7));
#pragma unroll
    for (int t = 0; t < KSW; ++t) joff[t][q] = min(16 * (kg + KG * t) + 2 * u, n - 2);
  }
  f4* const strip = reinterpret_cast<f4*>(strips) + (STRIP ? gwave * 128 : 0);

  u4 araw[MU];
  f4 braw[KSW][2];
  auto load_block = [&](int blk) {
    const auto b = blocks + size_t(blk) * (64 * UPL) + lane;
#pragma unroll
    for (int s = 0; s < MU; ++s) {
      const int k = wave + WPS * s;
      if (UPL % WPS == 0 || k < UPL) araw[s] = b[k * 64];
    }
  };
  auto load_panel = [&](int src) {
    const size_t x = size_t(src) * n;
#pragma unroll
    for (int t = 0; t < KSW; ++t)
#pragma unroll
      for (int q = 0; q < 2; ++q) braw[t][q] = *(gptr<f4>)(xq[q] + x + joff[t][q]);
  };
  auto store_block = [&](unsigned char* buf, float scale, bool trans) {
    if constexpr (P == P32) {
      float up, down;
      pow2_scale(scale, up, down);
      if (up != 1.f) {
#pragma unroll
        for (int s = 0; s < MU; ++s)
#pragma unroll
          for (int q = 0; q < 4; ++q) araw[s][q] = __float_as_uint(__uint_as_float(araw[s][q]) * up);
      }
    }
    // transposed: Gamma5 B^H Gamma5 = g_i g_j conj(B[j][i]); the masks negate
    // the imaginary (+) or the real part (-) of a packed pair
    unsigned char* base = buf + (trans ? lbase_t : lbase);
#pragma unroll
    for (int s = 0; s < MU; ++s) {
      const int k = wave + WPS * s;
      if (UPL % WPS != 0 && k >= UPL) continue;
#pragma unroll
      for (int q = 0; q < EPL; ++q) {
        const int e = k * EPL + q;
        const int a = e / T, b = e - a * T;
        uint32_t p[PIECES];
        if constexpr (P == P32)
          split_pair(__uint_as_float(araw[s][2 * q]), __uint_as_float(araw[s][2 * q + 1]), p);
        else
          split_pair(lo_h(araw[s][q]), hi_h(araw[s][q]), p);
        unsigned char* at = base + (trans ? b * LDA + a * 4 : a * LDA + b * 4);
        if (TT % EPL != 0 && e >= TT) at = buf + NP * LDA;
        const uint32_t m = (lr * T + a < half) == (lc * T + b < half) ? 0x80000000u : 0x00008000u;
#pragma unroll
        for (int i = 0; i < PIECES; ++i)
          *reinterpret_cast<uint32_t*>(at + i * PLANE) = trans ? p[i] ^ m : p[i];
      }
    }
  };

  f4 tre[RT], tim[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) tre[rt] = tim[rt] = f4{0.f, 0.f, 0.f, 0.f};
  load_block(site * 5);
  load_panel(site);
  // lane l holds the source site and the block scale of the l-th coupling, read
  // once: a table look-up inside the loop would wait for the panel and block
  // loads in flight before it
  const int lcoup = coupling(min(lane, 8));
  const int lsrc = lcoup == 0 ? site : nbr[(lcoup - 1) * V + site];
  const int lblk = lcoup < 5 ? site * 5 + lcoup : lsrc * 5 + (lcoup - 4);
  const float lsc = scales[lblk];
  auto source = [&](int step) { return __builtin_amdgcn_readlane(lsrc, step); };
  auto block_of = [&](int step) { return __builtin_amdgcn_readlane(lblk, step); };
  auto scale_of = [&](int step) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(lsc), step));
  };
  // rows and columns past the tiled layout stay zero
  if (NP != 8 * T) {
    for (int t = threadIdx.x * 16; t < SPB * SLDS; t += 256 * 16)
      *reinterpret_cast<u4*>(lds_all + t) = u4{0, 0, 0, 0};
    __syncthreads();
  }
  if (NBUF == 2) {
    store_block(lds, scale_of(0), false);
    load_block(block_of(1));
  }
#pragma unroll 1
  for (int c = 0; c < 9; ++c) {
    unsigned char* buf = lds + (NBUF == 2 ? (c & 1) * (PIECES * PLANE) : 0);
    if (NBUF == 1) {
      if (c > 0) __syncthreads();   // the products of the coupling before are done
      store_block(buf, scale_of(c), coupling(c) >= 5);
      if (c < 8) load_block(block_of(c + 1));
    }
    __syncthreads();   // buf is complete, and the other buffer's products are done
    // this coupling's panel as fragments (LDS keeps the order of a wave's
    // accesses to its strip)
    f4 fr[KSW][2];
#pragma unroll
    for (int t = 0; t < KSW; ++t) {
      if constexpr (STRIP) {
        strip[spos[0]] = braw[t][0];
        strip[spos[1]] = braw[t][1];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        fr[t][0] = strip[fpos[0]];
        fr[t][1] = strip[fpos[1]];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      } else {
        fr[t][0] = braw[t][0];
        fr[t][1] = braw[t][1];
      }
    }
    float mx = 0.f;
#pragma unroll
    for (int t = 0; t < KSW; ++t)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        mx = fmaxf(fmaxf(mx, fabsf(fr[t][q].x)), fabsf(fr[t][q].y));
        mx = fmaxf(fmaxf(mx, fabsf(fr[t][q].z)), fabsf(fr[t][q].w));
      }
    // no factor where each lane's largest entry is zero or in the range that needs none
    float down = 1.f;
    if (__builtin_amdgcn_ballot_w64(mx != 0.f && !(mx >= 0x1p-64f && mx < 0x1p64f)) != 0) {
      mx = fmaxf(mx, shfl_xor(mx, 16));
      mx = fmaxf(mx, shfl_xor(mx, 32));
      float up;
      pow2_scale(mx, up, down);
#pragma unroll
      for (int t = 0; t < KSW; ++t)
#pragma unroll
        for (int q = 0; q < 2; ++q) fr[t][q] *= up;
    }
    if (g5in) {
#pragma unroll
      for (int t = 0; t < KSW; ++t)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int j = 16 * (kg + KG * t) + 4 * lk + 2 * q;
          if (j >= half) fr[t][q].xy = -fr[t][q].xy;
          if (j + 1 >= half) fr[t][q].zw = -fr[t][q].zw;
        }
    }
    float fblk = scale_of(c);
    if (P == P32) {
      float u;
      pow2_scale(fblk, u, fblk);
    }
    if (c + 1 < 9) load_panel(source(c + 1));
    // the next panel and block are in flight (with two buffers, the next block's pieces
    // are written too) while this coupling multiplies
    if (NBUF == 2 && c + 1 < 9) {
      unsigned char* nb = lds + ((c + 1) & 1) * (PIECES * PLANE);
      if (coupling(c + 1) < 5) store_block(nb, scale_of(c + 1), false);
      else store_block(nb, scale_of(c + 1), true);
      if (c + 2 < 9) load_block(block_of(c + 2));
    }
    // both factors undone in one: what would overflow here overflows in the result (a
    // scale that is not finite stays so)
    const float f = fblk <= FLT_MAX ? fminf(fblk * down, FLT_MAX) : fblk;
#pragma unroll
    for (int t = 0; t < KSW; ++t) {
      if (KS % KG != 0 && kg + KG * t >= KS) continue;
      // pieces as (pi, pr) pairs, the Im operand, and (pr, -pi), the Re operand: swapped,
      // high half negated
      u4 bi[3], br[3];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const f4 z = fr[t][q];
        uint32_t h[2][3];
        split_pair(z.y, z.x, h[0]);
        split_pair(z.w, z.z, h[1]);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            bi[k][2 * q + i] = h[i][k];
            br[k][2 * q + i] = __builtin_amdgcn_alignbit(h[i][k], h[i][k], 16) ^ 0x80000000u;
          }
      }
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const unsigned char* row = buf + (rt * 16 + l16) * LDA + lk * 16 + kg * 64 + t * KG * 64;
        f4 re = {0.f, 0.f, 0.f, 0.f}, im = re;
        auto mul = [&](b8 a, int k) {
          re = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(b8, br[k]), re, 0, 0, 0);
          im = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(b8, bi[k]), im, 0, 0, 0);
        };
        // small products first
        const b8 a1 = *reinterpret_cast<const b8*>(row), a2 = *reinterpret_cast<const b8*>(row + PLANE);
        if constexpr (PIECES == 3) mul(*reinterpret_cast<const b8*>(row + 2 * PLANE), 0);
        mul(a2, 1);
        mul(a1, 2);
        mul(a2, 0);
        mul(a1, 1);
        mul(a1, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          tre[rt][q] = fmaf(re[q], f, tre[rt][q]);
          tim[rt][q] = fmaf(im[q], f, tim[rt][q]);
        }
      }
    }
  }
  // the k shares of a column tile added in wave order
  if (KG > 1) {
    __syncthreads();
    f4* part = reinterpret_cast<f4*>(lds) + lane;
    if (kg > 0) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        part[(((kg - 1) * CT + ct) * RT + rt) * 128] = tre[rt];
        part[(((kg - 1) * CT + ct) * RT + rt) * 128 + 64] = tim[rt];
      }
    }
    __syncthreads();
    if (kg > 0) return;
#pragma unroll
    for (int g = 1; g < KG; ++g) {
      if (KS % KG != 0 && g >= KS) continue;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        tre[rt] += part[(((g - 1) * CT + ct) * RT + rt) * 128];
        tim[rt] += part[(((g - 1) * CT + ct) * RT + rt) * 128 + 64];
      }
    }
  }
  // lane: rows 16 rt + 4 lk .. + 3 of right-hand side r; i tm Gamma5 x added here
  if (!live || r0 + ct * 16 + l16 >= R) return;
  const auto y = (gptr_w<z32>)(((gptr<void*>)op.yout)[rc]) + size_t(site) * n;
  const auto xs = xr + size_t(site) * n;
  const float tm = float(op.tm);
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
    for (int q = 0; q < 4; q += 2) {
      const int i = rt * 16 + lk * 4 + q;
      if (i >= n) continue;
      f4 z = {tre[rt][q], tim[rt][q], tre[rt][q + 1], tim[rt][q + 1]};
      if (tm != 0.f) {   // g_i (i tm) (g_i x_i with Gamma5 on the input)
        const f4 v = *(gptr<f4>)(xs + i);
        const float t0 = (g5in || i < half) ? tm : -tm, t1 = (g5in || i + 1 < half) ? tm : -tm;
        z.x = fmaf(-t0, v.y, z.x);
        z.y = fmaf(t0, v.x, z.y);
        z.z = fmaf(-t1, v.w, z.z);
        z.w = fmaf(t1, v.z, z.w);
      }
      if (g5out && i >= half) {
        z.x = -z.x;
        z.y = -z.y;
      }
      if (g5out && i + 1 >= half) {
        z.z = -z.z;
        z.w = -z.w;
      }
      *(gptr_w<f4>)(y + i) = z;
    }
  }
}

}  // namespace

static int multi_np(int n) { return (n + 15) / 16 * 16; }

template <int T, int P, int RB>
static void split_launch(const MultiOps& ops, unsigned sites, int rmax, hipStream_t st) {
  constexpr unsigned spb = SplitShape<T, P, RB>::SPB;
  const int chunk = int(((sites + spb - 1) / spb + 7) / 8);
  const unsigned rtiles = unsigned((rmax + RB - 1) / RB);
  hipLaunchKernelGGL((k_apply_multi_split<T, P, RB>), dim3(unsigned(chunk) * 8u, rtiles),
                     dim3(256), 0, st, ops, sites, chunk);
  DC_HIP(hipGetLastError());
}

template <int P>
static void split_T_launch(int rb, const MultiOps& ops, unsigned sites, int rmax, hipStream_t st) {
  switch (tile_T(ops.n)) {
#define DC_CASE(TV)                                                          \
  case TV:                                                                   \
    if (rb == 16) split_launch<TV, P, 16>(ops, sites, rmax, st);             \
    else if (rb == 32) split_launch<TV, P, 32>(ops, sites, rmax, st);        \
    else split_launch<TV, P, 64>(ops, sites, rmax, st);                      \
    break;
    DC_CASE(1) DC_CASE(2) DC_CASE(3) DC_CASE(4) DC_CASE(5) DC_CASE(6) DC_CASE(7) DC_CASE(8)
#undef DC_CASE
    default: throw InvalidArg("block size n > 64 is not supported");
  }
}

template <int T, int RB>
static void f64_launch(const MultiOps& ops, unsigned sites, int rmax, hipStream_t st) {
  const int chunk = int((sites + 7) / 8);
  const unsigned rtiles = unsigned((rmax + RB - 1) / RB);
  hipLaunchKernelGGL((k_apply_multi_f64<T, RB>), dim3(unsigned(chunk) * 8u, rtiles), dim3(256), 0,
                     st, ops, sites, chunk);
  DC_HIP(hipGetLastError());
}

static void multi_dispatch(Prec p, int rb, const MultiOps& ops, unsigned sites, int rmax,
                           hipStream_t st) {
  if (p == P32) return split_T_launch<P32>(rb, ops, sites, rmax, st);
  if (p == P16S) return split_T_launch<P16S>(rb, ops, sites, rmax, st);
  switch (tile_T(ops.n)) {
#define DC_CASE(TV)                                              \
  case TV:                                                       \
    if (rb == 16) f64_launch<TV, 16>(ops, sites, rmax, st);      \
    else f64_launch<TV, 32>(ops, sites, rmax, st);               \
    break;
    DC_CASE(1) DC_CASE(2) DC_CASE(3) DC_CASE(4) DC_CASE(5) DC_CASE(6) DC_CASE(7) DC_CASE(8)
#undef DC_CASE
    default: throw InvalidArg("block size n > 64 is not supported");
  }
}

// Autotuned right-hand-side tile (16, 32 or 64 per workgroup): the first launch
// of a shape class (block size, precision, right-hand-side and site-count
// buckets) times each candidate on the actual operands with HIP events and
// keeps the fastest; later launches of the class use it.
namespace {
struct TuneKey {
  int np, prec, rbucket, vbucket;
  bool operator<(const TuneKey& o) const {
    return std::tie(np, prec, rbucket, vbucket) < std::tie(o.np, o.prec, o.rbucket, o.vbucket);
  }
};
std::mutex g_tune_mu;
std::map<TuneKey, int> g_tune;
int g_tune_mode = 0;  // 0: autotune; 16/32/64: forced tile

TuneKey tune_key(Prec p, int n, int rmax, unsigned sites) {
  int rbk = 0;
  while ((16 << rbk) < rmax && rbk < 3) ++rbk;   // <=16, <=32, <=64, >64
  int vb = 0;
  while ((1u << (vb + 1)) <= sites && vb < 30) ++vb;  // floor(log2(sites))
  return TuneKey{multi_np(n), int(p), rbk, vb};
}
}  // namespace

int multi_tile_for(Prec p, int n, int rmax, unsigned sites) {
  std::lock_guard<std::mutex> lk(g_tune_mu);
  if (g_tune_mode) return g_tune_mode;
  const auto it = g_tune.find(tune_key(p, n, rmax, sites));
  return it == g_tune.end() ? 0 : it->second;
}

void set_multi_tile_mode(int mode) {
  if (mode != 0 && mode != 16 && mode != 32 && mode != 64)
    throw InvalidArg("tile mode must be 0 (autotune), 16, 32 or 64");
  std::lock_guard<std::mutex> lk(g_tune_mu);
  g_tune_mode = mode;
  if (mode == 0) g_tune.clear();
}

void launch_apply_multi_ops(Prec p, int n, const MultiOpDesc* desc, int n_ops, int g5io,
                            hipStream_t st) {
  if (n_ops < 1 || n_ops > kMaxMultiOps) throw InvalidArg("1..8 operators per multi-apply");
  if (multi_np(n) > 64) throw InvalidArg("block size n > 64 is not supported");
  MultiOps ops{};
  ops.n_ops = n_ops;
  ops.n = n;
  ops.g5io = g5io;
  unsigned sites = 0;
  int rmax = 0;
  for (int i = 0; i < n_ops; ++i) {
    if (1LL * desc[i].dims[0] * desc[i].dims[1] * desc[i].dims[2] * desc[i].dims[3] != desc[i].V)
      throw InvalidArg("lattice extents do not match the number of sites");
    if (p != P64 && !desc[i].scales) throw InvalidArg("reduced-precision multi-apply needs the block scales");
    ops.op[i] = desc[i];
    ops.op[i].site0 = int(sites);
    sites += unsigned(desc[i].V);
    rmax = std::max(rmax, desc[i].R);
  }
  if (rmax <= 0 || sites == 0) return;
  int rb = multi_tile_for(p, n, rmax, sites);
  if (rb == 0) {
    // time every candidate (each fully overwrites the outputs)
    hipEvent_t e0, e1;
    DC_HIP(hipEventCreate(&e0));
    DC_HIP(hipEventCreate(&e1));
    float best = 1e30f;
    for (int cand : {16, 32, 64}) {
      if (cand > 16 && (cand / 2) >= rmax) break;   // wider tiles than the batch
      if (cand == 64 && p == P64) break;            // FP64 accumulators of 64 would spill
      multi_dispatch(p, cand, ops, sites, rmax, st);   // warm
      DC_HIP(hipEventRecord(e0, st));
      for (int rep = 0; rep < 3; ++rep) multi_dispatch(p, cand, ops, sites, rmax, st);
      DC_HIP(hipEventRecord(e1, st));
      DC_HIP(hipEventSynchronize(e1));
      float ms = 0.f;
      DC_HIP(hipEventElapsedTime(&ms, e0, e1));
      if (ms < best) {
        best = ms;
        rb = cand;
      }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tune[tune_key(p, n, rmax, sites)] = rb;
    // the outputs come from the chosen tile, as in every later call (the FP32
    // tiles split their sums differently and agree only to rounding)
  }
  multi_dispatch(p, rb, ops, sites, rmax, st);
}

}  // namespace dc
