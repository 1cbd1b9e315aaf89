// Multi-right-hand-side apply on the matrix cores.
#include "kernels.hpp"
#include "device.hpp"

#include <algorithm>
#include <map>
#include <mutex>
#include <tuple>

namespace dc {

namespace {

// ------------------------------------------------------------------ multi-RHS apply
// Y_r = D X_r for R right-hand sides at once.  One workgroup (4 waves) per
// site accumulates the 9 couplings of the site into an n x R output panel
// held in MFMA accumulators: each coupling stages its block (as the vector
// precision) and the source panel in LDS, and the complex product runs as
// three real GEMMs (Re M Re P, Im M Im P, (Re M + Im M)(Re P + Im P)) on
// 16x16x4 MFMA tiles.
// Backward hops Gamma5 B^H Gamma5 read the staged forward block transposed.
// Every stored block is read once per site that uses it (9 block reads per
// site; the MFMA work, 72 V n^2 R flops, dominates for R >= 16).
// The grid runs over a work list of the sites of up to kMaxMultiOps operators
// (a mixed batch of lattices with one block size n): workgroup x belongs to the
// operator whose site range [site0, site0 + V) contains it; grid.y tiles the
// right-hand sides of the operator with the most, tiles past an operator's own
// count exit at entry.
template <int NP, int P, typename VT, int RB>
__global__ __launch_bounds__(256) void k_apply_multi(MultiOps ops) {
  static_assert(RB % 16 == 0 && RB <= 64, "right-hand-side tile of 16, 32 or 64");
  using acc_t = typename Mfma<VT>::acc_t;
  // select this workgroup's operator (uniform; fields copied by select so the
  // kernel-argument array is never indexed dynamically)
  int o = 0;
#pragma unroll
  for (int i = 1; i < kMaxMultiOps; ++i)
    if (i < ops.n_ops && int(blockIdx.x) >= ops.op[i].site0) o = i;
  const void* blocks = ops.op[0].blocks;
  const float* scales = ops.op[0].scales;
  const int* nbr = ops.op[0].nbr;
  const void* const* xin_v = ops.op[0].xin;
  void* const* yout_v = ops.op[0].yout;
  int V = ops.op[0].V, R = ops.op[0].R, site0 = ops.op[0].site0;
  double tm = ops.op[0].tm;
#pragma unroll
  for (int i = 1; i < kMaxMultiOps; ++i)
    if (i == o) {
      blocks = ops.op[i].blocks;
      scales = ops.op[i].scales;
      nbr = ops.op[i].nbr;
      xin_v = ops.op[i].xin;
      yout_v = ops.op[i].yout;
      V = ops.op[i].V;
      R = ops.op[i].R;
      site0 = ops.op[i].site0;
      tm = ops.op[i].tm;
    }
  const int n = ops.n, g5io = ops.g5io;
  const auto* const* xin = reinterpret_cast<const cx<VT>* const*>(xin_v);
  auto* const* yout = reinterpret_cast<cx<VT>* const*>(yout_v);
  if (int(blockIdx.y) * RB >= R) return;
  constexpr int LD = NP + 1;                  // padded row stride of every LDS plane
  extern __shared__ unsigned char smem[];
  VT* Mr = reinterpret_cast<VT*>(smem);       // [NP][LD] coupling matrix, real part
  VT* Mi = Mr + NP * LD;                      // imaginary part
  VT* Pr = Mi + NP * LD;                      // [RB][LD] panel: row r = x_r at the source
  VT* Pi = Pr + RB * LD;
  const int site = int(blockIdx.x) - site0;
  const int r0 = blockIdx.y * RB;
  const int Rc = min(RB, R - r0);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int l16 = lane & 15, lk = lane >> 4;
  const int T = (n + 7) / 8, TT = T * T;
  constexpr int epl = (P == P64) ? 1 : (P == P32 ? 2 : 4);   // block entries per 16-byte unit
  const int upl = (TT + epl - 1) / epl;                      // units per lane of a block
  const int nunits = 64 * upl;
  const int half = n >> 1;
  // output tiles (16 x 16): RT row tiles x RB/16 column tiles; a partial
  // right-hand-side tile computes on zero padding and stores only its Rc
  // columns.  FP32 products: every wave gets the same share of MFMA work --
  // the k range is split KS ways (KS = 4 / gcd(NT, 4)) and wave w takes k
  // part w % KS of the TPW tiles (w / KS) TPW .. + TPW - 1 (3 row tiles x 1
  // column tile, n = 48 with 16 right-hand sides, give each wave all 3 tiles
  // over a quarter of k), the KS partial panels summed in LDS at the end.
  // FP64 products keep one k range per tile (tile t = wave + 4 i): their
  // wider accumulators would cost the occupancy the balance gains.
  constexpr bool SPLIT = sizeof(VT) == 4;
  constexpr int RT = NP / 16;
  constexpr int NT = RT * (RB / 16);
  constexpr int KS = !SPLIT ? 1 : ((NT % 4 == 0) ? 1 : ((NT % 2 == 0) ? 2 : 4));
  constexpr int TPW = SPLIT ? NT * KS / 4 : (NT + 3) / 4;   // tiles per wave
  constexpr int KSTEPS = NP / 4 / KS;   // 4-deep k steps per wave
  static_assert((NP / 4) % KS == 0, "k range splits evenly");
  const int kpart = wave % KS, tile0 = (wave / KS) * TPW;
  auto tile_of = [&](int it) { return SPLIT ? tile0 + it : wave + 4 * it; };
  // Staging with 16-byte loads.  Blocks: thread t takes units u = t + 256 s of
  // the tiled block (lane u % 64, unit u / 64 of that lane), each holding epl
  // entries whose (row, column) are fixed per thread and computed once.
  // Panel: thread t takes 16-byte chunks c = t + 256 s (right-hand side c / CPR,
  // chunk c % CPR of its n entries at the source site).
  constexpr int TMAX = NP / 8;
  constexpr int MU = (64 * ((TMAX * TMAX + epl - 1) / epl) + 255) / 256;
  constexpr int VPC = 16 / int(sizeof(cx<VT>));             // vector entries per chunk
  constexpr int CPRMAX = NP / VPC;
  constexpr int PU = (RB * CPRMAX + 255) / 256;
  const int cpr = n / VPC;                                   // chunks per right-hand side
  int uoff[MU];                  // unit offset in the block (in 16-byte units), -1 if none
  int ij[MU][epl];               // packed (row, column) of each entry, -1 if padding
#pragma unroll
  for (int s2 = 0; s2 < MU; ++s2) {
    const int u = threadIdx.x + 256 * s2;
    uoff[s2] = -1;
#pragma unroll
    for (int q = 0; q < epl; ++q) ij[s2][q] = -1;
    if (u < nunits) {
      const int l = u % 64, k = u / 64;
      uoff[s2] = k * 64 + l;
#pragma unroll
      for (int q = 0; q < epl; ++q) {
        const int e = k * epl + q;
        if (e < TT) {
          const int i = (l / 8) * T + e / T, j = (l % 8) * T + e % T;
          if (i < n && j < n) ij[s2][q] = (i << 8) | j;
        }
      }
    }
  }
  const cx<VT>* prow[PU];        // this thread's panel chunk sources (right-hand-side base)
  int pr_[PU], pk_[PU];          // right-hand side and first component of each chunk
#pragma unroll
  for (int s2 = 0; s2 < PU; ++s2) {
    const int c = threadIdx.x + 256 * s2;
    const int r = c / cpr, k = (c % cpr) * VPC;
    pr_[s2] = -1;
    pk_[s2] = k;
    prow[s2] = nullptr;
    if (c < RB * cpr && r < Rc) {
      pr_[s2] = r;
      prow[s2] = xin[r0 + r];
    }
  }
  // zero both planes once: padding rows / columns are never written again
  for (int t = threadIdx.x; t < 2 * (NP + RB) * LD; t += blockDim.x) Mr[t] = VT(0);
  __syncthreads();   // the zero fill must land before any staged value
  // three real products per complex one: Re C = Mr Pr - Mi Pi,
  // Im C = (Mr + Mi)(Pr + Pi) - Mr Pr - Mi Pi
  acc_t crr[TPW], cii[TPW], css[TPW];
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    crr[t] = acc_t{0, 0, 0, 0};
    cii[t] = acc_t{0, 0, 0, 0};
    css[t] = acc_t{0, 0, 0, 0};
  }
  uint4 mreg[MU], preg[PU];      // the next coupling's raw 16-byte units
  int cblk = 0, csrc = 0;
  float csc = 1.0f;
  auto fetch = [&](int c, int& blk, int& src, float& sc) {
    // coupling c: 0 self, 1..4 forward hop mu = c-1, 5..8 backward hop mu = c-5
    if (c == 0) {
      src = site;
      blk = site * 5;
    } else if (c < 5) {
      src = nbr[(c - 1) * V + site];
      blk = site * 5 + c;
    } else {
      src = nbr[(4 + c - 5) * V + site];       // x - mu
      blk = src * 5 + (c - 4);                 // B[x-mu, mu]
    }
    sc = (P == P16S) ? scales[blk] : 1.0f;
    const uint4* bu = reinterpret_cast<const uint4*>(blocks) + size_t(blk) * size_t(upl) * 64;
#pragma unroll
    for (int s2 = 0; s2 < MU; ++s2)
      mreg[s2] = uoff[s2] >= 0 ? bu[uoff[s2]] : make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int s2 = 0; s2 < PU; ++s2)
      preg[s2] = pr_[s2] >= 0
                     ? *reinterpret_cast<const uint4*>(prow[s2] + size_t(src) * n + pk_[s2])
                     : make_uint4(0, 0, 0, 0);
  };
  fetch(0, cblk, csrc, csc);
  for (int c = 0; c < 9; ++c) {
    const bool trans = c >= 5;
    const float sc = csc;
    // raw units -> LDS planes (the previous coupling's products are done)
#pragma unroll
    for (int s2 = 0; s2 < MU; ++s2) {
      const uint32_t w[4] = {mreg[s2].x, mreg[s2].y, mreg[s2].z, mreg[s2].w};
#pragma unroll
      for (int q = 0; q < epl; ++q) {
        const int pij = ij[s2][q];
        if (pij < 0) continue;
        const int bi = pij >> 8, bj = pij & 255;
        VT re, im;
        if (P == P64) {
          re = VT(__builtin_bit_cast(double, (uint64_t(w[1]) << 32) | w[0]));
          im = VT(__builtin_bit_cast(double, (uint64_t(w[3]) << 32) | w[2]));
        } else if (P == P32) {
          re = VT(__builtin_bit_cast(float, w[2 * q]));
          im = VT(__builtin_bit_cast(float, w[2 * q + 1]));
        } else {
          re = VT(lo_h(w[q]) * sc);
          im = VT(hi_h(w[q]) * sc);
        }
        int i = bi, j = bj;
        if (trans) {
          // backward hop Gamma5 B^H Gamma5: M[i][j] = g_i g_j conj(B[j][i])
          i = bj;
          j = bi;
          const VT sg = ((i < half) == (j < half)) ? VT(1) : VT(-1);
          re = sg * re;
          im = -sg * im;
        }
        if (c == 0 && i == j) im += VT(i < half ? tm : -tm);  // i * tm * Gamma5
        Mr[i * LD + j] = re;
        Mi[i * LD + j] = im;
      }
    }
#pragma unroll
    for (int s2 = 0; s2 < PU; ++s2) {
      if (pr_[s2] < 0) continue;
      const uint32_t w[4] = {preg[s2].x, preg[s2].y, preg[s2].z, preg[s2].w};
      const int r = pr_[s2];
#pragma unroll
      for (int q = 0; q < VPC; ++q) {
        const int k = pk_[s2] + q;
        VT re, im;
        if (sizeof(VT) == 8) {
          re = VT(__builtin_bit_cast(double, (uint64_t(w[1]) << 32) | w[0]));
          im = VT(__builtin_bit_cast(double, (uint64_t(w[3]) << 32) | w[2]));
        } else {
          re = VT(__builtin_bit_cast(float, w[2 * q]));
          im = VT(__builtin_bit_cast(float, w[2 * q + 1]));
        }
        if ((g5io & 1) && k >= half) {
          re = -re;
          im = -im;
        }
        Pr[r * LD + k] = re;
        Pi[r * LD + k] = im;
      }
    }
    __syncthreads();
    // the next coupling's loads are in flight while this one multiplies
    if (c + 1 < 9) fetch(c + 1, cblk, csrc, csc);
    // C += M P with the three products Mr Pr, Mi Pi, (Mr + Mi)(Pr + Pi)
    // (16x16x4 tiles), k outermost so the wave's tiles interleave their MFMA
    // chains
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) {
      const int k = 4 * (kpart * KSTEPS + ks);
#pragma unroll
      for (int it = 0; it < TPW; ++it) {
        const int t = tile_of(it);
        if (SPLIT || t < NT) {   // split tiles always exist
          const int rt = t % RT, ct = t / RT;
          const int ao = (rt * 16 + l16) * LD + lk + k, bo = (ct * 16 + l16) * LD + lk + k;
          const VT a_r = Mr[ao], a_i = Mi[ao], b_r = Pr[bo], b_i = Pi[bo];
          crr[it] = Mfma<VT>::mma(a_r, b_r, crr[it]);
          cii[it] = Mfma<VT>::mma(a_i, b_i, cii[it]);
          css[it] = Mfma<VT>::mma(a_r + a_i, b_r + b_i, css[it]);
        }
      }
    }
    __syncthreads();
  }
  // accumulators -> LDS panel planes (row r = right-hand side) -> coalesced
  // stores; the k parts add their partial panels one after another
#pragma unroll
  for (int part = 0; part < KS; ++part) {
    if (kpart == part) {
#pragma unroll
      for (int it = 0; it < TPW; ++it) {
        const int t = tile_of(it);
        if (!SPLIT && t >= NT) continue;
        const int rt = t % RT, ct = t / RT;
        const int col = ct * 16 + l16;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          // accumulator value q of a lane: row 4*(lane/16)+q for the FP32
          // 16x16x4 MFMA, row lane/16 + 4*q for the FP64 one
          const int row = rt * 16 + Mfma<VT>::row(lk, q);
          const VT re = crr[it][q] - cii[it][q], im = css[it][q] - crr[it][q] - cii[it][q];
          if (part == 0) {
            Pr[col * LD + row] = re;
            Pi[col * LD + row] = im;
          } else {
            Pr[col * LD + row] += re;
            Pi[col * LD + row] += im;
          }
        }
      }
    }
    __syncthreads();
  }
  for (int t = threadIdx.x; t < Rc * n; t += blockDim.x) {
    const int r = t / n, i = t % n;
    cx<VT> z = mk(Pr[r * LD + i], Pi[r * LD + i]);
    if ((g5io & 2) && i >= half) z = mk(VT(-z.re), VT(-z.im));
    yout[r0 + r][size_t(site) * n + i] = z;
  }
}

// ---- FP32 vectors: FP16 pieces on the FP16 matrix cores
// The FP32 matrix instructions run at 1/16 of the FP16 rate.  An FP32 number
// scaled by a power of two is the sum of two FP16 numbers, h = fp16(x) and l =
// fp16(x - h), to 2^-24 of its magnitude, so a product of two is h h' + h l' + l h'
// to about its own FP32 rounding error (the dropped l l' is below 2^-24 of it):
// three FP16 products with FP32 accumulation.  FP16-stored blocks are one exact
// piece: two products.  Scales: each block by a power of two of its largest
// entry (kept at build time), each right-hand side's n entries at a source site
// by one of theirs, both to [2^14, 2^15), undone in FP32 on the coupling's
// accumulators; entries far below the largest keep 2^-39 of it.  Error against
// 64 bits, 16^4, n = 48, 64 right-hand sides: 1.2e-7 (FP32 matrix instructions
// with three real products per complex one: 6.3e-7).
// Layout: complex values stay interleaved, (re, im) pairs are two k entries:
// Re = (ar, ai) . (pr, -pi), Im = (ar, ai) . (pi, pr), on 16x16x32 tiles (16
// complex columns per step).  One workgroup per site and RB right-hand sides:
// its four waves take the RB / 16 column tiles, and the row tiles where there
// are fewer.  The couplings' blocks go through LDS as FP16 pairs (double
// buffered, one barrier per coupling, rows padded to an odd number of 16-byte
// units: conflict-free fragment reads); the panels go from memory to the wave
// that multiplies them, which holds its fragments in registers.
// Measured (16^4, n = 48, 64 right-hand sides; FP32 matrix instructions and
// planes in LDS before): FP32 6.69 -> 4.55 ms, FP16 blocks 6.88 -> 3.99 ms; 8^4:
// 0.69 -> 0.25 ms.  Matrix cores 20%, vector ALU (the splits) 39% busy; what is
// left is the wait for panels and blocks (19 GB through the L2s, 7.7 GB once
// each).  At three waves per SIMD the registers spill: 5.9 ms.

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

// Power-of-two scale that takes a largest magnitude m to [2^14, 2^15), and its
// inverse; both stay normal numbers (m below 2^-112 scales to less, infinite
// and NaN m leave finite factors, so they reach the result).
__device__ inline void pow2_scale(float m, float& up, float& down) {
  const uint32_t e = max((__float_as_uint(m) >> 23) & 255u, 15u);   // biased exponent
  up = __uint_as_float((268u - e) << 23);
  down = __uint_as_float((e - 14u) << 23);
}

// FP16 pieces of a scaled complex value, packed (re low, im high).
__device__ inline void split_pair(float re, float im, uint32_t& hi, uint32_t& lo) {
  const h2 h = __builtin_convertvector(f2{re, im}, h2);
  const h2 l = __builtin_convertvector(f2{re - float(h.x), im - float(h.y)}, h2);
  hi = __builtin_bit_cast(uint32_t, h);
  lo = __builtin_bit_cast(uint32_t, l);
}

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

template <int T, int P, int RB>
__global__ __launch_bounds__(256, 2) void k_apply_multi_split(MultiOps ops,
                                                                          unsigned sites, int chunk) {
  constexpr int NP = (8 * T + 15) / 16 * 16;      // block edge padded to whole tiles
  constexpr int PIECES = (P == P32) ? 2 : 1;      // FP16 pieces of a block
  constexpr int RT = NP / 16, KS = NP / 16;       // row tiles, k steps of 16 complex columns
  constexpr int CT = RB / 16, RG = 4 / CT;        // column tiles, waves per column tile
  constexpr int RTW = (RT + RG - 1) / RG;         // row tiles per wave
  constexpr int LDA = (NP + 4) * 4;               // bytes of an LDS row (NP pairs + padding)
  constexpr int PLANE = NP * LDA + 16;            // + a word that takes padding entries
  constexpr int TT = T * T;
  constexpr int EPL = (P == P32) ? 2 : 4;         // block entries per 16-byte unit
  constexpr int UPL = (TT + EPL - 1) / EPL;       // units per lane of a block
  constexpr int MU = (UPL + 3) / 4;               // units per thread
  __shared__ __align__(16) unsigned char lds[2 * PIECES * PLANE];
  // XCD-aware order: each XCD takes a contiguous range of sites, so neighbouring
  // sites share blocks and panels through its L2
  const unsigned item = (blockIdx.x & 7u) * unsigned(chunk) + (blockIdx.x >> 3);
  if (item >= sites) return;
  int o = 0;
#pragma unroll
  for (int i = 1; i < kMaxMultiOps; ++i)
    if (i < ops.n_ops && int(item) >= ops.op[i].site0) o = i;
  MultiOpDesc op = ops.op[0];
#pragma unroll
  for (int i = 1; i < kMaxMultiOps; ++i)
    if (i == o) op = ops.op[i];
  const int n = ops.n, half = n >> 1, R = op.R, V = op.V;
  const int r0 = int(blockIdx.y) * RB;
  if (r0 >= R) return;
  const int site = brick_site(op, item - unsigned(op.site0));
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int l16 = lane & 15, lk = lane >> 4;
  const int lr = lane >> 3, lc = lane & 7;
  const int ct = wave % CT, rg = wave / CT;
  const bool g5in = (ops.g5io & 1) != 0, g5out = (ops.g5io & 2) != 0;
  const auto blocks = (gptr<u4>)op.blocks;
  const auto scales = (gptr<float>)op.scales;   // FP16: block scales; FP32: largest magnitudes
  const auto nbr = (gptr<int>)op.nbr;

  // Unit k = wave + 4 s of the tiled block, entries e = k EPL + q = a T + b: lane
  // (lr, lc) holds (lr T + a, lc T + b).  Its LDS byte offset is a lane part plus
  // a wave-uniform one, as it is or transposed.  Entries past the n x n block but
  // inside the tiled layout are zeros there and land in the padding of the
  // plane; the slots of a unit past the tile go to the spare word.
  const int lbase = lr * T * LDA + lc * T * 4, lbase_t = lc * T * LDA + lr * T * 4;
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
  const int rc = min(r0 + ct * 16 + l16, R - 1);  // lanes past R repeat the last column
  const auto xr = (gptr<z32>)(((gptr<const void*>)op.xin)[rc]);
  // panel entries 16 ks + 4 lk + 2 q and the next; past n the last pair is read
  // again (the blocks are zero there)
  int joff[KS][2];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
#pragma unroll
    for (int q = 0; q < 2; ++q) joff[ks][q] = min(16 * ks + 4 * lk + 2 * q, n - 2);

  u4 araw[MU];
  f4 braw[KS][2];
  auto load_block = [&](int blk) {
    const auto b = blocks + size_t(blk) * (64 * UPL) + lane;
#pragma unroll
    for (int s = 0; s < MU; ++s) {
      const int k = wave + 4 * s;
      if (UPL % 4 == 0 || k < UPL) araw[s] = b[k * 64];
    }
  };
  auto load_panel = [&](int src) {
    const auto x = xr + size_t(src) * n;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int q = 0; q < 2; ++q) braw[ks][q] = *(gptr<f4>)(x + joff[ks][q]);
  };
  auto store_block = [&](unsigned char* buf, float scale, bool trans) {
    float up = 1.f, down = 1.f;
    if (P == P32) pow2_scale(scale, up, down);
    // transposed: Gamma5 B^H Gamma5 = g_i g_j conj(B[j][i]); the masks negate
    // the imaginary (+) or the real part (-) of a packed pair
    unsigned char* base = buf + (trans ? lbase_t : lbase);
#pragma unroll
    for (int s = 0; s < MU; ++s) {
      const int k = wave + 4 * s;
      if (UPL % 4 != 0 && k >= UPL) continue;
#pragma unroll
      for (int q = 0; q < EPL; ++q) {
        const int e = k * EPL + q;
        const int a = e / T, b = e - a * T;
        uint32_t hi, lo = 0;
        if constexpr (P == P32)
          split_pair(__uint_as_float(araw[s][2 * q]) * up, __uint_as_float(araw[s][2 * q + 1]) * up,
                     hi, lo);
        else
          hi = araw[s][q];
        unsigned char* at = base + (trans ? b * LDA + a * 4 : a * LDA + b * 4);
        if (TT % EPL != 0 && e >= TT) at = buf + NP * LDA;
        if (trans) {
          const uint32_t m = (lr * T + a < half) == (lc * T + b < half) ? 0x80000000u : 0x00008000u;
          hi ^= m;
          lo ^= m;
        }
        *reinterpret_cast<uint32_t*>(at) = hi;
        if (PIECES == 2) *reinterpret_cast<uint32_t*>(at + PLANE) = lo;
      }
    }
  };

  f4 tre[RTW], tim[RTW];
#pragma unroll
  for (int t = 0; t < RTW; ++t) tre[t] = tim[t] = f4{0.f, 0.f, 0.f, 0.f};
  load_block(block_of(0));
  load_panel(site);
  // rows and columns past the tiled layout stay zero
  if (NP != 8 * T) {
    for (int t = threadIdx.x * 16; t < 2 * PIECES * PLANE; t += 256 * 16)
      *reinterpret_cast<u4*>(lds + t) = u4{0, 0, 0, 0};
    __syncthreads();
  }
  store_block(lds, scale_of(0), false);
  load_block(block_of(1));
#pragma unroll 1
  for (int c = 0; c < 9; ++c) {
    unsigned char* buf = lds + (c & 1) * (PIECES * PLANE);
    __syncthreads();   // buf is complete, and the other buffer's products are done
    // this coupling's panel -> scaled FP16 fragments
    float mx = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        mx = fmaxf(fmaxf(mx, fabsf(braw[ks][q].x)), fabsf(braw[ks][q].y));
        mx = fmaxf(fmaxf(mx, fabsf(braw[ks][q].z)), fabsf(braw[ks][q].w));
      }
    mx = fmaxf(mx, shfl_xor(mx, 16));
    mx = fmaxf(mx, shfl_xor(mx, 32));
    float up, down;
    pow2_scale(mx, up, down);
    u4 bh[KS], bl[KS];     // (pi, pr) pairs: the Im operand
    u4 bhr[KS], blr[KS];   // (pr, -pi): swapped, the high half negated
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        float u0 = up, u1 = up;
        if (g5in) {
          u0 = joff[ks][q] < half ? up : -up;
          u1 = joff[ks][q] + 1 < half ? up : -up;
        }
        const f4 z = braw[ks][q];
        uint32_t h[2], l[2];
        split_pair(z.y * u0, z.x * u0, h[0], l[0]);
        split_pair(z.w * u1, z.z * u1, h[1], l[1]);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          bh[ks][2 * q + i] = h[i];
          bl[ks][2 * q + i] = l[i];
          bhr[ks][2 * q + i] = __builtin_amdgcn_alignbit(h[i], h[i], 16) ^ 0x80000000u;
          blr[ks][2 * q + i] = __builtin_amdgcn_alignbit(l[i], l[i], 16) ^ 0x80000000u;
        }
      }
    float fblk = scale_of(c);
    if (P == P32) {
      float u;
      pow2_scale(fblk, u, fblk);
    }
    // the next panel and block are in flight, and the next block's pieces are
    // written, while this coupling multiplies
    if (c + 1 < 9) {
      load_panel(source(c + 1));
      unsigned char* nb = lds + ((c + 1) & 1) * (PIECES * PLANE);
      if (coupling(c + 1) < 5) store_block(nb, scale_of(c + 1), false);
      else store_block(nb, scale_of(c + 1), true);
      if (c + 2 < 9) load_block(block_of(c + 2));
    }
#pragma unroll
    for (int t = 0; t < RTW; ++t) {
      const int rt = rg + t * RG;
      if (RT % RG != 0 && rt >= RT) continue;
      const unsigned char* row = buf + (rt * 16 + l16) * LDA + lk * 16;
      f4 are = f4{0.f, 0.f, 0.f, 0.f}, aim = are;
      h8 ah[KS];
      // small products first
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        ah[ks] = *reinterpret_cast<const h8*>(row + ks * 64);
        are = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[ks], __builtin_bit_cast(h8, blr[ks]), are, 0, 0, 0);
        aim = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[ks], __builtin_bit_cast(h8, bl[ks]), aim, 0, 0, 0);
        if constexpr (PIECES == 2) {
          const h8 al = *reinterpret_cast<const h8*>(row + PLANE + ks * 64);
          are = __builtin_amdgcn_mfma_f32_16x16x32_f16(al, __builtin_bit_cast(h8, bhr[ks]), are, 0, 0, 0);
          aim = __builtin_amdgcn_mfma_f32_16x16x32_f16(al, __builtin_bit_cast(h8, bh[ks]), aim, 0, 0, 0);
        }
      }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        are = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[ks], __builtin_bit_cast(h8, bhr[ks]), are, 0, 0, 0);
        aim = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[ks], __builtin_bit_cast(h8, bh[ks]), aim, 0, 0, 0);
      }
      // scales undone in FP32: the column's own, then the block's
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        tre[t][q] = fmaf(are[q] * down, fblk, tre[t][q]);
        tim[t][q] = fmaf(aim[q] * down, fblk, tim[t][q]);
      }
    }
  }
  // lane: rows 16 rt + 4 lk .. + 3 of right-hand side r; i tm Gamma5 x added here
  if (r0 + ct * 16 + l16 >= R) return;
  const auto y = (gptr_w<z32>)(((gptr<void*>)op.yout)[rc]) + size_t(site) * n;
  const auto xs = xr + size_t(site) * n;
  const float tm = float(op.tm);
#pragma unroll
  for (int t = 0; t < RTW; ++t) {
    const int rt = rg + t * RG;
    if (RT % RG != 0 && rt >= RT) continue;
#pragma unroll
    for (int q = 0; q < 4; q += 2) {
      const int i = rt * 16 + lk * 4 + q;
      if (i >= n) continue;
      f4 z = {tre[t][q], tim[t][q], tre[t][q + 1], tim[t][q + 1]};
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

size_t multi_lds_bytes(int n, bool dbl, int rb) {
  const int np = multi_np(n);
  return size_t(2) * (size_t(np) + rb) * (np + 1) * (dbl ? sizeof(double) : sizeof(float));
}

template <int NP, int P, typename VT, int RB>
static void multi_launch(const MultiOps& ops, unsigned sites, int rmax, hipStream_t st) {
  const size_t lds = multi_lds_bytes(ops.n, sizeof(VT) == 8, RB);
  DC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_apply_multi<NP, P, VT, RB>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)));
  const unsigned rtiles = unsigned((rmax + RB - 1) / RB);
  hipLaunchKernelGGL((k_apply_multi<NP, P, VT, RB>), dim3(sites, rtiles), dim3(256), lds, st, ops);
  DC_HIP(hipGetLastError());
}

template <int T, int P, int RB>
static void split_launch(const MultiOps& ops, unsigned sites, int rmax, hipStream_t st) {
  const int chunk = int((sites + 7) / 8);
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

template <int NP>
static void multi_np_launch(int rb, const MultiOps& ops, unsigned sites, int rmax, hipStream_t st) {
  if (rb == 16) multi_launch<NP, P64, double, 16>(ops, sites, rmax, st);
  else multi_launch<NP, P64, double, 32>(ops, sites, rmax, st);
}

static void multi_dispatch(Prec p, int rb, const MultiOps& ops, unsigned sites, int rmax,
                           hipStream_t st) {
  if (p == P32) return split_T_launch<P32>(rb, ops, sites, rmax, st);
  if (p == P16S) return split_T_launch<P16S>(rb, ops, sites, rmax, st);
  switch (multi_np(ops.n)) {
    case 16: multi_np_launch<16>(rb, ops, sites, rmax, st); break;
    case 32: multi_np_launch<32>(rb, ops, sites, rmax, st); break;
    case 48: multi_np_launch<48>(rb, ops, sites, rmax, st); break;
    case 64: multi_np_launch<64>(rb, ops, sites, rmax, st); break;
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
