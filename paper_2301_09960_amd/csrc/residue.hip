// Products of exact integers by residues modulo pairwise coprime bases
// (residue.h): split into residue planes, one INT8 matrix product per plane,
// and the Chinese remainder combination into the components of C.
//
// k_residue_split: one workgroup per 32 x 32 block of an operand.  The element's
// integer W is formed in 32-bit words, rounded to nearest (ties to even), and
// written in signed bytes; its residues modulo 32 bases are a matrix product
// (bases x bytes) (bytes x elements) with the residues of 256^j on the INT8 matrix
// cores, each reduced by one binary32 quotient.  Each plane of the block is
// written by one coalesced 4-byte store per thread.
//
// k_gemm_residue: gemm_int8_tile over the units of a plan.  A unit's exact sum
// is reduced modulo its base in registers and leaves as one byte per entry (the
// digit GEMM writes four): 7 vector instructions per entry after
// k / 32 matrix-core instructions per 32 x 32 block.
//
// k_residue_combine: V = sum_p t_p w_p over the planes in base-256 digits, a
// matrix product (digits x planes) (planes x entries) on the INT8 matrix cores,
// carried into words; then X = V - q M with q = rint(V / M) in binary64, and
// the components read off the leading bits of X.
//
// Measured at n = 4096, E = 16 (before: the digit pairs of int8.hip): DD 32
// products, 8.58 -> 2.63 ms (GEMM 8.14 -> 2.16 ms, 2.04 POP/s); QD 72 products,
// 28.9 -> 6.00 ms (GEMM 27.1 -> 4.58 ms).  256 DD products of 64 to 1024 as one
// batch: 4.69 -> 2.92 ms.
#include "residue.h"

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <map>
#include <mutex>
#include <tuple>

#include "int8_tile.h"
#include "mp_device.h"
#include "window.h"

namespace mp {
namespace {

constexpr int kThreads = 256;

// ---------------------------------------------------------------------------
// Constants of the bases.
// ---------------------------------------------------------------------------
struct Bases {
  int s[kNumBases];
};
constexpr Bases make_bases() {
  Bases b{};
  int n = 0;
  for (int c = 256; c > 1 && n < kNumBases; --c) {
    bool ok = true;
    for (int i = 0; i < n && ok; ++i) {
      int x = b.s[i], y = c;
      while (y) {
        const int t = x % y;
        x = y;
        y = t;
      }
      ok = x == 1;
    }
    if (ok) b.s[n++] = c;
  }
  return b;
}
constexpr Bases kHostBases = make_bases();
static_assert(kHostBases.s[0] == 256 && kHostBases.s[kNumBases - 1] == 29, "the greedy coprime sequence");

constexpr int kSplitRows = 64;
struct BaseInfo {
  int s;
  int c16;        // 2^16 mod s, balanced
  float inv;      // 1 / s
  uint32_t sinv;  // odd s: s^-1 mod 2^32
};
struct BaseTables {
  BaseInfo info[kSplitRows];  // bases, then ones
  float inv[kSplitRows];
  int ns[kSplitRows];  // -s
};
constexpr BaseTables make_tables() {
  BaseTables t{};
  for (int u = 0; u < kSplitRows; ++u) {
    const int s = u < kNumBases ? kHostBases.s[u] : 1;
    int c16 = 65536 % s;
    if (2 * c16 > s) c16 -= s;
    uint32_t inv = 1;
    if (s % 2)
      for (int i = 0; i < 5; ++i) inv *= 2u - (uint32_t)s * inv;  // Newton: s inv = 1 mod 2^32
    t.info[u] = {s, c16, 1.0f / (float)s, inv};
    t.inv[u] = 1.0f / (float)s;
    t.ns[u] = -s;
  }
  return t;
}
__constant__ BaseTables kBase = make_tables();

// Operands of the split's matrix products: rows u < 64 hold the balanced residues
// c of 256^j modulo base u, rows 64 + u the balanced (256^j - c) / s modulo s, so
// that 256^j = c + s h modulo s^2.  Bytes j = 0 .. 31 as blocks of 32 rows for the
// 32x32x32 instruction (lane l: row l % 32, bytes 16 (l / 32) + t), and j = 0 .. 15
// and 32 .. 47 for the 32x32x16 one (bytes 8 (l / 32) + t).
struct SplitRows {
  int8_t k32[4][64][16], k16[2][4][64][8];
};
constexpr SplitRows make_rows() {
  SplitRows t{};
  for (int u = 0; u < kNumBases; ++u) {
    const int64_t s = kHostBases.s[u];
    int64_t p = 1;  // 256^j mod s^2
    for (int j = 0; j < 48; ++j) {
      int64_t c = p % s;
      if (2 * c > s) c -= s;
      int64_t h = ((p - c) / s) % s;
      if (2 * h > s) h -= s;
      for (int g = 0; g < 2; ++g) {
        const int64_t v = g == 0 ? c : h;
        const int rb = 2 * g + u / 32, row = u % 32;
        if (j < 32) t.k32[rb][row + 32 * (j / 16)][j % 16] = (int8_t)v;
        if (j < 16) t.k16[0][rb][row + 32 * (j / 8)][j % 8] = (int8_t)v;
        if (j >= 32) t.k16[1][rb][row + 32 * ((j - 32) / 8)][j % 8] = (int8_t)v;
      }
      p = p * 256 % (s * s);
    }
  }
  return t;
}
__device__ const SplitRows kRows = make_rows();

// Planes: the first digits of a plan's (or a group's) n bases, then the second
// digits of the squared ones: digit g of base u is plane u + g n.
__host__ __device__ inline int group_planes(int u0, int u1, int nsq) {
  return u1 - u0 + (u0 < nsq ? (u1 < nsq ? u1 : nsq) - u0 : 0);
}

// Low byte of the balanced residue of r modulo the base (|r| < 2^22.2; for
// s = 256 the low byte of r).  q = rint(r / s) comes out of the low bits of
// r / s + 1.5 2^23: the quotient's error, below |r| 2^-24 / s < 0.3 / s, is less
// than the distance 1 / (2 s) of r / s from a half, so q is exact for odd s.
// The bits hold q + 2^22 in 24 bits, and 2^22 s is a multiple of 256.
__device__ __forceinline__ uint32_t residue_byte(int r, const BaseInfo &b) {
  const int qb = __float_as_int(__builtin_fmaf((float)r, b.inv, 12582912.0f));
  return (uint32_t)(__mul24(qb, -b.s) + r);
}
// r = v mod s with |r| < 2^22.2, for |v| < 2^31.
__device__ __forceinline__ int fold16(int v, const BaseInfo &b) {
  return __mul24(v >> 16, b.c16) + (v & 0xffff);
}
// The low bytes of a, b, c, d in one word.
__device__ __forceinline__ uint32_t pack4(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  const uint32_t lo = __builtin_amdgcn_perm(b, a, 0x0c0c0400u), hi = __builtin_amdgcn_perm(d, c, 0x0c0c0400u);
  return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}
// (v - t) / s for t = v mod s in the low byte of `byte` (balanced): exact.
__device__ __forceinline__ int divide_out(int v, uint32_t byte, const BaseInfo &b) {
  const int d = v - (int)(int8_t)byte;
  return b.s == 256 ? d >> 8 : (int)((uint32_t)d * b.sinv);
}

// ---------------------------------------------------------------------------
// Split.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void parts_of(double x, int64_t &M, int &q) { binary64_parts(x, M, q); }
__device__ __forceinline__ void parts_of(float x, int64_t &M, int &q) {
  const uint32_t b = __float_as_uint(x);
  const int ef = (int)((b >> 23) & 0xff);
  const int64_t f = (int64_t)(b & 0x7fffffu);
  const int64_t m = ef == 0 ? f : (f | (int64_t(1) << 23));
  q = ef == 0 ? -149 : ef - 150;
  M = (b >> 31) ? -m : m;
}

// The exponent of a vector with maximum bits mu.
template <typename T>
__device__ __forceinline__ int vector_exponent(typename bits_of<T>::type mu, int float_form) {
  using U = typename bits_of<T>::type;
  if (mu == 0) return kZeroExp;
  if (mu >= (sizeof(T) == 8 ? (U)0x7ff0000000000000ULL : (U)0x7f800000u)) return kNonFinite;
  const T x = from_bits(mu, T(0));
  if (float_form) return ceil_log2(x);
  int ex;
  if constexpr (sizeof(T) == 8)
    (void)frexp(x, &ex);
  else
    (void)frexpf(x, &ex);
  return ex;
}

// One block: bases [u_first, u_end) into planes counted from base u_first's; of
// the row blocks of 32 bases this workgroup takes every parts-th from part on.
// The FLOAT form's checks (below) run with `check`.
//
// The FLOAT form stands for D passes of Algorithm 1, whose grid follows the
// largest residual of the vector: pass 1 rounds to 2^(E - b), and pass a + 1 to
// b bits below the exponent e of the residual that pass a left, |r| <= 2^(g - 1)
// under a grid 2^g.  The fixed grid here must be no coarser than the last
// pass's.  An element whose bits i and i - 1 differ, with nonzero bits below
// them, leaves |r| > 2^(i - 1) under any grid above 2^i, so e >= i and the next
// grid is at least 2^(i - b); with i = g - 1, the usual case, a pass falls b + 1
// bits.  The places where some element of the vector has such a change give a lower
// bound of all D grids (last_grid_covered); random mantissas have one at nearly
// every place, so 32 elements that are not zero settle a vector: its first ones, or,
// where zeros are among them (triangular, banded, sparse operands), others (settle_strip,
// in the launch that finds the maxima).  A vector is safe if that bound says so, or if
// every element of it is exact on the fixed grid.  A vector that is neither, or that
// holds lower components as large as leading ones, sets the flag: the product is then
// formed from the slices.
constexpr int kChangeWords = 12;  // places 0 .. kMaxResidueBits + 1 and the words of a component that starts below them
static_assert(kMaxResidueBits / 32 + 3 <= kChangeWords, "three words a component");
__device__ __forceinline__ bool last_grid_covered(const uint32_t *changes, int bits, int b, int passes) {
  int g = bits - b;  // places count from the fixed grid
  for (int a = 1; a < passes; ++a) {
    int i = -1;  // the highest change below the grid
    for (int w = (g - 1) >> 5; w >= 0 && i < 0; --w) {
      const int top = g - 32 * w;  // places below g in this word
      const uint32_t c = changes[w] & (top >= 32 ? 0xffffffffu : (1u << top) - 1u);
      if (c) i = 32 * w + 31 - __clz((int)c);
    }
    g = i - b;
    if (g < 1) return false;  // one place to spare for the rounding of the leading components
  }
  return true;
}

// ORs the changes of an element, places from 2^(E - bits) up, into `changes`.  A component's two's complement has those of the element between its
// own last change (a borrow of the component below goes no higher) and its sign, so
// each is placed for itself, without its last change and the place above it.  An
// element whose components overlap or touch, or exceed 2^E, adds none.
template <typename T, int C>
__device__ __forceinline__ void add_changes(const T (&x)[C], int E, int bits, uint32_t *changes) {
  uint64_t c[C];
  int off[C], above = E + 2;
  bool apart = true;
#pragma unroll
  for (int r = 0; r < C; ++r) {
    int64_t M;
    int q;
    parts_of(x[r], M, q);
    c[r] = (uint64_t)M ^ ((uint64_t)M << 1);
    const uint64_t low = c[r] & (0u - c[r]);
    c[r] &= ~(low | (low << 1));
    off[r] = q - (E - bits);
    if (M != 0) {
      apart = apart && q + (sizeof(T) == 8 ? 53 : 24) < above;
      above = q;
    }
  }
#pragma unroll
  for (int r = 0; r < C; ++r) {
    if (!apart || off[r] <= -64) continue;
    const int at = off[r] > 0 ? off[r] : 0, sh = at & 31;
    const uint64_t u = off[r] < 0 ? c[r] >> -off[r] : c[r];
    const uint64_t lo = u << sh;
    const uint32_t hi = sh ? (uint32_t)(u >> (64 - sh)) : 0u;
    uint32_t *to = changes + (at >> 5);
    if ((uint32_t)lo) atomicOr(to, (uint32_t)lo);
    if (lo >> 32) atomicOr(to + 1, (uint32_t)(lo >> 32));
    if (hi) atomicOr(to + 2, hi);
  }
}

// Adds M 2^off (two's complement, off >= 0) into the words w: the three words of
// M 2^(off % 32), the sign above and zeros below, moved up by off / 32 in steps of
// 1, 2, 4 and 8 words.
template <int N>
__device__ __forceinline__ void window_add_shifted(uint32_t (&w)[N], int64_t M, int off) {
  const int q = off >> 5, sh = off & 31;
  const uint64_t u = (uint64_t)M << sh;
  const int hi = (int)(M >> 32);
  const uint32_t sign = (uint32_t)(hi >> 31);
  uint32_t a[N];
#pragma unroll
  for (int i = 0; i < N; ++i) a[i] = sign;
  a[0] = (uint32_t)u;
  if constexpr (N > 1) a[1] = (uint32_t)(u >> 32);
  if constexpr (N > 2) a[2] = (uint32_t)((hi >> (31 - sh)) >> 1);
  int filled = 3;  // words that may differ from the sign
#pragma unroll
  for (int st = 1; st < N; st *= 2) {
    const bool up = (q & st) != 0;
    filled += st;
#pragma unroll
    for (int i = N - 1; i >= 0; --i)
      if (i < filled) a[i] = up ? (i >= st ? a[i >= st ? i - st : 0] : 0u) : a[i];
  }
  uint32_t carry = 0;
#pragma unroll
  for (int i = 0; i < N; ++i) w[i] = __builtin_addc(w[i], a[i], carry, &carry);
}

// Whether an element at or just below half a step of its grid rounds up (nearest,
// ties to even).  g: its guard word, the floors of the components in 2^P added up;
// odd: the lowest bit above it.  Ties are common in short data (no floor cut
// anything off: g decides).  Else what the floors left, the fraction of a component
// or a whole one below 2^P, is added to the distance from a half in the components'
// order, which for normalized expansions leaves its sign exact.
template <typename T, int C>
__device__ __forceinline__ bool rounds_up(const T (&x)[C], int P, uint32_t g, bool odd) {
  bool lost = false;
#pragma unroll
  for (int r = 0; r < C; ++r) {
    int64_t M;
    int q;
    parts_of(x[r], M, q);
    const int sh = q >= P ? 0 : P - q < 63 ? P - q : 63;
    lost = lost || (M & ((int64_t(1) << sh) - 1)) != 0;
  }
  if (!lost) return g > 0x80000000u - (odd ? 1u : 0u);
  double d = (double)(int)(g - 0x80000000u), left[C];
#pragma unroll
  for (int r = 0; r < C; ++r) {
    int64_t M;
    int q;
    parts_of(x[r], M, q);
    const int sh = q >= P ? 0 : P - q < 63 ? P - q : 63;
    const bool below = sh > 0 && M >> sh == -1;  // its floor is -1: whole instead
    d += below ? 1.0 : 0.0;
    left[r] = ldexp((double)(below ? M : M & ((int64_t(1) << sh) - 1)), q < P ? q - P : 0);
  }
#pragma unroll
  for (int r = 0; r < C; ++r) d += left[r];
  return d > 0.0 || (d == 0.0 && odd);
}

// The integer W of one element in NW words, rounded to nearest on 32 guard bits, ties
// to even.  With `check`: whether bits were cut off, and whether a lower component is
// as large as leading ones (an infinity or NaN too).
template <typename T, int C, int NW>
__device__ __forceinline__ void element_words(const T (&x)[C], int E, int P, bool check, uint32_t (&W)[12],
                                              bool &inexact, bool &odd) {
  uint32_t w[NW + 1];
#pragma unroll
  for (int i = 0; i <= NW; ++i) w[i] = 0u;
  bool whole = false;  // the last component is there, and so all of the element
#pragma unroll
  for (int r = 0; r < C; ++r) {
    int64_t M;
    int q;
    parts_of(x[r], M, q);
    const int off = q - P;
    const int sh = off >= 0 ? 0 : off > -63 ? -off : 63;
    if (r == C - 1) whole = M != 0 && (M & ((int64_t(1) << sh) - 1)) == 0;
    if (check) {
      if (r > 0 && M != 0 && q + (sizeof(T) == 8 ? 53 : 24) > E - 20) odd = true;
      inexact = inexact || (M & ((int64_t(1) << sh) - 1)) != 0;
    }
    window_add_shifted<NW + 1>(w, M >> sh, off < 0 ? 0 : off);
  }
  inexact = inexact || w[0] != 0u;
  uint32_t carry = w[0] > 0x80000000u - (w[1] & 1u) ? 1u : 0u;
  const bool near_half = !whole && w[0] - (0x80000000u - C) <= (uint32_t)C;
  if (__builtin_expect(__any(near_half), 0)) {
    if (near_half) carry = rounds_up<T, C>(x, P, w[0], (w[1] & 1u) != 0u) ? 1u : 0u;
  }
#pragma unroll
  for (int i = 0; i < NW; ++i) W[i] = __builtin_addc(w[i + 1], 0u, carry, &carry);
}

// The same from the words of W (any element's).
template <int NW>
__device__ __forceinline__ void add_word_changes(const uint32_t (&W)[12], uint32_t (&change)[NW]) {
  bool more = false;  // a change further down
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    uint32_t c = W[i] ^ ((W[i] << 1) | (i > 0 ? W[i > 0 ? i - 1 : 0] >> 31 : 0u));
    const bool here = c != 0u;
    if (!more && here) {  // the lowest change, and the place above it
      const uint32_t low = c & (0u - c);
      c &= ~(low | (low << 1));
    }
    more = more || here;
    change[i] |= c;
  }
}

// State of a vector in the FLOAT form's check.
constexpr int kRounded = 1;    // an element was rounded
constexpr int kUnsettled = 2;  // its first 32 elements leave open how far down its slices reach
constexpr int kSettled = 4;    // others say: no further than the fixed grid

template <int NW>
struct SplitLds {
  static constexpr bool kSmall = NW <= 4, kMore = NW > 8;
  static constexpr int kQ = kSmall ? 2 : 4;  // words per lane of the first instruction
  __attribute__((aligned(16))) uint32_t first[kThreads / 64][4][64][2 * kQ];
  __attribute__((aligned(16))) uint32_t more[kMore ? kThreads / 64 : 1][4][64][4];
  uint32_t seen[kBlk8][NW | 1];  // rows in different banks
  int rounded[kBlk8];
};

// The first place p0 + 16 i of a vector's element that is not zero, or len.
template <typename T>
__device__ __forceinline__ int find_nonzero(const T *x, int64_t sp, int p0, int len) {
  for (int p = p0; p < len; p += 64) {
    T e[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) e[j] = p + 16 * j < len ? x[(int64_t)(p + 16 * j) * sp] : T(0);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (abs_bits(e[j]) != 0) return p + 16 * j;
  }
  return len;
}
template <typename T, int C>
__device__ __forceinline__ void load_element(const T *x, int64_t comp_stride, int64_t sp, int p, int len, T (&e)[C]) {
#pragma unroll
  for (int r = 0; r < C; ++r) e[r] = p < len ? x[r * comp_stride + (int64_t)p * sp] : T(0);
}

// kSettled where sampled elements settle a vector.  A workgroup takes 16 vectors, a
// thread of it every 16th element of one (x), with exponent E: the first two of them
// that are not zero.  all: room for the changes of the 16 vectors, dv this thread's.
template <typename T, int C>
__device__ __forceinline__ int settle_strip(const T *x, int64_t comp_stride, int64_t sp, int len, int dp, int dv, int E,
                                            int bits, int slice_bits, int passes, uint32_t (&all)[16][kChangeWords]) {
  if (threadIdx.x < 16 * kChangeWords) all[threadIdx.x / kChangeWords][threadIdx.x % kChangeWords] = 0u;
  __syncthreads();
  uint32_t *changes = all[dv];
  const bool finite = E != kZeroExp && E != kNonFinite;
  if (finite) {
    int p = dp - 16;
#pragma unroll 1
    for (int j = 0; j < 2; ++j) {
      T e[C];
      p = find_nonzero(x, sp, p + 16, len);
      load_element<T, C>(x, comp_stride, sp, p, len, e);
      add_changes<T, C>(e, E, bits, changes);
    }
  }
  __syncthreads();
  return finite && last_grid_covered(changes, bits, slice_bits, passes) ? kSettled : 0;
}

// Bound by memory for DD (1.6 GB at 3.3 TB/s, the planes in 1 KiB pieces; n = 4096)
// and by vector instructions from TD on: 4 per residue (conversion, quotient,
// remainder, byte) against 4 + words / 4 with v_dot4 sums, and the words placed by
// a shift in powers of two instead of one select chain per word.  Against those:
// DD n = 4096 (32 planes) 616 -> 496 us, QD (68 planes) 1566 -> 1334 us.  The chains
// of a residue are hidden by wavefronts only: four to a SIMD (operands in LDS, the
// checks before the products, scalar constants) against two or three took FLOAT DD
// (37 planes) from 781 to 611 us, QD from 1334 to 1091; now 581 and 1087, ties to even
// included (2 and 9 us).
template <typename T, int C, int NW, int ORIENT>
__device__ void residue_block(const ResidueOperand<T> &op, int64_t blk, bool live_only, int u_first, int u_end,
                              int part, int parts, bool check, SplitLds<NW> &lds) {
  using U = typename bits_of<T>::type;
  const int64_t nb = live_only ? ceil_div((int64_t)op.nvec, (int64_t)kBlk8) : op.nbp;
  const int64_t kbn = live_only ? ceil_div((int64_t)op.len, (int64_t)kKBlk8) : op.kbp;
  // A (rows, contiguous along the row index): walk row blocks fastest;
  // B (columns, contiguous along k): walk k blocks fastest.
  const int64_t vb = ORIENT == 0 ? blk % nb : blk / kbn;
  const int64_t kb = ORIENT == 0 ? blk / nb : blk % kbn;
  const int t = threadIdx.x, l = t >> 2, lane = t % 64;
  const int v = (int)(vb * kBlk8) + (l & 31);
  const int p0 = (int)(kb * kKBlk8) + 16 * (l >> 5) + 4 * (t & 3);
  int E = kZeroExp;
  if (v < op.nvec) E = vector_exponent<T>(static_cast<const U *>(op.mu)[v], op.float_form);
  const bool finite = E != kZeroExp && E != kNonFinite;
  const int P = finite ? E - op.bits - 32 : 0;  // place of the window's lowest bit: 32 guard bits
  // Matrix operands of the elements (columns) in LDS, each wavefront's its own:
  // words 0 .. 7 for the 32x32x32 instruction (with up to 4 words 0 .. 3 for the
  // 32x32x16 one), then words 8 .. 11.  Held in registers they left two or three
  // wavefronts to a SIMD, and the kernel waits on its chains.
  constexpr bool kSmall = SplitLds<NW>::kSmall, kMore = SplitLds<NW>::kMore;
  constexpr int kQ = SplitLds<NW>::kQ;
  auto &first_words = lds.first[t / 64];
  auto &more_words = lds.more[kMore ? t / 64 : 0];
  const int flagged = op.flag ? __hip_atomic_load(op.flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
  bool inexact = false, odd = false;
  uint32_t change[NW] = {};
  T xs[4][C];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const bool live = finite && v < op.nvec && p0 + j < op.len;
    const T *x = op.X + (live ? (int64_t)v * op.sv + (int64_t)(p0 + j) * op.sp : 0);
#pragma unroll
    for (int r = 0; r < C; ++r) xs[j][r] = live ? x[r * op.comp_stride] : T(0);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    __builtin_amdgcn_sched_barrier(0);  // one element after another: their words together take too many registers
    uint32_t W[12];  // then in signed bytes with the sum W: W + 0x80..80, each byte less 128
    element_words<T, C, NW>(xs[j], E, P, check, W, inexact, odd);
    if (check && kb == 0) add_word_changes<NW>(W, change);
    uint32_t carry = 0u;
#pragma unroll
    for (int i = 0; i < NW; ++i) W[i] = __builtin_addc(W[i], 0x80808080u, carry, &carry) ^ 0x80808080u;
#pragma unroll
    for (int i = NW; i < 12; ++i) W[i] = 0u;
#pragma unroll
    for (int i = 0; i < 2 * kQ; i += 4)
      *reinterpret_cast<i4v *>(&first_words[j][lane][i]) = i4v{(int)W[i], (int)W[i + 1], (int)W[i + 2], (int)W[i + 3]};
    if constexpr (kMore)
      *reinterpret_cast<i4v *>(&more_words[j][lane][0]) = i4v{(int)W[8], (int)W[9], (int)W[10], (int)W[11]};
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // other lanes' words are read from here on

  if (p0 == 0 && v < op.nvec && part == 0) op.exps[v] = E;
  if (check) {  // before the products: its words per element need not be kept through them
    auto fall_back = [&]() {
      *op.flag = 1;
      if (op.any) *op.any = 1;
    };
    if (kb == 0)
      for (int i = t; i < kBlk8 * NW; i += kThreads) lds.seen[i / NW][i % NW] = 0u;
    if (t < kBlk8) lds.rounded[t] = 0;
    __syncthreads();
    if (odd) fall_back();
    if (inexact) lds.rounded[l & 31] = 1;
    if (kb == 0) {
#pragma unroll
      for (int i = 0; i < NW; ++i) atomicOr(&lds.seen[l & 31][i], change[i]);
    }
    __syncthreads();
    if (t < kBlk8) {
      const int vt = (int)(vb * kBlk8) + t;
      if (vt < op.nvec) {
        int add = lds.rounded[t] ? kRounded : 0;
        if (kb == 0 && !last_grid_covered(lds.seen[t], op.bits, op.slice_bits, op.passes)) add |= kUnsettled;
        if (add & ~*(volatile int *)&op.state[vt]) {
          const int now = atomicOr(&op.state[vt], add) | add;
          if ((now & (kRounded | kUnsettled | kSettled)) == (kRounded | kUnsettled)) fall_back();
        }
      }
    }
  }

  // a product known to go by slices needs no planes (a late look would do)
  if (__builtin_amdgcn_readfirstlane(flagged) != 0) return;
  const int64_t plane = op.nbp * op.kbp * 1024;
  int8_t *dst = op.planes + (vb * op.kbp + kb) * 1024 + 4 * t;
  auto product = [&](int rb, int j, bool y) {  // 32 bases of row block rb, 32 elements j
    i16v acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0;
    const int col = lane % 32 + (y ? 32 : 0), half = lane / 32;
    if constexpr (kSmall) {
      const int64_t a = *reinterpret_cast<const int64_t *>(kRows.k16[0][rb][lane]);
      acc = __builtin_amdgcn_mfma_i32_32x32x16_i8(
          a, *reinterpret_cast<const int64_t *>(&first_words[j][col][2 * half]), acc, 0, 0, 0);
    } else {
      const i4v a = *reinterpret_cast<const i4v *>(kRows.k32[rb][lane]);
      acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(
          a, *reinterpret_cast<const i4v *>(&first_words[j][col][(2 * kQ - 4) * half]), acc, 0, 0, 0);
    }
    if constexpr (kMore) {
      const int64_t a = *reinterpret_cast<const int64_t *>(kRows.k16[1][rb][lane]);
      acc = __builtin_amdgcn_mfma_i32_32x32x16_i8(
          a, *reinterpret_cast<const int64_t *>(&more_words[j][col][2 * half]), acc, 0, 0, 0);
    }
    return acc;
  };
  auto insert = [](uint32_t word, uint32_t byte, int j) -> uint32_t {
    return j == 0 ? byte : __builtin_amdgcn_perm(byte, word, j == 1 ? 0x03020400u : j == 2 ? 0x03040100u : 0x04020100u);
  };
  // Row blocks of 32 bases: the (first) digits of blocks 0 and 1, then the second
  // digits of those with squared bases.  The halves of the two products of an
  // element number j (elements of lanes 0 .. 31 and 32 .. 63) are swapped, so that a
  // register holds one base for all 64 lanes and the constants are scalar.
  const int second = (op.nsq + 31) / 32;
  for (int pass = part; pass < 2 + second; pass += parts) {
    const bool digit2 = pass >= 2;
    const int rb = digit2 ? pass - 2 : pass, end = digit2 && u_end > op.nsq ? op.nsq : u_end;
    if (32 * rb >= end || 32 * rb + 32 <= u_first) continue;
    auto quotient = [&](int x, int u) { return __float_as_int(__builtin_fmaf((float)x, kBase.inv[32 * rb + u], 12582912.0f)); };
    uint32_t word[32] = {};  // bases 32 rb + u, bytes j
    auto swap = [](i16v &x, i16v &y) {  // register r of x: base 8 (r / 4) + r % 4, of y: four more
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const auto sw = __builtin_amdgcn_permlane32_swap((unsigned)x[r], (unsigned)y[r], false, false);
        x[r] = (int)sw[0];
        y[r] = (int)sw[1];
      }
    };
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      i16v x = product(rb, j, false), y = product(rb, j, true);
      if (digit2) {  // c-sum + s h-sum, without its digit 0
        i16v hx = product(rb + 2, j, false), hy = product(rb + 2, j, true);
        swap(x, y);
        swap(hx, hy);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int u = 8 * (r / 4) + r % 4;
          int q = quotient(x[r], u) - 0x4B400000;
          if (r == 0 && rb == 0) q = (x[0] + 128) >> 8;  // base 256: the byte 0x80 stands for -128
          x[r] = q + hx[r];
          y[r] = quotient(y[r], u + 4) - 0x4B400000 + hy[r];
        }
      } else {
        swap(x, y);
      }
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        if (a > 0 && 32 * rb + 8 * a >= end) break;  // no bases from here on
#pragma unroll
        for (int r = 4 * a; r < 4 * a + 4; ++r) {
          const int u = 8 * a + r % 4;
          word[u] = insert(word[u], (uint32_t)(__mul24(quotient(x[r], u), kBase.ns[32 * rb + u]) + x[r]), j);
          word[u + 4] = insert(word[u + 4], (uint32_t)(__mul24(quotient(y[r], u + 4), kBase.ns[32 * rb + u + 4]) + y[r]), j);
          asm volatile("" : "+v"(word[u]), "+v"(word[u + 4]));
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    int8_t *to = dst + (int64_t)(32 * rb - u_first + (digit2 ? u_end - u_first : 0)) * plane;
#pragma unroll
    for (int u = 0; u < 32; ++u) {
      if (32 * rb + u >= u_first && 32 * rb + u < end) *reinterpret_cast<uint32_t *>(to) = word[u];
      to += plane;
    }
  }
}

__device__ __forceinline__ int find_range(const int *prefix, int n, int b) {
  int lo = 0, hi = n - 1;  // the last i with prefix[i] <= b
  while (lo < hi) {
    const int mid = (lo + hi + 1) / 2;
    if (prefix[mid] <= b)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

// Workgroup (x, y): block x - prefix[i] of operand i, every gridDim.y-th row
// block of the bases [u_first, u_end) (u_end < 0: every base of the operand).
template <typename T, int C, int NW>
__global__ __launch_bounds__(kThreads, NW > 8 ? 3 : 4) void k_residue_split(const ResidueOperand<T> *__restrict__ ops,
                                                            const int *__restrict__ prefix, int nops, int live_only,
                                                            int u_first, int u_end) {
  const int i = __builtin_amdgcn_readfirstlane(find_range(prefix, nops, blockIdx.x));
  const ResidueOperand<T> op = ops[i];
  const int64_t blk = (int64_t)blockIdx.x - prefix[i];
  const int end = u_end < 0 ? op.nunits : u_end, part = blockIdx.y, parts = gridDim.y;
  const bool check = op.float_form != 0 && u_first == 0 && blockIdx.y == 0;
  __shared__ SplitLds<NW> lds;
  if (live_only && op.orient == 0) {  // A's blocks past those with elements: padding of k
    const int64_t nb = ceil_div((int64_t)op.nvec, (int64_t)kBlk8), kb = blk / nb;
    if (kb * kKBlk8 >= op.len) {
      if (op.padded && *op.padded == 0) return;
      int8_t *to = op.planes + (blk % nb * op.kbp + kb) * 1024 + 4 * threadIdx.x;
      for (int u = 0; u < end + op.nsq; ++u) *reinterpret_cast<uint32_t *>(to + u * (op.nbp * op.kbp * 1024)) = 0u;
      return;
    }
  }
  if (op.orient == 0)
    residue_block<T, C, NW, 0>(op, blk, live_only != 0, u_first, end, part, parts, check, lds);
  else
    residue_block<T, C, NW, 1>(op, blk, live_only != 0, u_first, end, part, parts, check, lds);
}

// ---------------------------------------------------------------------------
// GEMM.
// ---------------------------------------------------------------------------
// Work of one tile: bases u0 .. u1 - 1 of the plan.  Operand planes are those of
// a group of bases, result planes the plan's in this k chunk.
// Products are at most 2^14 in magnitude: 32768 k of them twice (the two pairs of
// a square's second diagonal) and a carry stay below 2^31, so longer k is cut into
// chunks with result planes of their own, which k_residue_fold adds up.
struct ResidueWork {
  int u0, u1, u_first, count, nsq, nunits;  // bases [u_first, u_first + count) of nunits have operand planes
  int8_t *R;
  int64_t plane, mbp;
  __device__ int pairs() const { return residue_pairs_below(u1, nsq) - residue_pairs_below(u0, nsq); }
  __device__ void first(PairCursor &c) const { c = {u0, 1, 1}; }
  __device__ void next(PairCursor &c) const {
    if (++c.s > c.g) {
      c.s = 1;
      if (++c.g > (c.u < nsq ? 2 : 1)) {
        c.g = 1;
        ++c.u;
      }
    }
  }
  __device__ int a_plane(const PairCursor &c) const { return c.u - u_first + (c.s - 1) * count; }
  __device__ int b_plane(const PairCursor &c) const { return c.u - u_first + (c.g - c.s) * count; }
  __device__ bool diagonal_ends(const PairCursor &c) const { return c.s == c.g; }
  template <int BI, int BJ>
  __device__ __forceinline__ void finish(const PairCursor &c, i16v (&acc)[BJ][BI], int64_t bi0, int64_t bj0,
                                         int lane) const {
    const BaseInfo b = kBase.info[c.u];
    int8_t *out = R + (int64_t)(c.u + (c.g - 1) * nunits) * plane;
#pragma unroll
    for (int y = 0; y < BJ; ++y)
#pragma unroll
      for (int x = 0; x < BI; ++x) {
        i4v o;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          uint32_t t[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) t[r] = residue_byte(fold16(acc[y][x][4 * v + r], b), b);
          o[v] = (int)pack4(t[0], t[1], t[2], t[3]);
          __builtin_amdgcn_sched_barrier(0);  // a few entries at a time: the accumulators leave few registers
        }
        *reinterpret_cast<i4v *>(out + (((bj0 + y) * mbp + bi0 + x) * 64 + lane) * 16) = o;
      }
    if (c.u < nsq && c.g == 1) {
#pragma unroll
      for (int y = 0; y < BJ; ++y)
#pragma unroll
        for (int x = 0; x < BI; ++x)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            int v = acc[y][x][r];
            asm volatile("" : "+v"(v));  // the byte is formed again rather than kept from above
            acc[y][x][r] = divide_out(v, residue_byte(fold16(v, b), b), b);
            __builtin_amdgcn_sched_barrier(0);
          }
    } else {
#pragma unroll
      for (int y = 0; y < BJ; ++y)
#pragma unroll
        for (int x = 0; x < BI; ++x)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[y][x][r] = 0;
    }
  }
};

template <int CFG>
__global__ __launch_bounds__(64 * Int8Cfg<CFG>::WM * Int8Cfg<CFG>::WN, 1) void k_gemm_residue(
    const int8_t *__restrict__ A, const int8_t *__restrict__ B, int64_t mbp, int64_t nbp, int64_t kbp, int u_first,
    int u_end, int nsq, int nplanes, int m, int n, int8_t *__restrict__ R, int64_t plane,
    const int *__restrict__ skip) {
  __shared__ __attribute__((aligned(16))) int8_t lds[Int8Cfg<CFG>::NS * int8_stage_bytes<CFG>()];
  const int quit = skip ? *skip : 0;
  constexpr int TB = Int8Cfg<CFG>::TB, KSB = Int8Cfg<CFG>::KSB;
  int tm, tn;
  int8_tile_coords(blockIdx.x, gridDim.x, (int)(mbp / TB), (int)(nbp / TB), tm, tn);
  const int u0 = residue_group_start(u_first, u_end, nsq, blockIdx.z, gridDim.z);
  const int u1 = residue_group_start(u_first, u_end, nsq, blockIdx.z + 1, gridDim.z);
  const int64_t kb0 = (int64_t)blockIdx.y * kChunkBlocks;
  const int64_t kb1 = kb0 + kChunkBlocks < kbp ? kb0 + kChunkBlocks : kbp;
  const int nks = (int)ceil_div(kb1 - kb0, KSB), last = (int)(kb1 - kb0) - (nks - 1) * KSB;
  const ResidueWork work{u0, u1, u_first, u_end - u_first, nsq, nplanes - nsq, R + (int64_t)blockIdx.y * nplanes * plane, plane, mbp};
  gemm_int8_tile<CFG>(work, A, B, mbp, nbp, kbp, kb0, nks, last, m, n, tm, tn, quit, lds);
}

// Persistent GEMM of a batch in tile configuration CFG: each workgroup takes
// (product, tile, k chunk, unit group) items from its XCD's list, then helps the
// other lists; lists are ordered by decreasing work.
template <int CFG>
__global__ __launch_bounds__(64 * Int8Cfg<CFG>::WM * Int8Cfg<CFG>::WN, 1) void k_gemm_residue_batched(
    const ResidueDesc *__restrict__ descs, const int4 *__restrict__ items, const int *__restrict__ bounds,
    int *__restrict__ counters) {
  __shared__ __attribute__((aligned(16))) int8_t lds[Int8Cfg<CFG>::NS * int8_stage_bytes<CFG>()];
  __shared__ int next;
  constexpr int TB = Int8Cfg<CFG>::TB, KSB = Int8Cfg<CFG>::KSB;
  for (;;) {
    if (threadIdx.x == 0) next = take_item(counters, bounds, blockIdx.x);
    __syncthreads();
    const int it = __builtin_amdgcn_readfirstlane(next);
    __syncthreads();
    if (it < 0) break;
    const int4 w = items[it];
    const ResidueDesc &d = descs[w.x];
    if (d.skip && *d.skip) continue;
    const int tiles_m = (int)(d.mbp / TB);
    const int tm = w.y % tiles_m, tn = w.y / tiles_m;
    const int64_t kb0 = (int64_t)w.z * kChunkBlocks;
    const int64_t kb1 = kb0 + kChunkBlocks < d.kbp ? kb0 + kChunkBlocks : d.kbp;
    const int nks = (int)ceil_div(kb1 - kb0, KSB), last = (int)(kb1 - kb0) - (nks - 1) * KSB;
    const ResidueWork work{residue_group_start(0, d.nunits, d.nsq, w.w, d.groups),
                           residue_group_start(0, d.nunits, d.nsq, w.w + 1, d.groups),
                           0,
                           d.nunits,
                           d.nsq,
                           d.nunits,
                           d.R + (int64_t)w.z * d.nplanes * d.plane,
                           d.plane,
                           d.mbp};
    gemm_int8_tile<CFG>(work, d.A, d.B, d.mbp, d.nbp, d.kbp, kb0, nks, last, d.m, d.n, tm, tn, 0, lds);
  }
}

// ---------------------------------------------------------------------------
// Combine.
// ---------------------------------------------------------------------------
typedef const __attribute__((address_space(4))) uint32_t *const_words;  // scalar loads

// 32-plane steps of the combine's matrix products.  The plan's moduli fill nwc
// words with at most so many planes (32 planes hold 242 bits, 64 hold 460).
__host__ __device__ constexpr int combine_steps(int nwc) { return nwc <= 8 ? 1 : nwc <= 15 ? 2 : 3; }
// 32-digit row blocks of nwc words.
__host__ __device__ constexpr int combine_rows(int nwc) { return (nwc + 7) / 8; }
// Words of the planes' weights: 4 nwc digits, a byte per plane of the steps.
__host__ __device__ constexpr int weight_words(int nwc) { return 4 * nwc * combine_steps(nwc) * 8; }

// w up by SH words, and its place down, if its top SH words are zero.
template <int NWC, int SH>
__device__ __forceinline__ void raise_words(uint32_t (&w)[NWC], int &place) {
  if constexpr (SH < NWC) {
    uint32_t any = 0u;
#pragma unroll
    for (int i = NWC - SH; i < NWC; ++i) any |= w[i];
    const bool up = any == 0u;
#pragma unroll
    for (int i = NWC - 1; i >= 0; --i) w[i] = up ? (i >= SH ? w[i >= SH ? i - SH : 0] : 0u) : w[i];
    place -= up ? 32 * SH : 0;
  }
}

// The components of X 2^e0, X = V mod M (balanced), from V's base-256 digit sums.
template <int NWC, typename T, int C>
__device__ __forceinline__ void combine_entry(const int (&S)[4 * NWC], const_words mod, double inv_m, int e0,
                                              T (&out)[C]) {
  int t0[NWC], t1[NWC];  // V = sum (t0 + t1 2^16) 2^(32 i)
#pragma unroll
  for (int i = 0; i < NWC; ++i) {
    t0[i] = S[4 * i] + (S[4 * i + 1] << 8);
    t1[i] = S[4 * i + 2] + (S[4 * i + 3] << 8);
  }
  // X = V - q M, q = rint(V / M) from the top three words: |X| < 0.48 M, and
  // what lies below them is less than 2^-26 M
  constexpr int kTop = NWC < 3 ? NWC : 3;
  double v = 0.0;
#pragma unroll
  for (int i = NWC - 1; i >= NWC - kTop; --i)
    v = __builtin_fma(__builtin_fma(v, 65536.0, (double)t1[i]), 65536.0, (double)t0[i]);
  const int nq = -(int)rint(v * inv_m);
  uint32_t w[NWC];
  int64_t c = 0;
#pragma unroll
  for (int i = 0; i < NWC; ++i) {
    c += (int64_t)nq * (int64_t)(int32_t)mod[i] + (int64_t)t0[i] + ((int64_t)t1[i] << 16);
    w[i] = (uint32_t)c;
    c >>= 32;
  }
  // magnitude and sign
  const uint32_t neg = (uint32_t)((int32_t)w[NWC - 1] >> 31);
  uint32_t up = neg & 1u;
#pragma unroll
  for (int i = 0; i < NWC; ++i) {
    const uint64_t s = (uint64_t)(w[i] ^ neg) + up;
    w[i] = (uint32_t)s;
    up = (uint32_t)(s >> 32);
  }
  // the leading nonzero word to the top: for the whole wavefront while it can
  // (its entries have much the same magnitude), then entry by entry
  int ex = 32 * NWC;
#pragma unroll 1
  for (int r = 0; r < NWC - 1 && __all(w[NWC - 1] == 0u); ++r) {
#pragma unroll
    for (int i = NWC - 1; i > 0; --i) w[i] = w[i - 1];
    w[0] = 0u;
    ex -= 32;
  }
  if (__any(w[NWC - 1] == 0u)) {
    raise_words<NWC, 16>(w, ex);
    raise_words<NWC, 8>(w, ex);
    raise_words<NWC, 4>(w, ex);
    raise_words<NWC, 2>(w, ex);
    raise_words<NWC, 1>(w, ex);
  }
  // the leading bit to the top: words s[0], s[1], ... of (w << lz), one shift
  // right by 1 and by 31 - lz so that both fit the instruction
  constexpr int K = sizeof(T) == 4 ? 2 : C + 1;  // 53-bit digits of the magnitude
  constexpr int kW = (53 * K + 31) / 32;
  const int lz = __clz((int)w[NWC - 1]);
  ex -= lz;
  uint32_t s[kW + 1];
#pragma unroll
  for (int i = 0; i <= kW; ++i) {
    auto word = [&](int j) -> uint32_t { return j >= 0 && j < NWC ? w[NWC - 1 - j] : 0u; };  // from the top
    const uint32_t hi = __builtin_amdgcn_alignbit(word(i - 1), word(i), 1), lo = __builtin_amdgcn_alignbit(word(i), word(i + 1), 1);
    s[i] = __builtin_amdgcn_alignbit(hi, lo, 31 - lz);
  }
  // 53-bit digits y_j, balanced: |y_j| <= 2^52 for j > 0, so y_0 is X rounded to
  // nearest and the rest follows it within half its last place
  double z[K];
#pragma unroll
  for (int j = 0; j < K; ++j) {
    auto bits = [&](int p) -> uint32_t {  // 32 bits from place p
      return p % 32 == 0 ? s[p / 32] : __builtin_amdgcn_alignbit(s[p / 32], s[p / 32 + 1 <= kW ? p / 32 + 1 : kW], 32 - p % 32);
    };
    z[j] = __builtin_fma((double)(bits(53 * j) >> 11), 4294967296.0, (double)bits(53 * j + 21));
  }
#pragma unroll
  for (int j = K - 1; j > 0; --j) {
    const bool half = z[j] >= 4503599627370496.0;
    z[j] -= half ? 9007199254740992.0 : 0.0;
    z[j - 1] += half ? 1.0 : 0.0;
  }
  const double sign = neg ? -1.0 : 1.0;
#pragma unroll
  for (int j = 0; j < K; ++j) z[j] *= sign * __builtin_ldexp(1.0, -53 * j);
  const int e = ex - 53 + e0;
  if constexpr (sizeof(T) == 8) {
    out[0] = ldexp(z[0], e);
    double rest = z[1];
#pragma unroll
    for (int r = 1; r < C; ++r) {
      double err;
      out[r] = ldexp(two_sum(rest, z[r + 1], err), e);
      rest = err;
    }
  } else {
    // nearest binary32 of the rest, three times
    double rest = z[0], low = z[1];
#pragma unroll
    for (int r = 0; r < C; ++r) {
      const float f = (float)rest;
      out[r] = ldexpf(f, e);
      double err;
      rest = two_sum(rest - (double)f, low, err);
      low = err;
    }
  }
}

// Products of several k chunks: the chunks' digits added into the first chunk's
// planes.  Workgroup: one 32 x 32 block of C.
__global__ __launch_bounds__(kThreads) void k_residue_fold(const ResidueDesc *__restrict__ descs,
                                                           const int *__restrict__ prefix, int nprod) {
  const int p = __builtin_amdgcn_readfirstlane(find_range(prefix, nprod, blockIdx.x));
  const ResidueDesc d = descs[p];
  if (d.nchunks <= 1 || (d.skip && *d.skip)) return;
  int8_t *at = d.R + ((int64_t)blockIdx.x - prefix[p]) * 1024 + 4 * threadIdx.x;
  for (int u = 0; u < d.nunits; ++u) {
    const BaseInfo b = kBase.info[u];
    const int digits = u < d.nsq ? 2 : 1;
    int sum[4] = {0, 0, 0, 0};
    for (int g = 0; g < digits; ++g) {
      int8_t *pl = at + (int64_t)(u + g * d.nunits) * d.plane;
      for (int ch = 0; ch < d.nchunks; ++ch) {
        const uint32_t x = *reinterpret_cast<const uint32_t *>(pl + (int64_t)ch * d.nplanes * d.plane);
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[e] += (int)(int8_t)(x >> (8 * e));
      }
      uint32_t t[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        t[e] = residue_byte(sum[e], b);
        sum[e] = divide_out(sum[e], t[e], b);
      }
      *reinterpret_cast<uint32_t *>(pl) = pack4(t[0], t[1], t[2], t[3]);
    }
  }
}

// Bound by the planes' bytes and C's (3.4 TB/s for DD) and, from 9 words on, by
// the vector instructions of combine_entry.  With v_dot4 sums instead of the
// matrix products and a renormalization of 48-bit chunks instead of the digits:
// DD n = 4096 (32 planes) 506 -> 234 us, QD (68 planes) 1458 -> 608 us; and C is
// now X rounded to nearest, where the renormalization left up to 0.57 units.
//
// Workgroup: one 32 x 32 block of C, wavefront q its quad q: entries 4 q .. 4 q + 3
// of every lane of the planes' layout (int8.hip).  Two half blocks (the lanes
// below and from 32 on) of 4 entries per lane, each as two matrix products
// digits x planes x 32 entries on the INT8 matrix cores: lane l of the
// instruction holds entry l % 32's bytes of 16 planes, its results the 16 digit
// rows 8 (r / 4) + 4 (l / 32) + r % 4.  Swapping the halves of two products
// (v_permlane32_swap) leaves every lane all digits of one entry.
template <typename T, int C, int NWC>
__global__ __launch_bounds__(kThreads, 2) void k_residue_combine(const ResidueDesc *__restrict__ descs,
                                                              const int *__restrict__ prefix, int nprod) {
  constexpr int RB = combine_rows(NWC), KS = combine_steps(NWC);
  const int p = __builtin_amdgcn_readfirstlane(find_range(prefix, nprod, blockIdx.x));
  const ResidueDesc d = descs[p];
  if (d.skip && *d.skip) return;
  const int64_t blk = (int64_t)blockIdx.x - prefix[p];
  const int lane = threadIdx.x % 64, quad = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
  const int64_t bi = blk % d.mbp, bj = blk / d.mbp;
  if (bi * 32 >= d.m || bj * 32 + 8 * quad >= d.n) return;
  const int i = (int)(bi * 32) + lane % 32;
  const int Ei = i < d.m ? d.EA[i] : kZeroExp;

  // weights: digits of the planes
  i4v wt[RB][KS];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int row = 32 * rb + lane % 32;  // results of rows past the last digit are not looked at
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      wt[rb][ks] = reinterpret_cast<const i4v *>(d.table)[((row < 4 * NWC ? row : 4 * NWC - 1) * KS + ks) * 2 + lane / 32];
  }
  const const_words mod = (const_words)d.table + weight_words(NWC);
  const double inv_m = __longlong_as_double((long long)((uint64_t)mod[NWC] | ((uint64_t)mod[NWC + 1] << 32)));

#pragma unroll 1
  for (int h = blockIdx.y; h < 2; h += gridDim.y) {
    if (bj * 32 + 8 * quad + 4 * h >= d.n) return;
    const int8_t *src = d.R + blk * 1024 + (h * 32 + lane % 32) * 16 + 4 * quad;
    i4v f[KS][4];  // entry e: its bytes in this lane's 16 planes of a step
    int upper = lane / 32;
    int64_t plane = d.plane;
    asm volatile("" : "+v"(upper), "+s"(plane));  // the planes' offsets are formed here, not kept in registers
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      uint32_t x[16];  // planes past the last have zero weights
#pragma unroll
      for (int v = 0; v < 4; ++v) {
#pragma unroll
        for (int t = 4 * v; t < 4 * v + 4; ++t) x[t] = 0u;
        if (ks > 0 && 32 * ks + 4 * v >= d.nplanes) continue;
#pragma unroll
        for (int t = 4 * v; t < 4 * v + 4; ++t) {
          const int lo = 32 * ks + t < d.nplanes ? 32 * ks + t : d.nplanes - 1;
          const int hi = 32 * ks + 16 + t < d.nplanes ? 32 * ks + 16 + t : d.nplanes - 1;
          x[t] = *reinterpret_cast<const uint32_t *>(src + (upper ? hi * plane : lo * plane));
          __builtin_amdgcn_sched_barrier(0);  // one address at a time
        }
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const uint32_t l0 = __builtin_amdgcn_perm(x[4 * v + 1], x[4 * v], 0x05010400u);
        const uint32_t h0 = __builtin_amdgcn_perm(x[4 * v + 3], x[4 * v + 2], 0x05010400u);
        const uint32_t l1 = __builtin_amdgcn_perm(x[4 * v + 1], x[4 * v], 0x07030602u);
        const uint32_t h1 = __builtin_amdgcn_perm(x[4 * v + 3], x[4 * v + 2], 0x07030602u);
        f[ks][0][v] = (int)__builtin_amdgcn_perm(h0, l0, 0x05040100u);
        f[ks][1][v] = (int)__builtin_amdgcn_perm(h0, l0, 0x07060302u);
        f[ks][2][v] = (int)__builtin_amdgcn_perm(h1, l1, 0x05040100u);
        f[ks][3][v] = (int)__builtin_amdgcn_perm(h1, l1, 0x07060302u);
      }
    }
#pragma unroll
    for (int e = 0; e < 4; e += 2) {
      i16v acc[2][RB];
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[x][rb][r] = 0;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int x = 0; x < 2; ++x)
            acc[x][rb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wt[rb][ks], f[ks][e + x], acc[x][rb], 0, 0, 0);
      int S[4 * NWC];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const auto sw = __builtin_amdgcn_permlane32_swap((unsigned)acc[0][rb][r], (unsigned)acc[1][rb][r], false, false);
          const int y = 32 * rb + 8 * (r / 4) + r % 4;
          if (y < 4 * NWC) S[y < 4 * NWC ? y : 0] = (int)sw[0];
          if (y + 4 < 4 * NWC) S[y + 4 < 4 * NWC ? y + 4 : 0] = (int)sw[1];
        }
      const int j = (int)(bj * 32) + 8 * quad + 4 * h + e + lane / 32;
      const bool inside = i < d.m && j < d.n;
      const int Fj = inside ? d.EB[j] : kZeroExp;
      T out[C];
      combine_entry<NWC, T, C>(S, mod, inv_m, Ei + Fj - 2 * d.bits, out);
      if (Ei == kZeroExp || Fj == kZeroExp) {
#pragma unroll
        for (int r = 0; r < C; ++r) out[r] = T(0);
      }
      if (Ei == kNonFinite || Fj == kNonFinite) {
#pragma unroll
        for (int r = 0; r < C; ++r) out[r] = (T)__builtin_nan("");
      }
      if (inside) {
        T *dst = static_cast<T *>(d.C) + i + (int64_t)j * d.ldc;
#pragma unroll
        for (int r = 0; r < C; ++r) dst[r * d.c_stride] = out[r];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Host data on its way to the device inside kernel arguments: no copy, so the
// sequence can be captured and keeps no host buffer.  Also clears two regions.
// ---------------------------------------------------------------------------
constexpr int kUploadWords = 976;
struct Upload {
  uint32_t w[kUploadWords];
};
__global__ __launch_bounds__(kThreads) void k_upload(Upload data, int n, uint32_t *dst, uint32_t *z0, int64_t n0,
                                                     uint32_t *z1, int64_t n1) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = t; i < n; i += step) dst[i] = data.w[i];
  for (int64_t i = t; i < n0; i += step) z0[i] = 0u;
  for (int64_t i = t; i < n1; i += step) z1[i] = 0u;
}

// Maxima of the vectors and the (last) upload in one launch, for vectors short
// enough that a workgroup reads 16 whole ones: no atomics, so nothing to clear for
// them first, and no shuffles (64 bit ones took most of k_split_max0's 8.5 us on
// two tiles).  Bound by the latency of its loads, 16 in flight per thread.
//
// In the FLOAT form strips with zeros among a vector's first 32 elements take their
// samples here (settle_strip).  For all strips, with the split's own look at the first
// elements left out, that took DD 64^3 from 30.4 to 31.5 us and TD 200 x 150 x 333 from
// 50.4 to 51.3.  Other strips do nothing for it: with the samples' room cleared and the
// vote counted by every launch, TS 55 x 1218 x 278 took 4.5 - 4.8 us, not 3.8 - 3.9.
template <typename T>
struct MaxOperand {
  const T *X;
  int64_t comp_stride, sv, sp;
  int nvec, len, orient;
  typename bits_of<T>::type *mu;
  int *state;
};
struct GridOfSlices {
  int bits, slice_bits, passes;
};
template <typename T, int C>  // C = 0: INT8 form, no samples
__global__ __launch_bounds__(kThreads) void k_residue_begin(Upload data, int n, int strips_a, uint32_t *dst,
                                                            MaxOperand<T> a, MaxOperand<T> b, GridOfSlices grid,
                                                            int *flag) {
  using U = typename bits_of<T>::type;
  const int t = threadIdx.x;
  const int64_t id = blockIdx.x * (int64_t)kThreads + t, step = (int64_t)gridDim.x * kThreads;
  const bool second = (int)blockIdx.x >= strips_a;
  const MaxOperand<T> op = second ? b : a;
  const int v0 = 16 * ((int)blockIdx.x - (second ? strips_a : 0));
  const int dv = op.orient == 0 ? t % 16 : t / 16, dp = op.orient == 0 ? t / 16 : t % 16;
  const int v = v0 + dv < op.nvec ? v0 + dv : op.nvec - 1;
  const T *x = op.X + (int64_t)v * op.sv;
  U best = 0;
  bool zeros = false;  // among the first 32 elements
  for (int p0 = dp; p0 < op.len; p0 += kThreads) {
    T e[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {  // past the end the last element again
      const int p = p0 + 16 * i < op.len ? p0 + 16 * i : op.len - 1;
      e[i] = x[(int64_t)p * op.sp];
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const U k = abs_bits(e[i]);
      best = k > best ? k : best;
    }
    if (C > 0 && p0 == dp) zeros = abs_bits(e[0]) == 0 || abs_bits(e[1]) == 0;
  }
  for (int64_t i = id; i < n; i += step) dst[i] = data.w[i];
  if (id == 0 && flag) *flag = 0;
  __shared__ U red[16][17];
  __shared__ int some[kThreads / 64];
  red[dp][dv] = best;
  if constexpr (C > 0) some[t / 64] = __any(zeros);
  __syncthreads();
  if (t < 16 && v0 + t < op.nvec) {
    U k = red[0][t];
#pragma unroll
    for (int i = 1; i < 16; ++i) k = red[i][t] > k ? red[i][t] : k;
    op.mu[v0 + t] = k;
  }
  if constexpr (C > 0) {
    if ((some[0] | some[1] | some[2] | some[3]) != 0) {
      __shared__ uint32_t changes[16][kChangeWords];
      U k = red[0][dv];
      for (int i = 1; i < 16; ++i) k = red[i][dv] > k ? red[i][dv] : k;
      const int s = settle_strip<T, C>(x, op.comp_stride, op.sp, op.len, dp, dv, vector_exponent<T>(k, 1), grid.bits,
                                       grid.slice_bits, grid.passes, changes);
      if (dp == 0 && v0 + dv < op.nvec) op.state[v0 + dv] = s;
    } else if (t < 16 && v0 + t < op.nvec) {
      op.state[v0 + t] = 0;
    }
  }
}

// The same for vectors whose maxima are known: workgroup x - prefix[i] of operand i.
// The states are cleared.
template <typename T, int C>
__global__ __launch_bounds__(kThreads) void k_residue_sample(const ResidueOperand<T> *__restrict__ ops,
                                                             const int *__restrict__ prefix, int nops) {
  using U = typename bits_of<T>::type;
  const int i = __builtin_amdgcn_readfirstlane(find_range(prefix, nops, blockIdx.x));
  const ResidueOperand<T> &op = ops[i];
  const int t = threadIdx.x, v0 = 16 * ((int)blockIdx.x - prefix[i]);
  const int dv = op.orient == 0 ? t % 16 : t / 16, dp = op.orient == 0 ? t / 16 : t % 16;
  const int v = v0 + dv < op.nvec ? v0 + dv : op.nvec - 1;
  const T *x = op.X + (int64_t)v * op.sv;
  __shared__ uint32_t changes[16][kChangeWords];
  bool zeros = false;
#pragma unroll
  for (int j = 0; j < 32; j += 16) zeros = zeros || dp + j >= op.len || abs_bits(x[(int64_t)(dp + j) * op.sp]) == 0;
  if (!__syncthreads_or(zeros)) return;
  const int s = settle_strip<T, C>(x, op.comp_stride, op.sp, op.len, dp, dv,
                                   vector_exponent<T>(static_cast<const U *>(op.mu)[v], 1), op.bits, op.slice_bits,
                                   op.passes, changes);
  if (dp == 0 && v0 + dv < op.nvec) op.state[v0 + dv] = s;
}
// Up to this length (one or two launches less): INT8 DD calls of 64^2 x 64 go from
// 58 to 49 us, 64^2 x 8192 from 127 to 114, n = 4096 from 2629 to 2584; a single pair
// of vectors of 100000 would take 989 us against 671 with the tiled maxima.
constexpr int kBeginLength = 8192;

// Big integers of 32-bit words, for the tables.
using Big = std::vector<uint32_t>;
void big_mul(Big &x, uint32_t f) {
  uint64_t c = 0;
  for (auto &w : x) {
    c += (uint64_t)w * f;
    w = (uint32_t)c;
    c >>= 32;
  }
  if (c) x.push_back((uint32_t)c);
}
uint32_t big_div(Big &x, uint32_t f) {  // x /= f, returns the remainder
  uint64_t r = 0;
  for (size_t i = x.size(); i-- > 0;) {
    r = (r << 32) | x[i];
    x[i] = (uint32_t)(r / f);
    r %= f;
  }
  return (uint32_t)r;
}
double big_value(const Big &x) {
  double v = 0.0;
  for (size_t i = x.size(); i-- > 0;) v = v * 4294967296.0 + (double)x[i];
  return v;
}

// Bits of the first n bases, for the plans: they are looked for on every call.
struct BaseBits {
  double sum[kNumBases + 1];
  BaseBits() {
    sum[0] = 0.0;
    for (int u = 0; u < kNumBases; ++u) sum[u + 1] = sum[u] + std::log2((double)kHostBases.s[u]);
  }
};
double log2_modulus(int nunits, int nsq) {
  static const BaseBits bits;
  return bits.sum[nunits] + bits.sum[nsq];
}

}  // namespace

bool residue_plan(int bits, int64_t k, ResiduePlan &p) {
  if (bits < 1 || bits > kMaxResidueBits || k < 1) return false;
  const double need = 2.0 * bits + std::log2((double)k) + 1.07;  // M > 2.1 k 2^(2 bits)
  p.bits = bits;
  p.nunits = 0;
  for (int n = 1; n <= kNumBases; ++n) {
    int sq = 0;
    while (log2_modulus(n, sq) < need && sq < n) ++sq;
    if (log2_modulus(n, sq) < need) continue;
    if (p.nunits == 0 || n + 2 * sq <= p.products()) {  // of equal ones that with fewer squares
      p.nunits = n;
      p.nsq = sq;
    }
  }
  if (p.nunits == 0) return false;
  p.nplanes = p.nunits + p.nsq;
  p.nw = (bits + 2 + 31) / 32;
  p.nchunks = (int)ceil_div(kblocks8_padded(k), (int64_t)kChunkBlocks);
  // |V| <= 64 nplanes M, a sign, and a bit for the logarithms' rounding
  const double top = log2_modulus(p.nunits, p.nsq) + 8.0 + std::log2((double)p.nplanes);
  p.nwc = std::max(2, (int)std::ceil(top / 32.0));
  return p.nwc <= kMaxCombineWords && p.nplanes <= 32 * combine_steps(p.nwc);
}

const std::vector<uint32_t> &residue_table(int nunits, int nsq, int nwc) {
  static std::mutex mu;
  static std::map<std::tuple<int, int, int>, std::vector<uint32_t>> tables;
  std::lock_guard<std::mutex> lock(mu);
  std::vector<uint32_t> &t = tables[std::make_tuple(nunits, nsq, nwc)];
  if (!t.empty()) return t;
  Big M{1};
  for (int u = 0; u < nunits; ++u)
    for (int e = 0; e < (u < nsq ? 2 : 1); ++e) big_mul(M, (uint32_t)kHostBases.s[u]);
  M.resize(nwc, 0u);
  const int KS = combine_steps(nwc);
  t.assign((size_t)weight_words(nwc) + nwc + 2, 0u);
  for (int u = 0; u < nunits; ++u) {
    const uint32_t s = (uint32_t)kHostBases.s[u], mod = u < nsq ? s * s : s;
    Big Mu = M;
    big_div(Mu, mod);
    Big tmp = Mu;
    const uint32_t r = big_div(tmp, mod);
    uint32_t inv = 1;  // (M / mod)^-1 mod mod
    while ((uint64_t)inv * r % mod != 1) ++inv;
    for (int g = 0; g < (u < nsq ? 2 : 1); ++g) {
      Big w = Mu;
      big_mul(w, g == 0 ? inv : (uint32_t)((uint64_t)inv * s % mod));
      w.resize(nwc, 0u);
      // w - M where that is the smaller in magnitude, two's complement
      Big other(nwc);
      uint64_t borrow = 0;
      bool larger = false;  // 2 w > M
      for (int i = 0; i < nwc; ++i) {
        const uint64_t d = (uint64_t)w[i] - M[i] - borrow;
        other[i] = (uint32_t)d;
        borrow = (d >> 32) & 1;
      }
      for (int i = nwc - 1; i >= 0; --i) {  // compare w with M - w = -other
        uint64_t neg = (uint64_t)(~other[i]);
        bool low_zero = true;
        for (int j = 0; j < i; ++j) low_zero = low_zero && other[j] == 0;
        if (low_zero) ++neg;
        const uint32_t mw = (uint32_t)neg;
        if (w[i] != mw) {
          larger = w[i] > mw;
          break;
        }
      }
      if (larger) w = other;
      const int pl = u + g * nunits;
      int carry = 0;
      for (int j = 0; j < 4 * nwc; ++j) {
        int digit = (int)((w[j / 4] >> (8 * (j % 4))) & 255u) + carry;
        carry = digit >= 128 ? 1 : 0;
        if (carry) digit -= 256;
        t[(size_t)(j * KS * 8 + pl / 4)] |= (uint32_t)(uint8_t)(int8_t)digit << (8 * (pl % 4));
      }
    }
  }
  // M in balanced words, and 2^(32 (nwc - 3)) / M (the top three words over M)
  const size_t at = (size_t)weight_words(nwc);
  uint32_t up = 0;
  for (int i = 0; i < nwc; ++i) {
    const uint64_t w = (uint64_t)M[i] + up;
    t[at + i] = (uint32_t)w;
    up = w >= (uint64_t(1) << 31) ? 1 : 0;
  }
  const double inv_m = std::ldexp(1.0, 32 * std::max(0, nwc - 3)) / big_value(M);
  uint64_t bits;
  __builtin_memcpy(&bits, &inv_m, 8);
  t[at + nwc] = (uint32_t)bits;
  t[at + nwc + 1] = (uint32_t)(bits >> 32);
  return t;
}

namespace {

size_t up256(size_t x) { return (x + 255) & ~size_t(255); }

// The descriptors before the table, which is read 16 bytes at a time.
constexpr size_t kHeadBytes = (2 * sizeof(ResidueOperand<double>) + sizeof(ResidueDesc) + 6 * 4 + 15) / 16 * 16;
// The planes behind them begin at a multiple of their blocks' 1 KiB: blocks across two
// of these cost the QD combine 3 % (n = 4096).
constexpr size_t kBlockBytes = 1024;
size_t header_bytes(const ResiduePlan &p) {
  const size_t words = (size_t)weight_words(p.nwc) + p.nwc + 2;
  return up256(kHeadBytes + words * 4) + kBlockBytes - 256;
}
char *planes_of(char *arena, const ResiduePlan &p) {
  const uintptr_t end = reinterpret_cast<uintptr_t>(arena) + header_bytes(p);
  return reinterpret_cast<char *>(end / kBlockBytes * kBlockBytes);
}

struct Shape {
  int64_t mbp, nbp, kbp, a_plane, b_plane, r_plane;
};
Shape shape_of(int cfg, int64_t m, int64_t n, int64_t k) {
  const int tb = int8_tile_blocks(cfg);
  Shape s;
  s.mbp = nblocks8_padded(m, tb);
  s.nbp = nblocks8_padded(n, tb);
  s.kbp = kblocks8_padded(k);
  s.a_plane = s.mbp * s.kbp * 1024;
  s.b_plane = s.nbp * s.kbp * 1024;
  s.r_plane = s.mbp * s.nbp * 1024;
  return s;
}

template <typename T, int C>
hipError_t split_launch(int nw, dim3 grid, const ResidueOperand<T> *ops, const int *prefix, int nops, int live_only,
                        int u_first, int u_end, hipStream_t st) {
  switch (nw) {
#define MP_RESIDUE_SPLIT_CASE(NW)                                                                                  \
  case NW:                                                                                                         \
    hipLaunchKernelGGL((k_residue_split<T, C, NW>), grid, dim3(kThreads), 0, st, ops, prefix, nops, live_only, u_first, \
                       u_end);                                                                                     \
    return hipGetLastError();
    MP_RESIDUE_SPLIT_CASE(1)
    MP_RESIDUE_SPLIT_CASE(2)
    MP_RESIDUE_SPLIT_CASE(3)
    MP_RESIDUE_SPLIT_CASE(4)
    MP_RESIDUE_SPLIT_CASE(5)
    MP_RESIDUE_SPLIT_CASE(6)
    MP_RESIDUE_SPLIT_CASE(7)
    MP_RESIDUE_SPLIT_CASE(8)
    MP_RESIDUE_SPLIT_CASE(9)
#undef MP_RESIDUE_SPLIT_CASE
    default:
      return hipErrorInvalidValue;
  }
}

template <typename T, int C>
hipError_t combine_launch(int nwc, bool chunks, int64_t blocks, const ResidueDesc *descs, const int *prefix, int nprod,
                          hipStream_t st) {
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  if (chunks) {
    hipLaunchKernelGGL(k_residue_fold, dim3((unsigned)blocks), dim3(kThreads), 0, st, descs, prefix, nprod);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
  }
  // a workgroup's two half blocks one after the other, or a workgroup each where
  // that still leaves some CUs idle
  const dim3 grid((unsigned)blocks, blocks <= 128 ? 2 : 1);
  switch (nwc) {
#define MP_RESIDUE_COMBINE_CASE(NWC)                                                                             \
  case NWC: {                                                                                                    \
    hipLaunchKernelGGL((k_residue_combine<T, C, NWC>), grid, dim3(kThreads), 0, st, descs, prefix, nprod); \
    return hipGetLastError();                                                                                    \
  }
    MP_RESIDUE_COMBINE_CASE(2)
    MP_RESIDUE_COMBINE_CASE(3)
    MP_RESIDUE_COMBINE_CASE(4)
    MP_RESIDUE_COMBINE_CASE(5)
    MP_RESIDUE_COMBINE_CASE(6)
    MP_RESIDUE_COMBINE_CASE(7)
    MP_RESIDUE_COMBINE_CASE(8)
    MP_RESIDUE_COMBINE_CASE(9)
    MP_RESIDUE_COMBINE_CASE(10)
    MP_RESIDUE_COMBINE_CASE(11)
    MP_RESIDUE_COMBINE_CASE(12)
    MP_RESIDUE_COMBINE_CASE(13)
    MP_RESIDUE_COMBINE_CASE(14)
    MP_RESIDUE_COMBINE_CASE(15)
    MP_RESIDUE_COMBINE_CASE(16)
    MP_RESIDUE_COMBINE_CASE(17)
    MP_RESIDUE_COMBINE_CASE(18)
    MP_RESIDUE_COMBINE_CASE(19)
    MP_RESIDUE_COMBINE_CASE(20)
#undef MP_RESIDUE_COMBINE_CASE
    default:
      return hipErrorInvalidValue;
  }
}

// Groups of the bases for `wgs` tiles and k chunks, `slots` workgroups running
// together: of the counts that fill 1, 2, ... rounds the one with the least rounds
// times products a round, with a quarter of a product for a round's start.  Against
// the first count that fills one round (9 tiles in 29 groups ran 261 workgroups in
// two rounds): INT8 DD n = 640 76 -> 66 us, 1100 193 -> 150, 3000 1717 -> 1284; QD
// FLOAT 3000 4727 -> 3358.
int base_groups(int64_t wgs, int slots, int bases, int products) {
  int best = 1;
  double least = 0.0;
  for (int rounds = (int)std::min<int64_t>(1 << 20, ceil_div(wgs, (int64_t)slots)), last = rounds + 7; rounds <= last; ++rounds) {
    const int g = (int)std::min<int64_t>(bases, (int64_t)rounds * slots / wgs);
    const double cost = rounds * ((double)ceil_div(products, g) + 0.25);
    if (least == 0.0 || cost < least) {
      least = cost;
      best = g;
    }
    if (g == bases) break;
  }
  return best;
}

hipError_t gemm_launch(int cfg, const ResiduePlan &p, const int8_t *A, const int8_t *B, const Shape &s, int u_first,
                       int u_end, int m, int n, int8_t *R, const int *skip, hipStream_t st) {
  const int tb = int8_tile_blocks(cfg);
  const int64_t tiles = (s.mbp / tb) * (s.nbp / tb);
  if (tiles > 0x7fffffffLL) return hipErrorInvalidValue;
  // the bases (independent results) spread over gridDim.z, so that the last of the
  // workgroups that run together (one of the 256 x 256 tiles per CU, two of the
  // smaller ones) are as many as the others
  const int64_t nchunks = ceil_div(s.kbp, (int64_t)kChunkBlocks);
  const int groups = base_groups(tiles * nchunks, cfg == 1 ? 512 : 256, u_end - u_first,
                                 residue_pairs_below(u_end, p.nsq) - residue_pairs_below(u_first, p.nsq));
  const dim3 grid((unsigned)tiles, (unsigned)nchunks, (unsigned)groups);
  if (cfg == 1)
    hipLaunchKernelGGL(k_gemm_residue<1>, grid, dim3(64 * Int8Cfg<1>::WM * Int8Cfg<1>::WN), 0, st, A, B, s.mbp, s.nbp,
                       s.kbp, u_first, u_end, p.nsq, p.nplanes, m, n, R, s.r_plane, skip);
  else  // every 256 x 256 configuration
    hipLaunchKernelGGL(k_gemm_residue<3>, grid, dim3(64 * Int8Cfg<3>::WM * Int8Cfg<3>::WN), 0, st, A, B, s.mbp, s.nbp,
                       s.kbp, u_first, u_end, p.nsq, p.nplanes, m, n, R, s.r_plane, skip);
  return hipGetLastError();
}

}  // namespace

// The 256 x 256 tiles, except for a product within one of them, which the smaller
// tiles spread over more CUs (200^2 x 100: INT8 DD 29.8 -> 26.0 us, QD FLOAT 55.7 ->
// 46.5), and where padding to them takes more than 1.4 times the area of the 128 x
// 128 ones (n = 640, 1.44 times: 66.5 -> 58.5 and 148 -> 122).  At 1.2 to 1.4 the two
// are within 4 % (n = 1100: INT8 DD 150 and 148, FLOAT DD 161 and 165), and at 1.0 the
// smaller tiles lose at most sizes (n = 2180: 756 and 844, QD 1974 and 2250); with the
// operands in the caches they gain (n = 512: QD 85.6 and 78.8) or not (DD 45.1 and
// 46.5).
int residue_tile_config(int64_t m, int64_t n, int cfg) {
  if (cfg >= 1 && cfg <= 4) return cfg;
  const int64_t tiles3 = ceil_div(m, 256) * ceil_div(n, 256), tiles1 = ceil_div(m, 128) * ceil_div(n, 128);
  return tiles3 == 1 || 20 * tiles3 > 7 * tiles1 ? 1 : 3;
}

size_t residue_bytes(const ResiduePlan &p, int cfg, int64_t m, int64_t n, int64_t k) {
  const Shape s = shape_of(cfg, m, n, k);
  return header_bytes(p) + (size_t)p.nplanes * (size_t)(s.a_plane + s.b_plane + p.nchunks * s.r_plane);
}

namespace {

// How a product is formed in an arena: whole, with `room` operand planes at a time
// (all of them where they fit), or, where its result planes alone take more than
// half of an arena that not everything fits, as two blocks of C of which the first
// is m x n (m = 0: not even one tile fits).
struct Pieces {
  bool whole = true;
  int room = 0, m = 0, n = 0;
  Pieces(const ResiduePlan &p, int cfg, int m_, int n_, int k, size_t arena) {
    const Shape s = shape_of(cfg, m_, n_, k);
    const size_t result = (size_t)p.nplanes * p.nchunks * s.r_plane;
    const int64_t left = (int64_t)arena - (int64_t)header_bytes(p) - (int64_t)result;
    room = (int)std::min<int64_t>(p.nplanes, left < 0 ? 0 : left / (s.a_plane + s.b_plane));
    if (room == p.nplanes || (2 * result <= arena && room >= 2)) return;
    whole = false;
    // halves of the longer side of C, at a tile edge
    const int longer = std::max(m_, n_), half = (int)(ceil_div(longer, 2 * 256) * 256);
    if (half >= longer) return;  // one tile
    m = m_ >= n_ ? half : m_;
    n = m_ >= n_ ? n_ : half;
  }
};

}  // namespace

ResidueFit residue_fit(const ResiduePlan &p, int cfg, int m, int n, int k, size_t arena) {
  const Pieces piece(p, cfg, m, n, k, arena);
  if (piece.whole) return ResidueFit::kWhole;
  if (piece.m == 0) return ResidueFit::kNone;
  const int m2 = piece.m < m ? m - piece.m : m, n2 = piece.m < m ? n : n - piece.n;
  return residue_fit(p, cfg, piece.m, piece.n, k, arena) == ResidueFit::kNone ||
                 residue_fit(p, cfg, m2, n2, k, arena) == ResidueFit::kNone
             ? ResidueFit::kNone
             : ResidueFit::kBlocks;
}

template <typename T, int C>
hipError_t launch_residue_sample(const ResidueOperand<T> *ops, const int *prefix, int nops, int strips, hipStream_t st) {
  if (strips <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_residue_sample<T, C>), dim3((unsigned)strips), dim3(kThreads), 0, st, ops, prefix, nops);
  return hipGetLastError();
}

template <typename T, int C>
hipError_t launch_residue(const ResidueCall &rc, const SplitOperand<T> &a, const SplitOperand<T> &b, T *Cout,
                          hipEvent_t between, bool first, hipStream_t st) {
  const ResiduePlan &p = rc.plan;
  const Shape s = shape_of(rc.cfg, rc.m, rc.n, rc.k);
  // arena: the uploaded descriptors and table, the result planes, then as many
  // operand planes as fit (Pieces)
  const Pieces piece(p, rc.cfg, rc.m, rc.n, rc.k, rc.arena_bytes);
  const size_t result = (size_t)p.nplanes * p.nchunks * s.r_plane;
  const int room = piece.room;
  if (!piece.whole) {
    if (piece.m == 0) return hipErrorInvalidValue;  // does not fit
    ResidueCall lo = rc, hi = rc;
    SplitOperand<T> a2 = a, b2 = b;
    T *C2 = Cout;
    lo.m = piece.m;
    lo.n = piece.n;
    if (lo.m < rc.m) {
      hi.m = rc.m - lo.m;
      hi.exp_a += lo.m;
      a2.X += lo.m * a.sv;
      C2 += lo.m;
    } else {
      hi.n = rc.n - lo.n;
      hi.exp_b += lo.n;
      b2.X += lo.n * b.sv;
      C2 += (int64_t)lo.n * rc.ldc;
    }
    SplitOperand<T> a1 = a, b1 = b;
    a1.nvec = lo.m;
    b1.nvec = lo.n;
    a2.nvec = hi.m;
    b2.nvec = hi.n;
    hipError_t err = launch_residue<T, C>(lo, a1, b1, Cout, between, first, st);
    if (err == hipSuccess) err = launch_residue<T, C>(hi, a2, b2, C2, nullptr, false, st);
    return err;
  }
  int8_t *R = reinterpret_cast<int8_t *>(planes_of(rc.arena, p));
  int8_t *Ap = R + result, *Bp = Ap + (size_t)room * s.a_plane;

  const std::vector<uint32_t> &table = residue_table(p.nunits, p.nsq, p.nwc);
  struct Head {
    ResidueOperand<T> op[2];
    ResidueDesc d;
    int prefix[6];  // of the split blocks, of the product, of the sampled strips
  } h{};
  static_assert(sizeof(Head) <= kHeadBytes && sizeof(Head) % 4 == 0, "uploaded in words");
  for (int i = 0; i < 2; ++i) {
    const SplitOperand<T> &o = i == 0 ? a : b;
    ResidueOperand<T> &r = h.op[i];
    r.X = o.X;
    r.comp_stride = o.comp_stride;
    r.sv = o.sv;
    r.sp = o.sp;
    r.nvec = o.nvec;
    r.len = o.len;
    r.orient = o.orient;
    r.bits = p.bits;
    r.float_form = rc.float_form;
    r.slice_bits = rc.slice_bits;
    r.passes = rc.passes;
    r.planes = i == 0 ? Ap : Bp;
    r.nbp = i == 0 ? s.mbp : s.nbp;
    r.kbp = s.kbp;
    r.mu = i == 0 ? rc.mu_a : rc.mu_b;
    r.exps = i == 0 ? rc.exp_a : rc.exp_b;
    r.state = i == 0 ? rc.state_a : rc.state_b;
    r.flag = rc.flag;
    r.nunits = p.nunits;
    r.nsq = p.nsq;
  }
  const int64_t ba = s.mbp * s.kbp, bb = s.nbp * s.kbp;
  if (ba + bb > 0x7fffffffLL) return hipErrorInvalidValue;
  h.prefix[0] = 0;
  h.prefix[1] = (int)ba;
  const int sa = ceil_div(rc.m, 16), sb = ceil_div(rc.n, 16);
  h.prefix[5] = sa;
  h.d.R = R;
  h.d.table = reinterpret_cast<const uint32_t *>(rc.arena + kHeadBytes);
  h.d.EA = rc.exp_a;
  h.d.EB = rc.exp_b;
  h.d.mbp = s.mbp;
  h.d.nbp = s.nbp;
  h.d.kbp = s.kbp;
  h.d.plane = s.r_plane;
  h.d.nunits = p.nunits;
  h.d.nsq = p.nsq;
  h.d.nplanes = p.nplanes;
  h.d.bits = p.bits;
  h.d.nchunks = p.nchunks;
  h.d.m = rc.m;
  h.d.n = rc.n;
  h.d.ldc = rc.ldc;
  h.d.C = Cout;
  h.d.c_stride = rc.c_stride;
  h.d.skip = rc.flag;

  hipError_t err = hipSuccess;
  const bool begin = rc.k <= kBeginLength;
  const size_t hw = kHeadBytes / 4, words = hw + table.size();
  for (size_t at = 0; at < words; at += kUploadWords) {
    Upload up;
    const size_t n = std::min<size_t>(kUploadWords, words - at);
    for (size_t i = 0; i < n; ++i)
      up.w[i] = at + i >= hw                  ? table[at + i - hw]
                : at + i < sizeof(Head) / 4 ? reinterpret_cast<const uint32_t *>(&h)[at + i]
                                            : 0u;
    uint32_t *dst = reinterpret_cast<uint32_t *>(rc.arena) + at;
    const bool last = at + n == words;
    int *flag = last && first ? rc.flag : nullptr;
    if (begin && last) {
      using U = typename bits_of<T>::type;
      const MaxOperand<T> va{a.X, a.comp_stride, a.sv, a.sp, a.nvec, a.len, 0, static_cast<U *>(rc.mu_a), rc.state_a};
      const MaxOperand<T> vb{b.X, b.comp_stride, b.sv, b.sp, b.nvec, b.len, 1, static_cast<U *>(rc.mu_b), rc.state_b};
      const GridOfSlices grid{p.bits, rc.slice_bits, rc.passes};
      if (rc.float_form)
        hipLaunchKernelGGL((k_residue_begin<T, C>), dim3((unsigned)(sa + sb)), dim3(kThreads), 0, st, up, (int)n, sa,
                           dst, va, vb, grid, flag);
      else
        hipLaunchKernelGGL((k_residue_begin<T, 0>), dim3((unsigned)(sa + sb)), dim3(kThreads), 0, st, up, (int)n, sa,
                           dst, va, vb, grid, flag);
    } else {
      const int64_t n0 = last ? rc.clear_words : 0;
      const int64_t blocks = std::min<int64_t>(256, std::max<int64_t>(4, ceil_div(n0, (int64_t)kThreads)));
      hipLaunchKernelGGL(k_upload, dim3((unsigned)blocks), dim3(kThreads), 0, st, up, (int)n, dst, rc.clear, n0,
                         reinterpret_cast<uint32_t *>(flag), (int64_t)(flag ? 1 : 0));
    }
    if ((err = hipGetLastError()) != hipSuccess) return err;
  }
  const auto *prefix = reinterpret_cast<const int *>(rc.arena + offsetof(Head, prefix));
  if (!begin) {
    SplitOperand<T> ma = a, mb = b;
    ma.mu = rc.mu_a;
    mb.mu = rc.mu_b;
    if ((err = launch_split_max0(ma, mb, st)) != hipSuccess) return err;
    if (rc.float_form &&
        (err = launch_residue_sample<T, C>(reinterpret_cast<const ResidueOperand<T> *>(rc.arena), prefix + 4, 2, sa + sb,
                                           st)) != hipSuccess)
      return err;
  }
  const auto *ops = reinterpret_cast<const ResidueOperand<T> *>(rc.arena);
  const auto *descs = reinterpret_cast<const ResidueDesc *>(rc.arena + offsetof(Head, d));
  for (int u0 = 0; u0 < p.nunits;) {
    int u1 = u0 + 1;
    while (u1 < p.nunits && group_planes(u0, u1 + 1, p.nsq) <= room) ++u1;
    // a grid of few blocks spreads the row blocks over gridDim.y, one pass each or two
    const int passes = 2 + (p.nsq + 31) / 32;
    const int parts = u1 - u0 <= 32 && p.nsq <= u0 ? 1 : ba + bb <= 128 ? passes : ba + bb <= 512 ? 2 : 1;
    if ((err = split_launch<T, C>(p.nw, dim3((unsigned)(ba + bb), (unsigned)parts), ops, prefix, 2, 0, u0, u1, st)) !=
        hipSuccess)
      return err;
    if (between && u0 == 0) (void)hipEventRecord(between, st);
    if ((err = gemm_launch(rc.cfg, p, Ap, Bp, s, u0, u1, rc.m, rc.n, R, rc.flag, st)) != hipSuccess) return err;
    u0 = u1;
  }
  return combine_launch<T, C>(p.nwc, p.nchunks > 1, s.mbp * s.nbp, descs, prefix + 2, 1, st);
}

template <typename T, int C>
hipError_t launch_residue(const ResidueCall &rc, const SplitOperand<T> &a, const SplitOperand<T> &b, T *Cout,
                          hipEvent_t between, hipStream_t st) {
  return launch_residue<T, C>(rc, a, b, Cout, between, true, st);
}

template <typename T, int C>
hipError_t launch_residue_split_batched(int nw, const ResidueOperand<T> *ops, const int *prefix, int nops, int blocks,
                                        hipStream_t st) {
  if (blocks <= 0) return hipSuccess;
  return split_launch<T, C>(nw, dim3((unsigned)blocks), ops, prefix, nops, 1, 0, -1, st);
}

hipError_t launch_gemm_residue_batched(const ResidueDesc *descs, const int4 *items, int nitems1, int nitems3,
                                       const int *bounds, int *counters, hipStream_t st) {
  // 128 x 128 tiles: two workgroups per CU; 256 x 256: one
  if (nitems1 > 0) {
    hipLaunchKernelGGL(k_gemm_residue_batched<1>, dim3(std::min(nitems1, 512)),
                       dim3(64 * Int8Cfg<1>::WM * Int8Cfg<1>::WN), 0, st, descs, items, bounds, counters);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
  }
  if (nitems3 > 0)
    hipLaunchKernelGGL(k_gemm_residue_batched<3>, dim3(std::min(nitems3, 256)),
                       dim3(64 * Int8Cfg<3>::WM * Int8Cfg<3>::WN), 0, st, descs, items + nitems1, bounds + kXcds + 1,
                       counters + kXcds);
  return hipGetLastError();
}

template <typename T, int C>
hipError_t launch_residue_combine_batched(int nwc, bool chunks, const ResidueDesc *descs, const int *prefix, int nprod,
                                          int64_t blocks, hipStream_t st) {
  if (blocks <= 0) return hipSuccess;
  return combine_launch<T, C>(nwc, chunks, blocks, descs, prefix, nprod, st);
}

#define MP_RESIDUE_INST(T, C)                                                                                   \
  template hipError_t launch_residue<T, C>(const ResidueCall &, const SplitOperand<T> &, const SplitOperand<T> &, T *, \
                                           hipEvent_t, hipStream_t);                                            \
  template hipError_t launch_residue_sample<T, C>(const ResidueOperand<T> *, const int *, int, int, hipStream_t); \
  template hipError_t launch_residue_split_batched<T, C>(int, const ResidueOperand<T> *, const int *, int, int, \
                                                         hipStream_t);                                          \
  template hipError_t launch_residue_combine_batched<T, C>(int, bool, const ResidueDesc *, const int *, int, int64_t, \
                                                           hipStream_t);
MP_RESIDUE_INST(double, 2)
MP_RESIDUE_INST(double, 3)
MP_RESIDUE_INST(double, 4)
MP_RESIDUE_INST(float, 3)
#undef MP_RESIDUE_INST

}  // namespace mp
