// Products of exact integers by residues (interfaces of residue.hip).
//
// Every operand element is rounded once to an integer W on its row's (column's)
// grid: x = W 2^(E - bits), |W| <= 2^bits.  The integer product
// X_ij = sum_p W_ip V_pj, |X| <= k 2^(2 bits), is formed exactly from its
// residues modulo pairwise coprime moduli whose product M exceeds 2 |X|: each
// residue is one product on the INT8 matrix cores, and the Chinese remainder
// theorem puts X together (Knuth, The Art of Computer Programming, volume 2,
// 4.3.2).  About 2 bits / 7.7 matrix products replace the D (D + 1) / 2 slice
// products of the same operands (bits ~ 7 D: 32 instead of 136 for DD at
// k = 4096, 73 instead of 465 for QD), and nothing is left out: X is the full
// product, where the slice triangle drops the pairs below its last diagonal.
//
// Moduli.  The bases s_0 = 256, s_1 = 255, ... s_48 = 29 are the greedy
// pairwise coprime sequence below 257 (every residue fits a signed byte).  A
// plan takes the first nunits of them; the first nsq enter squared, for their
// residue needs a second s-adic digit: with x = x0 + s x1 and y = y0 + s y1,
// x y mod s^2 = x0 y0 + s (x0 y1 + x1 y0), three INT8 products in two
// diagonals (the carry of the first, (sum - t0) / s, starts the second).  The
// 49 bases hold 341 bits at one product each; a square adds 8 to 5 bits for two.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "internal.h"
#include "layout.h"

namespace mp {

constexpr int kNumBases = 49;
constexpr int kMaxWindowWords = 9;                 // W in at most 9 words: bits <= 286
constexpr int kMaxResidueBits = 32 * kMaxWindowWords - 2;
constexpr int kMaxCombineWords = 20;               // words of the combine's sums
constexpr int kChunkBlocks = 1024;                 // k blocks of one 32-bit sum: 32768 k
constexpr int kNonFinite = INT32_MAX;              // exponent of a vector holding an infinity or NaN

struct ResiduePlan {
  int bits;                     // |W| <= 2^bits
  int nunits, nsq, nplanes;     // bases, of them squared, digit planes (nunits + nsq)
  int nchunks;                  // k chunks with result planes of their own
  int nw, nwc;                  // 32-bit words of W, and of the combine's sums
  int products() const { return nunits + 2 * nsq; }
};

// The cheapest plan whose moduli cover |X| <= k 2^(2 bits); false when none does.
bool residue_plan(int bits, int64_t k, ResiduePlan &p);

// Combine constants of a plan (host memory, kept for the process; a function of
// (nunits, nsq, nwc) alone): the weight of every plane in balanced base-256
// digits, a row of bytes (plane by plane, 32 or a multiple) per digit; then M in nwc balanced words; then a multiple of 1 / M
// as a binary64.
const std::vector<uint32_t> &residue_table(int nunits, int nsq, int nwc);

// One operand of the residue split.  E: FLOAT form ceil(log2 mu) of the
// vector, INT8 form 1 + ilogb(mu); kZeroExp for a zero vector.
template <typename T>
struct ResidueOperand {
  const T *X;
  int64_t comp_stride, sv, sp;
  int nvec, len, orient;
  int bits, float_form;
  int slice_bits, passes;  // float_form: b and D of the slices it stands for
  int8_t *planes;        // residue planes (layout.h, INT8 blocks)
  int64_t nbp, kbp;
  void *mu;              // maxima (launch_split_max0)
  int *exps;
  int *state;            // float_form: one word per vector, from the samples (launch_residue_sample)
  int *flag, *any;       // float_form: set when the slices must be used instead (any may be null)
  int nunits, nsq;
  const int *padded;     // where it is given and 0 the padding of k is zero already
};

struct ResidueDesc {
  const int8_t *A, *B;
  int8_t *R;              // residue planes of the product (blocked as the INT8 sums)
  const uint32_t *table;
  const int *EA, *EB;
  int64_t mbp, nbp, kbp, plane;
  int nunits, nsq, nplanes, nchunks, groups, bits, m, n, ldc;
  void *C;
  int64_t c_stride;
  const int *skip;        // FLOAT form: where set, C is left to the slices, whose split may read A or B from it
};

// One product by residues.  clear: device memory holding the maxima, cleared by the
// call where it has to be.  arena: a call takes
// residue_bytes() of it; with less, the product is formed in parts (bases, then
// blocks of C), with the same result.
struct ResidueCall {
  ResiduePlan plan;
  int cfg;               // INT8 tile configuration
  int float_form, slice_bits, passes;
  int m, n, k, ldc;
  int64_t c_stride;
  int *exp_a, *exp_b;    // m and n exponents
  void *mu_a, *mu_b;     // m and n maxima
  int *state_a, *state_b;  // FLOAT form: m and n words; INT8 form null
  uint32_t *clear;
  int64_t clear_words;
  int *flag;             // FLOAT form: cleared, then set if the slices must form the product
  char *arena;
  size_t arena_bytes;
};
// Tile configuration of one m x n product by residues (cfg > 0 forces one).
int residue_tile_config(int64_t m, int64_t n, int cfg);
size_t residue_bytes(const ResiduePlan &p, int cfg, int64_t m, int64_t n, int64_t k);
// How launch_residue forms a product in an arena of a size: with every operand
// element read before C is written (whole), in blocks of C one after the other, or
// not at all.
enum class ResidueFit { kNone, kBlocks, kWhole };
ResidueFit residue_fit(const ResiduePlan &p, int cfg, int m, int n, int k, size_t arena);
template <typename T, int C>
hipError_t launch_residue(const ResidueCall &rc, const SplitOperand<T> &a, const SplitOperand<T> &b, T *Cout,
                          hipEvent_t between, hipStream_t st);


// Many products at once (batch.hip): descriptors, prefix sums and work items in
// device memory.  The residue split writes the blocks that hold elements, and A's
// padding of k; prefix: running sums of these blocks per operand, and of the 32 x 32 blocks of C per product for the combine.  nw is the
// batch's largest; a combine launch takes products of one nwc
// (chunks: some of them have several k chunks).  Items (product, tile, k chunk, unit group) as two
// sets of kXcds per-XCD lists (take_item): nitems1 of 128 x 128 tiles, then
// nitems3 of 256 x 256; counters: 2 kXcds words, cleared by the caller.
template <typename T>
hipError_t launch_residue_max_batched(const ResidueOperand<T> *ops, const int *prefix, int nops, int tiles,
                                      hipStream_t st);
// FLOAT form, behind the maxima: states from samples (residue.hip) of the operands'
// vectors, in strips of 16; prefix: running sums of the strips.
template <typename T, int C>
hipError_t launch_residue_sample(const ResidueOperand<T> *ops, const int *prefix, int nops, int strips, hipStream_t st);
template <typename T, int C>
hipError_t launch_residue_split_batched(int nw, const ResidueOperand<T> *ops, const int *prefix, int nops, int blocks,
                                        hipStream_t st);
hipError_t launch_gemm_residue_batched(const ResidueDesc *descs, const int4 *items, int nitems1, int nitems3,
                                       const int *bounds, int *counters, hipStream_t st);
template <typename T, int C>
hipError_t launch_residue_combine_batched(int nwc, bool chunks, const ResidueDesc *descs, const int *prefix, int nprod,
                                          int64_t blocks, hipStream_t st);

// The first unit of each of `groups` parts of the units [first, end) of nearly
// equal pair counts, as the kernels cut them.
__host__ __device__ inline int residue_pairs_below(int u, int nsq) { return u <= nsq ? 3 * u : 2 * nsq + u; }
__host__ __device__ inline int residue_group_start(int first, int end, int nsq, int z, int groups) {
  if (z >= groups) return end;
  const int base = residue_pairs_below(first, nsq), pairs = residue_pairs_below(end, nsq) - base;
  const int target = (int)((int64_t)pairs * z / groups);
  int u = first;
  while (u < end && residue_pairs_below(u, nsq) - base < target) ++u;
  return u;
}

}  // namespace mp
