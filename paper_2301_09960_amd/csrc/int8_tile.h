// One tile of C on the INT8 matrix cores, shared by the digit-sum GEMM
// (int8.hip) and the residue GEMM (residue.hip).
//
// Both multiply pairs of INT8 planes of A and B: a sequence of diagonals, each
// the sum of a few pairs A_x B_y with the k loops of the pairs concatenated in
// one 32-bit accumulator.  What a diagonal is, and what happens to its exact
// sum, is the `Work` type's business:
//   int pairs() const                  pairs of this work item in all
//   void first(PairCursor &) const     its first pair
//   void next(PairCursor &) const      the pair after it
//   int a_plane / b_plane(cursor)      the planes of a pair
//   bool diagonal_ends(cursor)         the pair is its diagonal's last
//   void finish<BI, BJ>(cursor, acc, bi, bj, lane)   takes a complete sum and
//                                      leaves what the next diagonal starts from
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "layout.h"

namespace mp {

typedef int i4v __attribute__((ext_vector_type(4)));
typedef int i16v __attribute__((ext_vector_type(16)));

constexpr int kInt8GroupM = 8;      // tile rows of a group in the tile order

__device__ __forceinline__ void int8_tile_coords(int bid, int nblocks, int tiles_m, int tiles_n, int &tm, int &tn) {
  const int q = nblocks / 8, r = nblocks % 8;
  const int xcd = bid % 8, local = bid / 8;
  const int L = xcd * q + (xcd < r ? xcd : r) + local;
  const int per_group = kInt8GroupM * tiles_n;
  const int group = L / per_group;
  const int first_m = group * kInt8GroupM;
  const int gsize = (tiles_m - first_m) < kInt8GroupM ? (tiles_m - first_m) : kInt8GroupM;
  const int in_group = L % per_group;
  tm = first_m + in_group % gsize;
  tn = in_group / gsize;
}

__device__ __forceinline__ void load_lds16(const void *src, void *lds_dst) {
  __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void *)lds_dst, 16, 0, 0);
}
template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Waits until this wavefront's loads of the step about to be computed have
// landed: with an NS-stage ring, min(NS - 2, later) later steps (kL loads
// each) may stay in flight.
template <int NS, int kL>
__device__ __forceinline__ void wait_step(int64_t later) {
  static_assert(NS >= 2 && NS <= 4, "wait chain covers rings of 2 to 4 stages");
  if constexpr (NS >= 4) {
    if (later >= 2)
      wait_vm<2 * kL>();
    else if (later == 1)
      wait_vm<kL>();
    else
      wait_vm<0>();
  } else if constexpr (NS == 3) {
    if (later >= 1)
      wait_vm<kL>();
    else
      wait_vm<0>();
  } else {
    wait_vm<0>();
  }
}

// Tile configurations (in 32 x 32 blocks): TB x TB tile of C, WM x WN
// wavefronts, KSB 32-wide k blocks per pipeline step, NS LDS stages.
//   config 1: 128 x 128 tile, 4 wavefronts of 64 x 64 (small products), k
//             steps of 128 in a 2-stage ring (two workgroups per CU), each
//             step's loads over its first half
//   config 2: 256 x 256 tile, 4 wavefronts of 128 x 128 (accumulators in AGPRs;
//             LDS traffic per instruction halved)
//   config 4: 256 x 256 tile, 16 wavefronts of 64 x 64 (more wavefronts to
//             hide latency, more LDS reads per instruction), k steps of 128
//   config 3: 256 x 256 tile, 8 wavefronts of 128 x 64, k steps of 128 in a
//             2-stage ring (half the barriers of 64-wide steps, and 64 KiB
//             requested per step)
// KSB is 1 or 2 times kKStepBlocks8, the k padding unit of the INT8 slices (64
// k): with 4-block steps a pair's last step in a k chunk may hold 2 blocks.
template <int CFG> struct Int8Cfg;
template <> struct Int8Cfg<1> { static constexpr int TB = 4, WM = 2, WN = 2, KSB = 4, NS = 2, SPACING = 1; };
template <> struct Int8Cfg<2> { static constexpr int TB = 8, WM = 2, WN = 2, KSB = 2, NS = 4, SPACING = 0; };
template <> struct Int8Cfg<3> { static constexpr int TB = 8, WM = 2, WN = 4, KSB = 4, NS = 2, SPACING = 3; };
template <> struct Int8Cfg<4> { static constexpr int TB = 8, WM = 4, WN = 4, KSB = 4, NS = 2, SPACING = 0; };

// Matrix-core instructions between two loads of the next step: spread over the
// whole step by default, fewer where a configuration issues its loads earlier.
template <typename G>
constexpr int load_spacing(int even) {
  return G::SPACING > 0 ? G::SPACING : even;
}

template <int CFG>
constexpr int int8_stage_bytes() {
  return 2 * Int8Cfg<CFG>::TB * Int8Cfg<CFG>::KSB * 1024;  // A panel, then B panel
}

struct PairCursor {
  int u, g, s;  // unit, diagonal within it, pair within the diagonal (g and s from 1)
};

// The pairs of `work` on one tile (tm, tn) and k chunk: operand panels (TB
// blocks x KSB k blocks of a plane of A and one of B) move global -> LDS by
// direct loads into a ring of NS stages, NS - 1 steps ahead; each step waits
// for its own loads and passes one barrier.
//
// Each wavefront moves kL 1 KiB pieces of one operand per step.  Their global
// offsets from the step's panel base and their LDS offsets are fixed for the
// whole tile, so a load costs one 64-bit add; and the loads of the next step
// are spread between this step's matrix-core instructions (one per kEvery),
// which keeps the matrix cores fed where a burst of LDS-direct loads would
// stall them.  With `quit` (uniform) nothing is formed: it is looked at behind the
// first loads, whose latency covers that of a word just read (in front of them it
// took 0.9 of 17 us, TD 200 x 150 x 333).  The 256 x 256 configuration with its 2-stage ring issues them
// over the first three quarters of the step (one per 3 instructions instead of
// one per 4), so that the last ones land before the step ends.
template <int CFG, typename Work>
__device__ __forceinline__ void gemm_int8_tile(const Work &work, const int8_t *__restrict__ Apk,
                                               const int8_t *__restrict__ Bpk, int64_t mbp, int64_t nbp, int64_t kbp,
                                               int64_t kb0, int nks, int last, int m, int n, int tm, int tn,
                                               int quit, int8_t *lds) {
  using G = Int8Cfg<CFG>;
  constexpr int TB = G::TB, WM = G::WM, WN = G::WN, KSB = G::KSB, NS = G::NS;
  constexpr int BI = TB / WM, BJ = TB / WN;
  constexpr int NW = WM * WN;
  constexpr int kPanel = TB * KSB * 1024;
  constexpr int kInst = 2 * TB * KSB;  // 1 KiB wavefront instructions per step
  constexpr int kL = kInst / NW;
  constexpr int kMma = KSB * BI * BJ;  // matrix-core instructions per wavefront per step
  constexpr int kEvery = load_spacing<G>(kMma / kL);
  static_assert(kInst % NW == 0, "staging split");
  static_assert((TB * KSB) % kL == 0, "a wavefront's loads of a step come from one operand");
  static_assert(kMma % kL == 0, "one load per fixed number of matrix-core instructions");
  static_assert(kEvery * kL <= kMma, "every load of the next step is issued within this step");
  // a pair's k blocks in the chunk are a multiple of kKStepBlocks8: its steps
  // are full but the last, which holds `last` blocks (KSB / 2 or KSB)
  static_assert(KSB % kKStepBlocks8 == 0 && KSB <= 2 * kKStepBlocks8, "k steps and the k padding unit");

  const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
  // wavefront -> (wm, wn).  With 2 x 4 wavefronts (two per SIMD: w and w + 4)
  // the two of a SIMD differ in both wm and wn, so that a tile padded in m or
  // in n leaves each SIMD a wavefront with work.
  int wm, wn;
  if constexpr (WM == 2 && WN == 4) {
    const int sw = wave & 3, hw = wave >> 2;
    wm = (sw & 1) ^ hw;
    wn = (sw >> 1) + 2 * hw;
  } else {
    wm = wave % WM;
    wn = wave / WM;
  }
  const int64_t total = (int64_t)work.pairs() * nks;

  // this wavefront's share of a step: operand op_w, pieces j = 0..kL-1
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  const int op_w = (wave_u * kL) / (TB * KSB);
  uint32_t goff[kL];  // byte offset from the step's panel base (per lane; k <= 2^20 keeps it below 2^32)
  int loff[kL];       // byte offset in the stage (uniform)
  uint32_t beyond[kL];  // in a pair's short last step the piece lies past the pair's k: load piece kb - KSB / 2
#pragma unroll
  for (int j = 0; j < kL; ++j) {
    const int r = (wave_u * kL + j) % (TB * KSB);
    const int blk = r / KSB, kb = r % KSB;
    goff[j] = (uint32_t)(((int64_t)blk * kbp + kb) * 1024) + 16u * (uint32_t)lane;
    loff[j] = op_w * kPanel + (blk * KSB + kb) * 1024;
    beyond[j] = kb >= KSB / 2 ? (uint32_t)(KSB / 2) * 1024u : 0u;
  }
  // every step loads kL pieces (the wait counts assume it): a pair's short
  // last step re-loads pieces of its own range into stage slots that no
  // matrix-core instruction reads
  auto piece = [&](int j, int ks) -> uint32_t { return goff[j] - (ks == nks - 1 && last < KSB ? beyond[j] : 0u); };

  PairCursor lc;  // load cursor: pair, and k step within it
  int lks = 0;
  work.first(lc);
  int64_t issued = 0;
  // panel base of the step at the load cursor, and its ring slot
  auto panel_base = [&]() -> const int8_t * {
    return op_w == 0 ? Apk + (((int64_t)work.a_plane(lc) * mbp + (int64_t)tm * TB) * kbp + kb0 + (int64_t)lks * KSB) * 1024
                     : Bpk + (((int64_t)work.b_plane(lc) * nbp + (int64_t)tn * TB) * kbp + kb0 + (int64_t)lks * KSB) * 1024;
  };
  auto advance = [&]() {
    ++issued;
    if (++lks == nks) {
      lks = 0;
      work.next(lc);
    }
  };

  i16v acc[BJ][BI];
#pragma unroll
  for (int y = 0; y < BJ; ++y)
#pragma unroll
    for (int x = 0; x < BI; ++x)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[y][x][r] = 0;

  wait_vm<0>();
#pragma unroll
  for (int s0 = 0; s0 < NS - 1; ++s0)
    if (issued < total) {
      const int8_t *src = panel_base();
      int8_t *dst = lds + (issued % NS) * int8_stage_bytes<CFG>();
#pragma unroll
      for (int j = 0; j < kL; ++j) load_lds16(src + piece(j, lks), dst + loff[j]);
      advance();
    }

  if (__builtin_amdgcn_readfirstlane(quit)) {
    wait_vm<0>();
    return;
  }

  // A wavefront whose blocks are all padding (rows from m or columns from n
  // on) has no matrix-core work: it only moves its share of the panels, at the
  // places and about the pace (64 cycles per two instructions) of the others,
  // and passes the same barriers.  It leaves its blocks of the result planes
  // unwritten; no element outside m x n is read from them.
  if (__builtin_amdgcn_readfirstlane(((int64_t)tm * TB + wm * BI) * 32 >= m || ((int64_t)tn * TB + wn * BJ) * 32 >= n
                                         ? 1
                                         : 0)) {
    for (int64_t step = 0; step < total; ++step) {
      wait_step<NS, kL>(total - 1 - step);
      __builtin_amdgcn_s_barrier();
      const bool more = issued < total;
      const int8_t *nsrc = more ? panel_base() : Apk;
      int8_t *ndst = lds + (issued % NS) * int8_stage_bytes<CFG>();
      const uint32_t next_short = lks == nks - 1 && last < KSB ? 1u : 0u;
#pragma unroll
      for (int mma = 0; mma < kMma; ++mma) {
        if (mma % kEvery == 0 && mma / kEvery < kL && more)
          load_lds16(nsrc + (goff[mma / kEvery] - next_short * beyond[mma / kEvery]), ndst + loff[mma / kEvery]);
        if (mma % 2 == 1) __builtin_amdgcn_s_sleep(1);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (more) advance();
    }
    __builtin_amdgcn_s_barrier();
    return;
  }

  PairCursor cc;  // compute cursor
  int cks = 0;
  work.first(cc);
  for (int64_t step = 0; step < total; ++step) {
    wait_step<NS, kL>(total - 1 - step);
    __builtin_amdgcn_s_barrier();
    // the step NS - 1 ahead goes into the slot computed in the previous step
    const bool more = issued < total;
    const int8_t *nsrc = more ? panel_base() : Apk;
    int8_t *ndst = lds + (issued % NS) * int8_stage_bytes<CFG>();

    const int8_t *stage = lds + (step % NS) * int8_stage_bytes<CFG>();
    // a pair's short last step holds the first KSB / 2 k blocks (the only
    // short length): its second half is skipped, on a uniform branch
    const bool short_step = cks == nks - 1 && last < KSB;
    const uint32_t next_short = lks == nks - 1 && last < KSB ? 1u : 0u;  // the step being loaded is short
#pragma unroll
    for (int kb = 0; kb < KSB; ++kb) {
      const bool run = kb < KSB / 2 || !short_step;
      i4v fa[BI], fb[BJ];
      if (run) {
#pragma unroll
        for (int x = 0; x < BI; ++x)
          fa[x] = *reinterpret_cast<const i4v *>(stage + ((wm * BI + x) * KSB + kb) * 1024 + 16 * lane);
#pragma unroll
        for (int y = 0; y < BJ; ++y)
          fb[y] = *reinterpret_cast<const i4v *>(stage + kPanel + ((wn * BJ + y) * KSB + kb) * 1024 + 16 * lane);
      }
#pragma unroll
      for (int y = 0; y < BJ; ++y)
#pragma unroll
        for (int x = 0; x < BI; ++x) {
          const int mma = (kb * BJ + y) * BI + x;
          if (mma % kEvery == 0 && mma / kEvery < kL && more)
            load_lds16(nsrc + (goff[mma / kEvery] - next_short * beyond[mma / kEvery]), ndst + loff[mma / kEvery]);
          if (run) acc[y][x] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fb[y], fa[x], acc[y][x], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);  // keep the loads where they were placed
        }
    }
    if (more) advance();
    if (++cks == nks) {
      cks = 0;
      if (work.diagonal_ends(cc))
        work.template finish<BI, BJ>(cc, acc, (int64_t)tm * TB + wm * BI, (int64_t)tn * TB + wn * BJ, lane);
      work.next(cc);
    }
  }
  __builtin_amdgcn_s_barrier();
}

}  // namespace mp
