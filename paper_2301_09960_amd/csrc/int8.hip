// INT8-slice form (the precision form; not in the paper): digit slices on the
// INT8 matrix cores with exact 32-bit integer sums.
//
// With digit units u_s = 2^(E - 6 - 7 (s - 1)) (split.hip), every product
// A_s B_t on the anti-diagonal s + t = g + 1 has the same unit
// 2^(E_i + F_j + 2 - 7 (g + 1)), so the D (D + 1) / 2 slice products collapse
// into D exact integer diagonal sums S_g = sum_{s + t = g + 1} A_s B_t, each a
// GEMM with the k loops of its g pairs concatenated.  |digit| <= 64, so a
// 32-bit sum of up to 2^31 / 4096 digit products is exact; k is cut into
// chunks short enough for that bound, each chunk writing its own partial S_g.
//
// k_gemm_int8: one workgroup per tile of C (128 x 128 or 256 x 256), k chunk
// and group of diagonals (the diagonal sums are independent, so a small
// product spreads its diagonals over the grid); each wavefront owns a grid of
// 32 x 32 blocks of v_mfma_i32_32x32x32_i8.  Panels of A_s and B_t (64 or 128
// k per step) move global -> LDS by direct loads into a ring of 2 to 4
// stages, as in the floating-point kernel.  After the last pair of a diagonal
// the 32-bit tile is written to the S_g plane in a blocked layout (16-byte
// stores per lane).
//
// The DD, TD and QD products take the residues of residue.hip instead (32
// INT8 products for 136 digit pairs at DD, k = 4096); this kernel forms the
// longer expansions and the diagonal sums that mpgemm_debug_products returns.
//
// k_int8_combine: per element, C = sum_g S_g 2^(E_i + F_j + 2 - 7 (g + 1)):
// runs of consecutive diagonals summed exactly in 64-bit integers, each run
// split exactly into two binary64 values, added with TwoSum into a (c+1)-term
// accumulator and renormalized into the c components of C (it reads D 32-bit
// sums per element per chunk and writes C once).
#include <algorithm>

#include "int8_tile.h"
#include "internal.h"
#include "layout.h"
#include "mp_device.h"

namespace mp {
namespace {

// Work of one tile: the diagonals g0 .. g1 - 1 of the digit planes, each
// written as an exact 32-bit partial sum (blocked layout, below).
struct SumsWork {
  int g0, g1;
  int32_t *S;
  int64_t plane, mbp;
  int chunk, nchunks;
  __device__ int pairs() const { return (g1 - 1) * g1 / 2 - (g0 - 1) * g0 / 2; }
  __device__ void first(PairCursor &c) const { c = {0, g0, 1}; }
  __device__ void next(PairCursor &c) const {
    if (++c.s > c.g) {
      ++c.g;
      c.s = 1;
    }
  }
  __device__ int a_plane(const PairCursor &c) const { return c.s - 1; }
  __device__ int b_plane(const PairCursor &c) const { return c.g - c.s; }
  __device__ bool diagonal_ends(const PairCursor &c) const { return c.s == c.g; }
  template <int BI, int BJ>
  __device__ __forceinline__ void finish(const PairCursor &c, i16v (&acc)[BJ][BI], int64_t bi0, int64_t bj0,
                                         int lane) const {
    int32_t *out = S + ((int64_t)(c.g - 1) * nchunks + chunk) * plane;
#pragma unroll
    for (int y = 0; y < BJ; ++y)
#pragma unroll
      for (int x = 0; x < BI; ++x) {
        i4v *dst = reinterpret_cast<i4v *>(out + (((bj0 + y) * mbp + bi0 + x) * 64 + lane) * 16);
#pragma unroll
        for (int v = 0; v < 4; ++v) dst[v] = i4v{acc[y][x][4 * v], acc[y][x][4 * v + 1], acc[y][x][4 * v + 2],
                                                 acc[y][x][4 * v + 3]};
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[y][x][r] = 0;
      }
  }
};

// Diagonals [g0, g1) of group z of `groups`: the D (D + 1) / 2 pairs cut into
// nearly equal parts at diagonal boundaries (a group may be empty).
__device__ __forceinline__ void diagonal_group(int D, int z, int groups, int &g0, int &g1) {
  g0 = 1;
  g1 = D + 1;
  if (groups <= 1) return;
  const int64_t pairs = (int64_t)D * (D + 1) / 2;
  auto first_reaching = [&](int64_t target) {  // smallest g with g (g + 1) / 2 >= target
    int g = 0;
    while ((int64_t)g * (g + 1) / 2 < target) ++g;
    return g;
  };
  g0 = first_reaching(pairs * z / groups) + 1;
  g1 = first_reaching(pairs * (z + 1) / groups) + 1;
}

template <int CFG>
__global__ __launch_bounds__(64 * Int8Cfg<CFG>::WM * Int8Cfg<CFG>::WN, 1) void k_gemm_int8(
    const int8_t *__restrict__ Apk, const int8_t *__restrict__ Bpk, int64_t mbp, int64_t nbp, int64_t kbp,
    int kb_chunk, int D, int m, int n, int32_t *__restrict__ S, int64_t plane) {
  __shared__ __attribute__((aligned(16))) int8_t lds[Int8Cfg<CFG>::NS * int8_stage_bytes<CFG>()];
  constexpr int TB = Int8Cfg<CFG>::TB;
  int tm, tn;
  int8_tile_coords(blockIdx.x, gridDim.x, (int)(mbp / TB), (int)(nbp / TB), tm, tn);
  const int chunk = blockIdx.y, nchunks = gridDim.y;
  const int64_t kb0 = (int64_t)chunk * kb_chunk;
  const int64_t kb1 = kb0 + kb_chunk < kbp ? kb0 + kb_chunk : kbp;
  constexpr int KSB = Int8Cfg<CFG>::KSB;
  const int nks = (int)ceil_div(kb1 - kb0, KSB), last = (int)(kb1 - kb0) - (nks - 1) * KSB;
  // diagonal group blockIdx.z of gridDim.z
  int g0, g1;
  diagonal_group(D, blockIdx.z, gridDim.z, g0, g1);
  const SumsWork work{g0, g1, S, plane, mbp, chunk, nchunks};
  gemm_int8_tile<CFG>(work, Apk, Bpk, mbp, nbp, kbp, kb0, nks, last, m, n, tm, tn, 0, lds);
}

// Diagonal-sum planes are blocked: the 32 x 32 block (bi, bj) of C holds, for
// lane l and accumulator r of the 32x32x32 instruction, element
// (32 bi + l % 32, 32 bj + 8 (r / 4) + 4 (l / 32) + r % 4) at
// ((bj * mbp + bi) * 64 + l) * 16 + r.  A combine thread takes four
// consecutive r of one (block, lane): one 16-byte load per diagonal and chunk.
//
// Consecutive diagonals differ in weight by 2^7, so a run of L of them is
// summed exactly in a 64-bit integer, T = sum_j S_(g0 + j) 2^(7 (L - 1 - j)),
// at the weight of its last diagonal, and enters the accumulator as the two
// binary64 values hi = RN(T) and lo = T - hi (exact: |lo| < 2^9 while
// |T| < 2^62).  With digits of at most 64 in magnitude, |S_g| <= g K 2^12 <=
// D K 2^12 (K the padded k); for 2^B >= D K 2^12, |T| < 2^(B + 7 (L - 1) + 1),
// so L = 1 + (61 - B) / 7 keeps |T| below 2^62 (L = 5 for QD at k = 4096).
// Two accumulator additions per run instead of one per diagonal: the combine
// is bound by its binary64 additions, not by its loads.
__host__ __device__ inline int combine_run(int D, int64_t kbp) {
  int64_t x = (int64_t)(D > 0 ? D : 1) * (kbp > 0 ? kbp : 1) * kKBlk8;  // D K
  int b = 12;
  while (x > 1) {  // b = 12 + ceil(log2(D K))
    x = (x + 1) / 2;
    ++b;
  }
  return b <= 61 ? 1 + (61 - b) / 7 : 1;
}

// Combine thread t (0 <= t < mbp * nbp * 256) of one product: four
// consecutive accumulator entries r of one (block, lane).
template <int C>
__device__ __forceinline__ void combine_one(int64_t t, const int32_t *__restrict__ S, int64_t plane, int nchunks,
                                            int D, int run, const int *__restrict__ EA, const int *__restrict__ EB,
                                            int64_t mbp, int m, int n, double *__restrict__ Cout, int ldc,
                                            int64_t c_stride, int debug_g, int64_t *__restrict__ Sdbg, int lddbg) {
  const int q = (int)(t % 4);
  const int lane = (int)((t / 4) % 64);
  const int64_t blk = t / 256;
  const int64_t bi = blk % mbp, bj = blk / mbp;
  const int i = (int)(bi * 32 + lane % 32);
  const int j0 = (int)(bj * 32 + 8 * q + 4 * (lane / 32));
  if (i >= m || j0 >= n) return;
  const int64_t off = (blk * 64 + lane) * 16 + 4 * q;
  const int Ei = EA[i];
  double acc[4][C + 1];
  int Fj[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    Fj[e] = j0 + e < n ? EB[j0 + e] : kZeroExp;
#pragma unroll
    for (int c = 0; c <= C; ++c) acc[e][c] = 0.0;
  }
  for (int g0 = 1; g0 <= D; g0 += run) {
    const int g1 = g0 + run <= D + 1 ? g0 + run : D + 1;  // diagonals g0 .. g1 - 1
    int64_t T[4] = {0, 0, 0, 0};
    for (int g = g0; g < g1; ++g) {
      int64_t s[4] = {0, 0, 0, 0};
      for (int c = 0; c < nchunks; ++c) {
        const i4v v = *reinterpret_cast<const i4v *>(S + ((int64_t)(g - 1) * nchunks + c) * plane + off);
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] += v[e];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (debug_g == g && j0 + e < n) Sdbg[i + (int64_t)(j0 + e) * lddbg] = s[e];
        T[e] = T[e] * 128 + s[e];
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (j0 + e >= n || Ei == kZeroExp || Fj[e] == kZeroExp || T[e] == 0) continue;
      const double hi = (double)T[e];
      const double lo = (double)(T[e] - (int64_t)hi);
      const int w = Ei + Fj[e] + 2 - 7 * g1;  // the weight of diagonal g1 - 1
      acc_add<double, C + 1>(acc[e], ldexp(hi, w));
      acc_add<double, C + 1>(acc[e], ldexp(lo, w));
    }
  }
  if (debug_g > 0) return;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (j0 + e >= n) continue;
    renorm<double, C + 1>(acc[e]);
#pragma unroll
    for (int c = 0; c < C; ++c) Cout[c * c_stride + i + (int64_t)(j0 + e) * ldc] = acc[e][c];
  }
}

template <int C>
__global__ __launch_bounds__(256) void k_int8_combine(const int32_t *__restrict__ S, int64_t plane, int nchunks, int D,
                                                      int run, const int *__restrict__ EA, const int *__restrict__ EB,
                                                      int64_t mbp, int64_t nbp, int m, int n,
                                                      double *__restrict__ Cout, int ldc, int64_t c_stride,
                                                      int debug_g, int64_t *__restrict__ Sdbg, int lddbg) {
  const int64_t total = mbp * nbp * 64 * 4;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x)
    combine_one<C>(t, S, plane, nchunks, D, run, EA, EB, mbp, m, n, Cout, ldc, c_stride, debug_g, Sdbg, lddbg);
}

}  // namespace

// Longest k chunk (in 32-wide k blocks, a multiple of the k step) whose
// diagonal sums stay within 32 bits: D * k_chunk * 64 * 64 < 2^31.
int int8_kblocks_per_chunk(int D) {
  int64_t kc = ((int64_t(1) << 31) - 1) / (int64_t(4096) * (D > 0 ? D : 1));
  int64_t blocks = kc / (kKBlk8 * kKStepBlocks8) * kKStepBlocks8;
  return (int)(blocks > kKStepBlocks8 ? blocks : kKStepBlocks8);
}

// Tile configuration for an m x n product (cfg > 0 forces one): the 256 x 256
// tiles unless padding to them more than doubles the padded area of 128 x 128
// tiles.  Small grids are filled by spreading the diagonals over the grid, and
// the larger tile ran 1.6 to 2 times faster from n = 1024 up
// (DD and QD at n = 1024, 2048, 3072).
int int8_tile_config(int64_t m, int64_t n, int cfg) {
  if (cfg >= 1 && cfg <= 4) return cfg;
  const int64_t area3 = ceil_div(m, 256) * ceil_div(n, 256) * 4, area1 = ceil_div(m, 128) * ceil_div(n, 128);
  return area3 <= 2 * area1 ? 3 : 1;
}

template <int C>
hipError_t launch_gemm_int8(const void *Apk, const void *Bpk, const int *EA, const int *EB, int32_t *Sws, int64_t mbp,
                            int64_t nbp, int64_t kbp, int m, int n, int D, double *Cout, int ldc, int64_t c_stride,
                            int debug_g, int64_t *Sdbg, int lddbg, int cfg, hipStream_t st) {
  if (mbp <= 0 || nbp <= 0 || m <= 0 || n <= 0) return hipSuccess;
  const int kbc = int8_kblocks_per_chunk(D);
  const int nchunks = (int)ceil_div(kbp, kbc);
  const int64_t plane = mbp * nbp * 1024;  // blocked, padded diagonal-sum plane
  const auto *a = static_cast<const int8_t *>(Apk);
  const auto *b = static_cast<const int8_t *>(Bpk);
  const int use = int8_tile_config(m, n, cfg);
  const int tb = int8_tile_blocks(use);
  if (mbp % tb != 0 || nbp % tb != 0) return hipErrorInvalidValue;  // slices padded for another tile
  // small products: diagonals (independent sums, each with its own plane) spread
  // over gridDim.z so the grid still fills the chip (256 workgroups of the
  // 256 x 256 configuration, 512 of the smaller ones)
  const int64_t wgs = (mbp / tb) * (nbp / tb) * nchunks;
  const int64_t want = use >= 3 ? 256 : 512;
  const int groups = wgs >= want ? 1 : (int)std::min<int64_t>(D, ceil_div(want, wgs));
  if (use == 2) {
    const int64_t tiles = (mbp / 8) * (nbp / 8);
    hipLaunchKernelGGL((k_gemm_int8<2>), dim3((unsigned)tiles, (unsigned)nchunks, (unsigned)groups), dim3(64 * Int8Cfg<2>::WM * Int8Cfg<2>::WN), 0, st, a, b, mbp, nbp,
                       kbp, kbc, D, m, n, Sws, plane);
  } else if (use == 4) {
    const int64_t tiles = (mbp / 8) * (nbp / 8);
    hipLaunchKernelGGL((k_gemm_int8<4>), dim3((unsigned)tiles, (unsigned)nchunks, (unsigned)groups), dim3(64 * Int8Cfg<4>::WM * Int8Cfg<4>::WN), 0, st,
                       a, b, mbp, nbp, kbp, kbc, D, m, n, Sws, plane);
  } else if (use == 3) {
    const int64_t tiles = (mbp / 8) * (nbp / 8);
    hipLaunchKernelGGL((k_gemm_int8<3>), dim3((unsigned)tiles, (unsigned)nchunks, (unsigned)groups), dim3(64 * Int8Cfg<3>::WM * Int8Cfg<3>::WN), 0, st, a, b, mbp, nbp,
                       kbp, kbc, D, m, n, Sws, plane);
  } else {
    const int64_t tiles = (mbp / 4) * (nbp / 4);
    hipLaunchKernelGGL((k_gemm_int8<1>), dim3((unsigned)tiles, (unsigned)nchunks, (unsigned)groups), dim3(64 * Int8Cfg<1>::WM * Int8Cfg<1>::WN), 0, st, a, b, mbp, nbp,
                       kbp, kbc, D, m, n, Sws, plane);
  }
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  const int64_t blocks = ceil_div(mbp * nbp * 256, 256);
  hipLaunchKernelGGL((k_int8_combine<C>), dim3((unsigned)(blocks < 65536 ? blocks : 65536)), dim3(256), 0, st, Sws,
                     plane, nchunks, D, combine_run(D, kbp), EA, EB, mbp, nbp, m, n, Cout, ldc, c_stride, debug_g,
                     Sdbg, lddbg);
  return hipGetLastError();
}

#define MP_INT8_INST(C)                                                                                     \
  template hipError_t launch_gemm_int8<C>(const void *, const void *, const int *, const int *, int32_t *, int64_t, \
                                          int64_t, int64_t, int, int, int, double *, int, int64_t, int, int64_t *, \
                                          int, int, hipStream_t);
MP_INT8_INST(2)
MP_INT8_INST(3)
MP_INT8_INST(4)
MP_INT8_INST(5)
MP_INT8_INST(6)
MP_INT8_INST(7)
MP_INT8_INST(8)
MP_INT8_INST(9)
MP_INT8_INST(10)
MP_INT8_INST(11)
MP_INT8_INST(12)
MP_INT8_INST(13)
MP_INT8_INST(14)
#undef MP_INT8_INST

}  // namespace mp
