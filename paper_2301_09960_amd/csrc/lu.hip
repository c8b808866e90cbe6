// Blocked LU factorization of a DD or TD matrix with the Schur updates done by
// the slice-product GEMM (Section 4.6), and the triangular solves that use it.
//
// For a block width K the algorithm of Section 4.6 repeats, on the trailing
// matrix: factor the K x K diagonal block A11 = L11 U11; turn A12 into
// U12 = L11^-1 A12 and A21 into L21 = A21 U11^-1; update A22 := A22 - L21 U12,
// the product formed by the GEMM of this library.  No pivoting, as in the
// paper.  L (unit lower, without its diagonal) and U overwrite A.
//
// A matrix is c planes of components, each column-major with leading dimension
// ld, plane r `r * plane` elements after the first.  Everything here is DD
// (dd.h) or TD (mc.h) arithmetic in a fixed order, so a factorization is
// reproducible.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "dd.h"
#include "internal.h"
#include "layout.h"
#include "mc.h"

namespace mp {
namespace {

// The scalar operations, for DD (dd.h) and TD (mc.h) values.
__device__ __forceinline__ dd nadd(dd a, dd b) { return dd_add(a, b); }
__device__ __forceinline__ dd nsub(dd a, dd b) { return dd_sub(a, b); }
__device__ __forceinline__ dd nmul(dd a, dd b) { return dd_mul(a, b); }
__device__ __forceinline__ dd ndiv(dd a, dd b) { return dd_div(a, b); }
__device__ __forceinline__ dd nfms(dd s, dd a, dd b) { return dd_sub(s, dd_mul(a, b)); }
using td = mc<3>;
__device__ __forceinline__ td nadd(const td &a, const td &b) { return mc_add<3>(a, b); }
__device__ __forceinline__ td nsub(const td &a, const td &b) { return mc_sub<3>(a, b); }
__device__ __forceinline__ td nmul(const td &a, const td &b) { return mc_mul<3>(a, b); }
__device__ __forceinline__ td ndiv(const td &a, const td &b) { return mc_div<3>(a, b); }
// s - a b (TD: one renormalization of 8 terms)
__device__ __forceinline__ td nfms(const td &s, const td &a, const td &b) { return mc_fms<3>(s, a, b); }
// 1 / b, by the division above: a solve multiplies by it so that the division
// leaves the chain of dependent steps.
__device__ __forceinline__ dd ninv(dd b) { return dd_div(dd{1.0, 0.0}, b); }
__device__ __forceinline__ td ninv(const td &b) { return mc_div<3>(td{{1.0, 0.0, 0.0}}, b); }

template <typename Num>
struct Comps;
template <>
struct Comps<dd> {
  static constexpr int C = 2;
  __device__ static double get(const dd &v, int r) { return r == 0 ? v.hi : v.lo; }
  __device__ static void set(dd &v, int r, double x) { (r == 0 ? v.hi : v.lo) = x; }
};
template <>
struct Comps<td> {
  static constexpr int C = 3;
  __device__ static double get(const td &v, int r) { return v.x[r]; }
  __device__ static void set(td &v, int r, double x) { v.x[r] = x; }
};

template <typename Num>
__device__ __forceinline__ Num nzero() {
  Num v;
#pragma unroll
  for (int r = 0; r < Comps<Num>::C; ++r) Comps<Num>::set(v, r, 0.0);
  return v;
}

// A c-component vector stored as planes of n (x[r * n + i]).
template <typename Num>
__device__ __forceinline__ Num vget(const double *x, int n, int i) {
  Num v;
#pragma unroll
  for (int r = 0; r < Comps<Num>::C; ++r) Comps<Num>::set(v, r, x[(int64_t)r * n + i]);
  return v;
}
template <typename Num>
__device__ __forceinline__ void vput(double *x, int n, int i, const Num &v) {
#pragma unroll
  for (int r = 0; r < Comps<Num>::C; ++r) x[(int64_t)r * n + i] = Comps<Num>::get(v, r);
}

template <typename Num>
struct Mat {
  double *p;
  int64_t ld, plane;
  __device__ __forceinline__ Num get(int64_t i, int64_t j) const {
    Num v;
#pragma unroll
    for (int r = 0; r < Comps<Num>::C; ++r) Comps<Num>::set(v, r, p[r * plane + i + j * ld]);
    return v;
  }
  __device__ __forceinline__ void put(int64_t i, int64_t j, const Num &v) const {
#pragma unroll
    for (int r = 0; r < Comps<Num>::C; ++r) p[r * plane + i + j * ld] = Comps<Num>::get(v, r);
  }
};

constexpr int kLuThreads = 1024;

// The value of lane `src` (the same for the whole wavefront) in all lanes.
template <typename Num>
__device__ __forceinline__ Num read_num(const Num &v, int src) {
  Num o;
#pragma unroll
  for (int r = 0; r < Comps<Num>::C; ++r) {
    const long long x = __double_as_longlong(Comps<Num>::get(v, r));
    const int lo = __builtin_amdgcn_readlane((int)x, src), hi = __builtin_amdgcn_readlane((int)(x >> 32), src);
    Comps<Num>::set(o, r, __longlong_as_double(((long long)hi << 32) | (unsigned)lo));
  }
  return o;
}

// Unblocked LU of the K x K block at (j0, j0), K <= kDiagLds, in one workgroup, a
// thread per entry: for each column, divide below the pivot, then the rank-1 update
// of the rest.  Bound by the chain of the pivots: update, division, hand over.  A
// step passes on its column of L, its row of U and the diagonal entry after it
// through LDS, and the threads of the next column form the next pivot themselves,
// so a step has one barrier; with the block in LDS and two barriers a block of 32
// took 25 us (DD), now 22: 0.55 us a step, of it some 0.3 the division.
constexpr int kDiagLds = 32;

template <typename Num>
__global__ __launch_bounds__(kLuThreads) void k_lu_diag(Mat<Num> A, int j0, int K) {
  static_assert(kDiagLds * kDiagLds == kLuThreads, "a thread per entry");
  __shared__ Num below[2][kDiagLds], right[2][kDiagLds], diag[2];
  const int i = threadIdx.x % kDiagLds, l = threadIdx.x / kDiagLds;
  const bool inside = i < K && l < K;
  Num a = inside ? A.get(j0 + i, j0 + l) : nzero<Num>();
  if (threadIdx.x == 0) diag[1] = a;
  __syncthreads();
  if (inside) {
    if (l == 0 && i > 0) {
      a = ndiv(a, diag[1]);
      below[0][i] = a;
    }
    if (i == 0) right[0][l] = a;
    if (i == 1 && l == 1) diag[0] = a;
  }
  __syncthreads();
  for (int j = 0; j < K - 1; ++j) {
    const int now = j & 1, then = now ^ 1;
    if (inside && i > j && l > j) {
      a = nfms(a, below[now][i], right[now][l]);
      if (l == j + 1 && i > j + 1) {
        a = ndiv(a, nfms(diag[now], below[now][j + 1], right[now][j + 1]));
        below[then][i] = a;
      }
      if (i == j + 1) right[then][l] = a;
      if (i == j + 2 && l == j + 2) diag[then] = a;
    }
    __syncthreads();
  }
  if (inside) A.put(j0 + i, j0 + l, a);
}

// U12 = L11^-1 A12 in place: thread per column l of A12, forward substitution
// down the column with the unit lower L11.
template <typename Num>
__global__ __launch_bounds__(256) void k_trsm_lower(Mat<Num> A, int j0, int K, int n) {
  const int l = j0 + K + blockIdx.x * 256 + threadIdx.x;
  if (l >= n) return;
  for (int i = 1; i < K; ++i) {
    Num s = A.get(j0 + i, l);
    for (int q = 0; q < i; ++q) s = nfms(s, A.get(j0 + i, j0 + q), A.get(j0 + q, l));
    A.put(j0 + i, l, s);
  }
}

// L21 = A21 U11^-1 in place: thread per row i of A21, solving x U11 = a left to
// right; x_q is the remaining sum times the reciprocal of u_qq.
template <typename Num>
__global__ __launch_bounds__(256) void k_trsm_upper(Mat<Num> A, int j0, int K, int n) {
  const int i = j0 + K + blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  for (int q = 0; q < K; ++q) {
    Num s = A.get(i, j0 + q);
    for (int r = 0; r < q; ++r) s = nfms(s, A.get(i, j0 + r), A.get(j0 + r, j0 + q));
    A.put(i, j0 + q, nmul(s, ninv(A.get(j0 + q, j0 + q))));
  }
}

// Both solves for K <= kSweepMax, one wavefront per column of A12 or row of A21:
// its entries lie in registers (entry t in lane t % 64, E of them per lane), and
// at step q the lanes update the entries after q with x_q, which is read from its
// lane.  Every entry receives the same operations in the same order as in the
// kernels above (the subtractions for q = 0, 1, ... and then, for U, the product
// with 1 / u_qq), so the results are identical; the chain per wavefront is K steps
// instead of K^2 / 2, and the reciprocals of U's diagonal are formed before it, all
// at once.
//
// Bound by that chain (product, subtraction and, for U, the product with the
// reciprocal: some 30 dependent binary64 operations a step).  The multipliers of
// Q steps go through LDS, read along memory for L and for U and one chunk ahead:
// read by each step for itself they cost an L2 round trip a step, for U a cache
// line per lane.  DD, n = 2048, K = 128: 66 + 85 us a panel on average in two
// launches, now 69 in one; the widest panels (15 wavefronts a CU) are bound by the
// binary64 rate instead.
constexpr int kSweepMax = 512;
constexpr int kSweepWaves = 4;

template <typename F, int... I>
__device__ __forceinline__ void each(F &f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}

template <typename Num, int E>
__global__ __launch_bounds__(64 * kSweepWaves) void k_panel_sweep(Mat<Num> A, int j0, int K, int n, int lower_blocks) {
  constexpr int C = Comps<Num>::C, Q = E <= 2 ? 16 : 32 / E, N = Q * E / kSweepWaves;
  __shared__ double mul[C][Q][64 * E + 1];
  __shared__ Num inv[64 * E];
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64), lane = threadIdx.x % 64;
  const bool upper = (int)blockIdx.x >= lower_blocks;
  const int vec = j0 + K + ((int)blockIdx.x - (upper ? lower_blocks : 0)) * kSweepWaves + w;
  const bool live = vec < n;
  Num x[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int t = 64 * e + lane;
    x[e] = !live || t >= K ? nzero<Num>() : upper ? A.get(vec, j0 + t) : A.get(j0 + t, vec);
  }
  Num ahead[N];  // the next chunk's multipliers, of step q for entry t
  auto place = [&](int s, int &q, int &t) {
    const int idx = (int)threadIdx.x + 64 * kSweepWaves * s;
    q = upper ? idx % Q : idx / (64 * E);
    t = upper ? idx / Q : idx % (64 * E);
  };
  auto load = [&](int q0) {
#pragma unroll
    for (int s = 0; s < N; ++s) {
      int q, t;
      place(s, q, t);
      q += q0;
      ahead[s] = q >= K || t >= K ? nzero<Num>() : upper ? A.get(j0 + q, j0 + t) : A.get(j0 + t, j0 + q);
    }
  };
  load(0);
  if (upper)
    for (int t = threadIdx.x; t < K; t += 64 * kSweepWaves) inv[t] = ninv(A.get(j0 + t, j0 + t));
  auto sweep = [&](auto of) {  // the steps whose x_q lie in register e
    constexpr int e = decltype(of)::value;
    for (int first = 0; first < 64 && 64 * e + first < K; first += Q) {
      const int q0 = 64 * e + first, steps = K - q0 < Q ? K - q0 : Q;
      __syncthreads();
#pragma unroll
      for (int s = 0; s < N; ++s) {
        int q, t;
        place(s, q, t);
#pragma unroll
        for (int r = 0; r < C; ++r) mul[r][q][t] = Comps<Num>::get(ahead[s], r);
      }
      __syncthreads();
      if (q0 + Q < K) load(q0 + Q);
      for (int part = 0; part < steps; part += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int q = part + u;
          if (q >= steps) break;
          Num f[E];
#pragma unroll
          for (int d = e; d < E; ++d)
#pragma unroll
            for (int r = 0; r < C; ++r) Comps<Num>::set(f[d], r, mul[r][q][64 * d + lane]);
          Num xq = read_num(x[e], first + q);
          if (upper) {
            xq = nmul(xq, inv[q0 + q]);
            if (lane == first + q) x[e] = xq;
            if (lane > first + q) x[e] = nfms(x[e], xq, f[e]);
#pragma unroll
            for (int d = e + 1; d < E; ++d) x[d] = nfms(x[d], xq, f[d]);
          } else {
            if (lane > first + q) x[e] = nfms(x[e], f[e], xq);
#pragma unroll
            for (int d = e + 1; d < E; ++d) x[d] = nfms(x[d], f[d], xq);
          }
        }
      }
    }
  };
  each(sweep, std::make_integer_sequence<int, E>{});
  if (!live) return;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int t = 64 * e + lane;
    if (t >= K) continue;
    if (upper)
      A.put(vec, j0 + t, x[e]);
    else
      A.put(j0 + t, vec, x[e]);
  }
}

// Both panel sweeps for a K x K diagonal block at (j0, j0), rows and columns up
// to `end`.
template <typename Num>
void launch_sweeps(const Mat<Num> &M, int j0, int K, int end, hipStream_t st) {
  const int blocks = (int)ceil_div(end - j0 - K, kSweepWaves);
  const dim3 grid((unsigned)(2 * blocks)), wg(64 * kSweepWaves);
  if (K <= 64)
    hipLaunchKernelGGL((k_panel_sweep<Num, 1>), grid, wg, 0, st, M, j0, K, end, blocks);
  else if (K <= 128)
    hipLaunchKernelGGL((k_panel_sweep<Num, 2>), grid, wg, 0, st, M, j0, K, end, blocks);
  else if (K <= 256)
    hipLaunchKernelGGL((k_panel_sweep<Num, 4>), grid, wg, 0, st, M, j0, K, end, blocks);
  else
    hipLaunchKernelGGL((k_panel_sweep<Num, 8>), grid, wg, 0, st, M, j0, K, end, blocks);
}

// Diagonal blocks wider than kInner are factored in inner blocks of kInner (see
// lu_panel).
constexpr int kInner = 32;

// A[r0 + i, c0 + l] -= sum over q in [q0, q0 + kb) of A[r0 + i, q] A[q, c0 + l]
// (q ascending, kb <= kInner), thread per entry: the trailing update inside a
// diagonal block factored in inner blocks.  Bound by latency (at most a few dozen
// workgroups): the operands come in one round of loads and the chain reads them
// from LDS; read from memory along the chain the update took 13.2 us (DD, K = 128,
// on average), now 5.3.
constexpr int kRankTile = 16;

template <typename Num>
__global__ __launch_bounds__(kRankTile *kRankTile) void k_rank_update(Mat<Num> A, int r0, int c0, int rows, int cols,
                                                                      int q0, int kb) {
  __shared__ Num left[kInner][kRankTile], top[kRankTile][kInner + 1];
  const int i0 = r0 + (int)blockIdx.x * kRankTile, l0 = c0 + (int)blockIdx.y * kRankTile;
  const int t = threadIdx.x, i = i0 + t % kRankTile, l = l0 + t / kRankTile;
  const bool inside = i < r0 + rows && l < c0 + cols;
  Num s = inside ? A.get(i, l) : nzero<Num>();
#pragma unroll
  for (int idx = t; idx < kInner * kRankTile; idx += kRankTile * kRankTile) {
    const int row = i0 + idx % kRankTile, ql = idx / kRankTile;
    left[ql][idx % kRankTile] = row < r0 + rows && ql < kb ? A.get(row, q0 + ql) : nzero<Num>();
    const int qt = idx % kInner, col = l0 + idx / kInner;
    top[idx / kInner][qt] = col < c0 + cols && qt < kb ? A.get(q0 + qt, col) : nzero<Num>();
  }
  __syncthreads();
#pragma unroll 4
  for (int q = 0; q < kb; ++q) s = nfms(s, left[q][t % kRankTile], top[t / kRankTile][q]);
  if (inside) A.put(i, l, s);
}

// out = A[r0 .. r0 + rows, c0 .. c0 + cols) as a contiguous DD matrix
// (leading dimension rows, lo plane rows * cols later).
template <typename Num>
__global__ __launch_bounds__(256) void k_copy_block(Mat<Num> A, int r0, int c0, int rows, int cols, double *out) {
  const int64_t total = (int64_t)rows * cols;
  for (int64_t idx = blockIdx.x * 256 + threadIdx.x; idx < total; idx += (int64_t)gridDim.x * 256) {
    const int i = (int)(idx % rows), j = (int)(idx / rows);
    const Num v = A.get(r0 + i, c0 + j);
#pragma unroll
    for (int r = 0; r < Comps<Num>::C; ++r) out[r * total + idx] = Comps<Num>::get(v, r);
  }
}

// A[r0 + i, c0 + j] -= P[i, j] (P contiguous as written by the GEMM).
template <typename Num>
__global__ __launch_bounds__(256) void k_sub_block(Mat<Num> A, int r0, int c0, int rows, int cols, const double *P) {
  const int64_t total = (int64_t)rows * cols;
  for (int64_t idx = blockIdx.x * 256 + threadIdx.x; idx < total; idx += (int64_t)gridDim.x * 256) {
    const int i = (int)(idx % rows), j = (int)(idx / rows);
    Num p;
#pragma unroll
    for (int r = 0; r < Comps<Num>::C; ++r) Comps<Num>::set(p, r, P[r * total + idx]);
    A.put(r0 + i, c0 + j, nsub(A.get(r0 + i, c0 + j), p));
  }
}

// Blocked solve of L U x = b (x holds b on entry): blocks of kSolveB rows.
// Forward: one wavefront solves the block's rows against the unit lower
// diagonal block (lane per row, x_q read from its lane), then every later row
// subtracts the block's contribution (k_solve_update).  Backward: the same
// from the last block up, with the product by the reciprocal of U's diagonal
// entry (each lane forms its own before the chain).  Every entry's operations
// come in a fixed order, so the solve is reproducible.
constexpr int kSolveB = 64;

// The diagonal blocks' multipliers are read kSolveAhead steps at a time and as many
// ahead: read by each step for itself, a step waited on the L2 (25 us a block of 64
// in DD, now 12 and 14).
constexpr int kSolveAhead = 8;

template <typename Num>
__global__ __launch_bounds__(64) void k_solve_fwd_diag(Mat<Num> A, int n, double *x, int b0, int B) {
  const int lane = threadIdx.x, i = b0 + lane;
  Num xi = lane < B ? vget<Num>(x, n, i) : nzero<Num>();
  Num f[kSolveAhead], next[kSolveAhead];
  auto load = [&](Num(&to)[kSolveAhead], int q0) {
#pragma unroll
    for (int d = 0; d < kSolveAhead; ++d) to[d] = lane < B && q0 + d < B ? A.get(i, b0 + q0 + d) : nzero<Num>();
  };
  load(next, 0);
  for (int q0 = 0; q0 < B; q0 += kSolveAhead) {
#pragma unroll
    for (int d = 0; d < kSolveAhead; ++d) f[d] = next[d];
    load(next, q0 + kSolveAhead);
#pragma unroll
    for (int d = 0; d < kSolveAhead; ++d) {
      const int q = q0 + d;
      if (q >= B - 1) break;
      const Num xq = read_num(xi, q);
      if (lane > q && lane < B) xi = nfms(xi, f[d], xq);
    }
  }
  if (lane < B) vput<Num>(x, n, i, xi);
}

template <typename Num>
__global__ __launch_bounds__(64) void k_solve_bwd_diag(Mat<Num> A, int n, double *x, int b0, int B) {
  const int lane = threadIdx.x, i = b0 + lane;
  Num xi = lane < B ? vget<Num>(x, n, i) : nzero<Num>();
  Num inv = nzero<Num>();
  Num f[kSolveAhead], next[kSolveAhead];
  auto load = [&](Num(&to)[kSolveAhead], int q0) {
#pragma unroll
    for (int d = 0; d < kSolveAhead; ++d) to[d] = lane < B && q0 - d >= 0 ? A.get(i, b0 + q0 - d) : nzero<Num>();
  };
  load(next, B - 1);
  if (lane < B) inv = ninv(A.get(i, i));
  for (int q0 = B - 1; q0 >= 0; q0 -= kSolveAhead) {
#pragma unroll
    for (int d = 0; d < kSolveAhead; ++d) f[d] = next[d];
    load(next, q0 - kSolveAhead);
#pragma unroll
    for (int d = 0; d < kSolveAhead; ++d) {
      const int q = q0 - d;
      if (q < 0) break;
      if (lane == q) xi = nmul(xi, inv);
      const Num xq = read_num(xi, q);
      if (lane < q) xi = nfms(xi, f[d], xq);
    }
  }
  if (lane < B) vput<Num>(x, n, i, xi);
}

// x_i -= sum over q in [b0, b0 + B) of A(i, q) x_q for the rows i in
// [r0, r0 + rows): the sum in kSolveChunks runs of consecutive q, one thread
// each (32 rows per workgroup), then added to x_i in run order.
constexpr int kSolveChunks = 8;
constexpr int kSolveRows = 256 / kSolveChunks;

template <typename Num>
__global__ __launch_bounds__(256) void k_solve_update(Mat<Num> A, int n, double *x, int b0, int B, int r0,
                                                      int rows) {
  __shared__ Num part[kSolveChunks][kSolveRows];
  const int rl = threadIdx.x % kSolveRows, c = threadIdx.x / kSolveRows;
  const int i = r0 + blockIdx.x * kSolveRows + rl;
  const bool live = i < r0 + rows;
  const int per = (B + kSolveChunks - 1) / kSolveChunks;
  const int q0 = b0 + c * per, q1 = std::min(b0 + B, q0 + per);
  Num p = nzero<Num>();  // minus the run's sum
  if (live) {
#pragma unroll 8
    for (int q = q0; q < q1; ++q) p = nfms(p, A.get(i, q), vget<Num>(x, n, q));
  }
  part[c][rl] = p;
  __syncthreads();
  if (live && c == 0) {
    Num s = vget<Num>(x, n, i);
#pragma unroll
    for (int r = 0; r < kSolveChunks; ++r) s = nadd(s, part[r][rl]);
    vput<Num>(x, n, i, s);
  }
}

unsigned grid_for(int64_t work) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>(ceil_div(work, 256), 8192)); }

// Diagonal blocks wider than kInner are factored in inner blocks of kInner:
// the unblocked kernel on the inner diagonal block, the two panel
// solves restricted to the diagonal block, and a rank-kInner update of its
// rest (DD at n = 2048: K = 512 170 -> 13.6 ms, and K = 64 12.0 -> 10.7 ms
// once blocks of up to kInner were held in LDS).
template <typename Num>
hipError_t lu_panel(double *A, int64_t ld, int64_t plane, int j0, int K, int n, hipStream_t st) {
  const Mat<Num> M{A, ld, plane};
  static_assert(kInner <= kDiagLds, "an inner block fits the unblocked kernel");
  if (K <= kInner) {
    hipLaunchKernelGGL((k_lu_diag<Num>), dim3(1), dim3(kLuThreads), 0, st, M, j0, K);
  } else {
    const int end = j0 + K;
    for (int jj = j0; jj < end; jj += kInner) {
      const int kb = std::min(kInner, end - jj), r = end - jj - kb;
      hipLaunchKernelGGL((k_lu_diag<Num>), dim3(1), dim3(kLuThreads), 0, st, M, jj, kb);
      if (r == 0) break;
      launch_sweeps<Num>(M, jj, kb, end, st);
      const unsigned tiles = (unsigned)ceil_div(r, kRankTile);
      hipLaunchKernelGGL((k_rank_update<Num>), dim3(tiles, tiles), dim3(kRankTile * kRankTile), 0, st, M, jj + kb,
                         jj + kb, r, r, jj, kb);
    }
  }
  if (j0 + K < n && K <= kSweepMax) {
    launch_sweeps<Num>(M, j0, K, n, st);
  } else if (j0 + K < n) {
    hipLaunchKernelGGL((k_trsm_lower<Num>), dim3((unsigned)ceil_div(n - j0 - K, 256)), dim3(256), 0, st, M, j0, K,
                       n);
    hipLaunchKernelGGL((k_trsm_upper<Num>), dim3((unsigned)ceil_div(n - j0 - K, 256)), dim3(256), 0, st, M, j0, K,
                       n);
  }
  return hipGetLastError();
}

template <typename Num>
hipError_t lu_solve(const double *A, int64_t ld, int64_t plane, int n, double *x, hipStream_t st) {
  const Mat<Num> M{const_cast<double *>(A), ld, plane};
  for (int b0 = 0; b0 < n; b0 += kSolveB) {
    const int B = std::min(kSolveB, n - b0);
    hipLaunchKernelGGL((k_solve_fwd_diag<Num>), dim3(1), dim3(64), 0, st, M, n, x, b0, B);
    if (b0 + B < n)
      hipLaunchKernelGGL((k_solve_update<Num>), dim3((unsigned)ceil_div(n - b0 - B, kSolveRows)), dim3(256), 0, st, M,
                         n, x, b0, B, b0 + B, n - b0 - B);
  }
  for (int b0 = (n - 1) / kSolveB * kSolveB; b0 >= 0; b0 -= kSolveB) {
    const int B = std::min(kSolveB, n - b0);
    hipLaunchKernelGGL((k_solve_bwd_diag<Num>), dim3(1), dim3(64), 0, st, M, n, x, b0, B);
    if (b0 > 0)
      hipLaunchKernelGGL((k_solve_update<Num>), dim3((unsigned)ceil_div(b0, kSolveRows)), dim3(256), 0, st, M, n, x,
                         b0, B, 0, b0);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_lu_panel(int comps, double *A, int64_t ld, int64_t plane, int j0, int K, int n, hipStream_t st) {
  return comps == 2 ? lu_panel<dd>(A, ld, plane, j0, K, n, st) : lu_panel<td>(A, ld, plane, j0, K, n, st);
}

hipError_t launch_lu_copy(int comps, double *A, int64_t ld, int64_t plane, int r0, int c0, int rows, int cols,
                          double *out, hipStream_t st) {
  if (comps == 2)
    hipLaunchKernelGGL((k_copy_block<dd>), dim3(grid_for((int64_t)rows * cols)), dim3(256), 0, st,
                       Mat<dd>{A, ld, plane}, r0, c0, rows, cols, out);
  else
    hipLaunchKernelGGL((k_copy_block<td>), dim3(grid_for((int64_t)rows * cols)), dim3(256), 0, st,
                       Mat<td>{A, ld, plane}, r0, c0, rows, cols, out);
  return hipGetLastError();
}

hipError_t launch_lu_sub(int comps, double *A, int64_t ld, int64_t plane, int r0, int c0, int rows, int cols,
                         const double *P, hipStream_t st) {
  if (comps == 2)
    hipLaunchKernelGGL((k_sub_block<dd>), dim3(grid_for((int64_t)rows * cols)), dim3(256), 0, st,
                       Mat<dd>{A, ld, plane}, r0, c0, rows, cols, P);
  else
    hipLaunchKernelGGL((k_sub_block<td>), dim3(grid_for((int64_t)rows * cols)), dim3(256), 0, st,
                       Mat<td>{A, ld, plane}, r0, c0, rows, cols, P);
  return hipGetLastError();
}

hipError_t launch_lu_solve(int comps, const double *A, int64_t ld, int64_t plane, int n, double *x, hipStream_t st) {
  return comps == 2 ? lu_solve<dd>(A, ld, plane, n, x, st) : lu_solve<td>(A, ld, plane, n, x, st);
}

}  // namespace mp
