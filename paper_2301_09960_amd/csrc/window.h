// Exact fixed-point windows of multi-component numbers: the value of an
// element as a two's complement integer of 32-bit words.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mp {

// x = M 2^q exactly, |M| < 2^53 (zero gives M = 0).
__device__ __forceinline__ void binary64_parts(double x, int64_t &M, int &q) {
  const uint64_t b = (uint64_t)__double_as_longlong(x);
  const int ef = (int)((b >> 52) & 0x7ff);
  const int64_t f = (int64_t)(b & 0xfffffffffffffULL);
  const int64_t m = ef == 0 ? f : (f | (int64_t(1) << 52));
  q = ef == 0 ? -1074 : ef - 1075;
  M = (b >> 63) ? -m : m;
}

// w += M 2^off over all NW words (two's complement; off >= 0).  With
// off = 32 q + sh, M 2^sh spans three words x0, x1, x2 (the sign beyond), and
// word i receives the one of them numbered i - q: selects, no branches.
template <int NW>
__device__ __forceinline__ void window_add(uint32_t (&w)[NW], int64_t M, int off) {
  const int q = off >> 5, sh = off & 31;
  const uint64_t u = (uint64_t)M << sh;
  const uint32_t sign = (uint32_t)(M >> 63);
  const uint32_t x0 = (uint32_t)u, x1 = (uint32_t)(u >> 32);
  const uint32_t x2 = sh ? (uint32_t)(M >> (64 - sh)) : sign;
  uint32_t carry = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const int d = i - q;
    const uint32_t part = d < 0 ? 0u : d == 0 ? x0 : d == 1 ? x1 : d == 2 ? x2 : sign;
    const uint64_t sum = (uint64_t)w[i] + part + carry;
    w[i] = (uint32_t)sum;
    carry = (uint32_t)(sum >> 32);
  }
}

}  // namespace mp
