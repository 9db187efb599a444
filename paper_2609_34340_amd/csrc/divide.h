// 64-bit quotients without an integer division, which the compiler expands to
// some 150 dependent instructions.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace vp {

// floor(x / d) for 0 <= x < 2^53 and 1 <= d < 2^53, without a 64-bit
// integer division: the correctly rounded double quotient is within one of
// it (below 2^52), and one step against the integer remainder makes it
// exact.  Callers that cannot bound x check q * d against x.
__host__ __device__ inline int64_t fdiv53(int64_t x, int64_t d) {
  int64_t q = (int64_t)((double)x / (double)d);
  const int64_t r = x - q * d;
  if (r < 0)
    --q;
  else if (r >= d)
    ++q;
  return q;
}

// x / d for any x and d >= 1 (rounded towards zero, as x / d is): values
// outside fdiv53's range take the integer division.
__device__ inline int64_t exact_div(int64_t x, int64_t d) {
  if (x < 0 || x >= (int64_t(1) << 52) || d >= (int64_t(1) << 52)) return x / d;
  return fdiv53(x, d);
}

}  // namespace vp
