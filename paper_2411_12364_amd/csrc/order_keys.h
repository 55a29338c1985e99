// Monotone keys of the selections' scores: plain C++, compiled for the device and the host alike.
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define UMEM_HD __host__ __device__ __forceinline__
#else
#define UMEM_HD inline
#endif

namespace umem {

// Monotone map of a float to an unsigned key: larger float -> larger key.  -0.0 maps like +0.0
// and NaN maps to 0, below every number including -inf.
UMEM_HD uint32_t order_key(float x) {
  if (x != x) return 0u;
  uint32_t u = __builtin_bit_cast(uint32_t, x);
  if ((u << 1) == 0u) u = 0u;
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// The float of a key: of a number's key that number (0.0 for either zero).
UMEM_HD float key32_value(uint32_t k) {
  return __builtin_bit_cast(float, (k >> 31) ? (k & 0x7FFFFFFFu) : ~k);
}

// Whether x >= key32_value(L) says of every float x what order_key(x) >= L says, for an L up to
// +inf's key (a k-th largest score with bits cleared).  Up to -inf's own key it does not: 0 lets NaNs
// in, and the keys in between belong to no float (key32_value gives NaNs, which nothing reaches).
UMEM_HD bool key32_is_limit(uint32_t L) { return L > 0x007FFFFFu; }

}  // namespace umem
