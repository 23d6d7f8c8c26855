// Quotients of many values by one scale, shared by the quantizing kernels.
#ifndef CQ_QUOTIENT_H_
#define CQ_QUOTIENT_H_

#include <hip/hip_runtime.h>

// x / s from the reciprocal of s, with the remainder of the product taken into account (Markstein's division): three operations
// per value instead of about ten.  It is the correctly rounded quotient where the reciprocal is correctly rounded, which one
// Newton step from an approximation within a unit in the last place gives unless the significand of s is all ones; that s,
// and the ends of the exponent range, keep the division itself.
struct cq_quotient {
  float s, inv;
  bool fast;
  __device__ __forceinline__ explicit cq_quotient(float scale)
      : s(scale), fast(scale > 1e-30f && scale < 1e30f && (__float_as_uint(scale) & 0x7fffffu) != 0x7fffffu) {
    inv = __builtin_amdgcn_rcpf(scale);
    inv = fmaf(fmaf(-scale, inv, 1.f), inv, inv);
  }
  template <bool FAST>
  __device__ __forceinline__ float get(float x) const {
    if constexpr (!FAST) return x / s;
    const float q = x * inv;
    return fmaf(fmaf(-q, s, x), inv, q);
  }
};

#endif  // CQ_QUOTIENT_H_
