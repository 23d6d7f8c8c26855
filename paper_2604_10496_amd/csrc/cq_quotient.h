// Quotients of many values by one scale, shared by the quantizing kernels.
#ifndef CQ_QUOTIENT_H_
#define CQ_QUOTIENT_H_

#include <hip/hip_runtime.h>

// x / s from the reciprocal of s, with the remainder of the product taken into account (Markstein's division: the correctly
// rounded quotient but for the ends of the exponent range, where the division itself is kept): three operations per value
// instead of about ten.
struct cq_quotient {
  float s, inv;
  bool fast;
  __device__ __forceinline__ explicit cq_quotient(float scale) : s(scale), fast(scale > 1e-30f && scale < 1e30f) {
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
