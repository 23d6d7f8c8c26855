// Register-resident decoding of packed 4-bit indices (Eq. W_c): shared by the HIP kernels of libcq.
#ifndef CQ_DECODE_H_
#define CQ_DECODE_H_

#include "cq_internal.h"

__device__ __forceinline__ uint32_t cq_bf16_to_f16_bits(uint32_t b) {
  const _Float16 h = (_Float16)__uint_as_float(b << 16);
  return (uint32_t) __builtin_bit_cast(uint16_t, h);
}

// Byte tables of one row's 16 centroids, for a lookup by whole nibbles: lo[] yields the low bytes, hi[] the high ones,
//   byte of entry n  =  v_perm_b32(t[1], t[0], n) ^ v_perm_b32(t[3], t[2], n ^ 8).
// v_perm_b32 takes the bytes 0..7 of its two sources for the selectors 0..7; for 8, 9, 10 and 11 it returns eight copies of
// the sign of byte 1, 3, 5 and 7, for 12 zero and for 13..15 0xff.  So whichever half an entry is not in also contributes,
// but with a value that depends on the entry's number and the table alone, and the tables hold the entries with that value
// xored in (cq_fold_halves).  Masking the nibbles to three bits and choosing between the halves with a third permutation,
// steered by the fourth, costs 23 instructions per 8 weights, 18 of them of three operands; this way 21, 12 of three operands.
struct RowTable {
  uint32_t lo[4], hi[4];
};

// t: bytes 0..15 of a plane.  t[0] gets the signs of t[2], t[3] (selectors 8..11 of the second lookup, entries 0..3), t[2]
// those of t[0], t[1]; bytes 2 and 3 of either depend on t[3] or t[1] only, byte 1 on byte 3 and byte 0 on byte 1 of the
// other, so that the second time round finds them all.
__device__ __forceinline__ void cq_fold_halves(uint32_t (&t)[4]) {
  t[1] ^= 0xffffff00u;   // entries 5..7: selectors 13..15 of the second lookup
  t[3] ^= 0xffffff00u;   // entries 13..15: selectors 13..15 of the first
  const uint32_t first = t[0], second = t[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    t[2] = second ^ __builtin_amdgcn_perm(t[1], t[0], 0x0b0a0908u);
    t[0] = first ^ __builtin_amdgcn_perm(t[3], t[2], 0x0b0a0908u);
  }
}

// p[i] = centroid entries 2i (low half) and 2i+1 as bf16 bits
template <bool F16>
__device__ __forceinline__ RowTable make_row_table(uint32_t (&p)[8]) {
  if constexpr (F16) {
#pragma unroll
    for (int i = 0; i < 8; ++i) p[i] = cq_bf16_to_f16_bits(p[i] & 0xffffu) | (cq_bf16_to_f16_bits(p[i] >> 16) << 16);
  }
  RowTable t;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    // entries 4q..4q+3 live in p[2q] (4q, 4q+1) and p[2q+1] (4q+2, 4q+3)
    t.lo[q] = __builtin_amdgcn_perm(p[2 * q + 1], p[2 * q], 0x06040200u);
    t.hi[q] = __builtin_amdgcn_perm(p[2 * q + 1], p[2 * q], 0x07050301u);
  }
  cq_fold_halves(t.lo);
  cq_fold_halves(t.hi);
  return t;
}

template <bool F16>
__device__ __forceinline__ RowTable make_row_table(const uint16_t* crow) {
  const uint4 c0 = reinterpret_cast<const uint4*>(crow)[0];
  const uint4 c1 = reinterpret_cast<const uint4*>(crow)[1];
  uint32_t p[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
  return make_row_table<F16>(p);
}

// 8 packed indices (one dword) -> 4 dwords of 16-bit pairs.  GROUPED = false: canonical bytes (weight 2i in
// the low nibble of byte i, 2i+1 in the high one).  GROUPED = true: the prepacked arrangement (weight i in the
// low nibble of byte i, weight i+4 in the high one): the two nibble planes are then the first and the second
// four weights, and the final re-pairing of even and odd weights falls away.
template <bool GROUPED>
__device__ __forceinline__ cq_v4u decode8(uint32_t d, const RowTable& t) {
  // selectors: low nibbles (even weights, or weights 0..3), high nibbles (odd, or 4..7)
  const uint32_t sA = d & 0x0f0f0f0fu, sB = (d >> 4) & 0x0f0f0f0fu;
  const uint32_t uA = sA ^ 0x08080808u, uB = sB ^ 0x08080808u;
  const uint32_t loA = __builtin_amdgcn_perm(t.lo[1], t.lo[0], sA) ^ __builtin_amdgcn_perm(t.lo[3], t.lo[2], uA);
  const uint32_t hiA = __builtin_amdgcn_perm(t.hi[1], t.hi[0], sA) ^ __builtin_amdgcn_perm(t.hi[3], t.hi[2], uA);
  const uint32_t loB = __builtin_amdgcn_perm(t.lo[1], t.lo[0], sB) ^ __builtin_amdgcn_perm(t.lo[3], t.lo[2], uB);
  const uint32_t hiB = __builtin_amdgcn_perm(t.hi[1], t.hi[0], sB) ^ __builtin_amdgcn_perm(t.hi[3], t.hi[2], uB);
  // 16-bit values: xa01 = {low-nibble weights 0, 1}, xa23 = {2, 3}; same for the high-nibble weights
  const uint32_t xa01 = __builtin_amdgcn_perm(hiA, loA, 0x05010400u), xa23 = __builtin_amdgcn_perm(hiA, loA, 0x07030602u);
  const uint32_t xb01 = __builtin_amdgcn_perm(hiB, loB, 0x05010400u), xb23 = __builtin_amdgcn_perm(hiB, loB, 0x07030602u);
  if constexpr (GROUPED) return cq_v4u{xa01, xa23, xb01, xb23};
  cq_v4u o;
  o[0] = __builtin_amdgcn_perm(xb01, xa01, 0x05040100u);  // weights 0,1
  o[1] = __builtin_amdgcn_perm(xb01, xa01, 0x07060302u);  // weights 2,3
  o[2] = __builtin_amdgcn_perm(xb23, xa23, 0x05040100u);  // weights 4,5
  o[3] = __builtin_amdgcn_perm(xb23, xa23, 0x07060302u);  // weights 6,7
  return o;
}

#endif  // CQ_DECODE_H_
