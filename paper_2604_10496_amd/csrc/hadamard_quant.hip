// Online-Hadamard variant (evaluation section, the "had" setting): the intermediate of the expert FFN is
// rotated by a Hadamard matrix in front of the down projection, h' = h H_I / sqrt(I), and quantized per row
// like the layer's input.
//
// H_I = H_m (x) H_p with p = 2^k and m = 1 (I a power of two) or m = 4 * (odd part of I) in {12, 28, 44}, H_m
// from Paley's constructions (index i = a*p + b).  The general kernel: one workgroup per row keeps it in LDS, k butterfly
// stages over the blocks of p (a fast Walsh-Hadamard transform, two stages per barrier), then every thread
// combines the m values at its positions b with the signs of H_m (a compile-time table), scales, and the row
// maximum gives the integer codes.  Cost O(I (log p + m)) per row instead of O(I^2).
#include <type_traits>

#include "cq_internal.h"
#include "cq_quotient.h"

namespace {

constexpr int kHadThreads = 512;
constexpr int kHadMaxI = 16384;   // the row as fp32 in 64 KiB of LDS

// Legendre symbol of x modulo the odd prime q
constexpr int legendre(int x, int q) {
  x = ((x % q) + q) % q;
  if (x == 0) return 0;
  for (int y = 1; y < q; ++y)
    if ((y * y) % q == x) return 1;
  return -1;
}

// H_m[a][a2], m in {12, 44}: I + S, S = [[0, 1^T], [-1, Q]], Q[i][j] = chi(j - i) (Paley, q = m - 1 = 3 mod 4);
// m = 28: S (x) [[1,1],[1,-1]] + I (x) [[1,-1],[-1,-1]], S = [[0, 1^T], [1, Q]], Q[i][j] = chi(i - j) (q = 13)
constexpr int paley_entry(int m, int a, int a2) {
  if (m == 12 || m == 44) {
    const int q = m - 1;
    if (a == a2) return 1;
    if (a == 0) return 1;
    if (a2 == 0) return -1;
    return legendre((a2 - 1) - (a - 1), q);
  }
  const int q = 13;
  const int i = a >> 1, u = a & 1, j = a2 >> 1, v = a2 & 1;
  int s = 0;
  if (i == 0 && j == 0) s = 0;
  else if (i == 0 || j == 0) s = 1;
  else s = legendre((i - 1) - (j - 1), q);
  const int A = (u == 1 && v == 1) ? -1 : 1;
  const int B = (u == 0 && v == 0) ? 1 : -1;
  return s * A + (i == j ? B : 0);
}

// the signs as a compile-time table: the unrolled combination below becomes plain additions and subtractions
template <int M_>
struct PaleySigns {
  bool neg[M_][M_];
  constexpr PaleySigns() : neg{} {
    for (int a = 0; a < M_; ++a)
      for (int a2 = 0; a2 < M_; ++a2) neg[a][a2] = M_ > 1 && paley_entry(M_, a, a2) < 0;
  }
};

template <int M_>
__global__ __launch_bounds__(kHadThreads) void hadamard_quant_kernel(const float* __restrict__ Hin, int I, int p, int k,
                                                                     float qmax,
                                                                     int8_t* __restrict__ Q, uint16_t* __restrict__ Q16,
                                                                     float* __restrict__ scale,
                                                                     float* __restrict__ HR) {
  extern __shared__ float row[];
  __shared__ float red[kHadThreads / 64];
  const int tid = threadIdx.x;
  const size_t r = blockIdx.x;
  const float* src = Hin + r * (size_t)I;
  for (int c = tid * 4; c < I; c += kHadThreads * 4)
    *reinterpret_cast<float4*>(row + c) = *reinterpret_cast<const float4*>(src + c);
  __syncthreads();

  // ---- Walsh-Hadamard butterflies inside every block of p = 2^k values, two stages per barrier ----
  int s = 0;
  for (; s + 1 < k; s += 2) {
    // quadruple (i, i+d, i+2d, i+3d), d = 2^s: index bits s and s+1 are the local ones
    const int d = 1 << s;
    for (int idx = tid; idx < (I >> 2); idx += kHadThreads) {
      const int i = ((idx >> s) << (s + 2)) | (idx & (d - 1));
      const float a = row[i], b = row[i + d], c = row[i + 2 * d], e = row[i + 3 * d];
      const float ab = a + b, amb = a - b, ce = c + e, cme = c - e;
      row[i] = ab + ce;
      row[i + d] = amb + cme;
      row[i + 2 * d] = ab - ce;
      row[i + 3 * d] = amb - cme;
    }
    __syncthreads();
  }
  if (s < k) {
    const int d = 1 << s;
    for (int idx = tid; idx < (I >> 1); idx += kHadThreads) {
      const int i = ((idx >> s) << (s + 1)) | (idx & (d - 1));
      const float a = row[i], b = row[i + d];
      row[i] = a + b;
      row[i + d] = a - b;
    }
    __syncthreads();
  }

  // ---- the m blocks are combined with the signs of H_m: out[a2] = sum_a v[a] H_m[a][a2]; scaling ----
  const float norm = 1.f / sqrtf((float)I);
  float amax = 0.f;
  for (int b = tid; b < p; b += kHadThreads) {
    float v[M_];
#pragma unroll
    for (int a = 0; a < M_; ++a) v[a] = row[a * p + b];
    if constexpr (M_ == 1) {
      const float o = v[0] * norm;
      row[b] = o;
      amax = fmaxf(amax, fabsf(o));
    } else {
      constexpr PaleySigns<M_> sg{};
#pragma unroll
      for (int a2 = 0; a2 < M_; ++a2) {
        float acc = 0.f;
#pragma unroll
        for (int a = 0; a < M_; ++a) acc += sg.neg[a][a2] ? -v[a] : v[a];
        const float o = acc * norm;
        row[a2 * p + b] = o;   // only this thread touches position b of any block
        amax = fmaxf(amax, fabsf(o));
      }
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off));
  if ((tid & 63) == 0) red[tid >> 6] = amax;
  __syncthreads();
  amax = red[0];
#pragma unroll
  for (int i = 1; i < kHadThreads / 64; ++i) amax = fmaxf(amax, red[i]);
  const float sc = amax == 0.f ? 1.f : amax / qmax;
  if (tid == 0) scale[r] = sc;

  // ---- integer codes: round to nearest, ties to even ----
  for (int c = tid * 4; c < I; c += kHadThreads * 4) {
    const float4 v = *reinterpret_cast<const float4*>(row + c);
    if (HR) *reinterpret_cast<float4*>(HR + r * (size_t)I + c) = v;
    const float r0 = fminf(fmaxf(rintf(v.x / sc), -qmax), qmax);
    const float r1 = fminf(fmaxf(rintf(v.y / sc), -qmax), qmax);
    const float r2 = fminf(fmaxf(rintf(v.z / sc), -qmax), qmax);
    const float r3 = fminf(fmaxf(rintf(v.w / sc), -qmax), qmax);
    const uint32_t packed = ((uint32_t)(int)r0 & 0xffu) | (((uint32_t)(int)r1 & 0xffu) << 8) |
                            (((uint32_t)(int)r2 & 0xffu) << 16) | (((uint32_t)(int)r3 & 0xffu) << 24);
    if (Q) *reinterpret_cast<uint32_t*>(Q + r * (size_t)I + c) = packed;
    if (Q16)  // the same codes as bf16 bit patterns (exact: small integers)
      *reinterpret_cast<uint2*>(Q16 + r * (size_t)I + c) =
          make_uint2((__float_as_uint(r0) >> 16) | (__float_as_uint(r1) & 0xffff0000u),
                     (__float_as_uint(r2) >> 16) | (__float_as_uint(r3) & 0xffff0000u));
  }
}

// ---- in registers ----
// H_I = H_A (x) H_P with P = 32 .. 512: A is the Paley order, or for a power of two 16 or 32 of its factors of 2.
// Bound by memory (4 bytes in, 1 to 7 out per value); one pass through LDS is what is left of the exchanges:
//   1. thread b of a row loads its A values (whole cache lines per wavefront), combines them with H_A in registers and
//      writes them to LDS;
//   2. 16 lanes take one of the A blocks of P, a lane the values b = 64 h + 4 l + j of it: the bits of j and h are
//      butterflies in registers, those of l are data-parallel moves inside a row of 16 lanes.
// The general kernel above (an LDS pass per two bits, every value combined from LDS) against this one, back-to-back calls
// that also store the fp32 rows: 4096 rows of 14336 174 / 103 us (5.1 TB/s of what it reads and writes), of 4096 47.5 / 24.4,
// of 2048 29.9 / 18.0, of 1408 56 / 15.5, of 768 16.4 / 14.7 (a call alone takes 14); 1001 rows of 14336 47.6 / 25.9.  In
// a graph, 16 and 4096 rows: 1024 3.9 / 3.5 and 18.5 / 8.4, 1536 4.3 / 3.8 and 21.9 / 12.1, 1792 5.2 / 4.8 and 29.7 / 13.3, 3072
// 5.0 / 3.8 and 33.8 / 19.2, 3584 6.7 / 5.6 and 45.6 / 23.9, 5632 9.7 / 8.6 and 86.5 / 39.4, 6144 7.3 / 5.3 and 63.4 / 40.3, 7168
// 8.3 / 5.7 and 70.9 / 42.4, 8192 9.7 / 5.2 and 92.5 / 52.8, 11264 12.6 / 8.8 and 153.7 / 85.9, 16384 16.0 / 6.1 and 202.9 / 112.7.
// Error against float64 over 17 of the widths, 1024 rows and six draws each, general kernel / this one: 0.85e-7 .. 1.48e-7 /
// 0.85e-7 .. 1.47e-7 in the 2-norm and no larger at any width; largest, of a row's maximum, 1.8e-7 .. 5.4e-7 / 1.9e-7 .. 2.8e-7;
// codes on the other side of a rounding tie than float64's, of 561 million, 119 / 108 (4 bits) and 2080 / 1954 (8 bits).
//
// Step 2 across lanes.  With s_j the sign of bit j of the lane and P_j the exchange of lanes that differ in it, a stage is
// v <- s_j v + P_j v.  On x = (product of all s_j) v it becomes x <- x - s_j P_j x, one multiply-add on a moved operand, and
// after the last stage x = v.  There is no move for lanes that differ in bit 2 alone; lanes that differ in bits 0..2 have
// one (row_half_mirror), so bits are taken in the basis {1, 2, 7, 8} of the lane number: lane l then ends with output
// y(l) = (l0 ^ l2, l1 ^ l2, l0 ^ l1 ^ l2, l3) of the 16 instead of l.

template <int CTRL>
__device__ __forceinline__ float lane_move(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}

// v <- H_A v (rows of the sign tables: inputs, columns: outputs)
template <int A>
__device__ __forceinline__ void combine(float (&v)[A]) {
  if constexpr ((A & (A - 1)) == 0) {
#pragma unroll
    for (int d = 1; d < A; d <<= 1)
#pragma unroll
      for (int i = 0; i < A; ++i)
        if (!(i & d)) {
          const float a = v[i], b = v[i | d];
          v[i] = a + b;
          v[i | d] = a - b;
        }
  } else if constexpr (A == 28) {
    // H_28 = S (x) [[1,1],[1,-1]] + I (x) [[1,-1],[-1,-1]]: with p = x0 + x1 and d = x0 - x1 of a pair, out0 = S p + d and
    // out1 = S d - p (418 additions instead of 756)
    constexpr PaleySigns<28> sg{};
    float p[14], d[14];
#pragma unroll
    for (int i = 0; i < 14; ++i) {
      p[i] = v[2 * i] + v[2 * i + 1];
      d[i] = v[2 * i] - v[2 * i + 1];
    }
#pragma unroll
    for (int j = 0; j < 14; ++j) {
      float a = d[j], b = -p[j];
#pragma unroll
      for (int i = 0; i < 14; ++i)
        if (i != j) {   // (S[i][j]: the sign of the pair's first entry)
          a += sg.neg[2 * i][2 * j] ? -p[i] : p[i];
          b += sg.neg[2 * i][2 * j] ? -d[i] : d[i];
        }
      v[2 * j] = a;
      v[2 * j + 1] = b;
    }
  } else {
    constexpr PaleySigns<A> sg{};
    float o[A];
#pragma unroll
    for (int j = 0; j < A; ++j) {
      float a = 0.f;
#pragma unroll
      for (int i = 0; i < A; ++i) a += sg.neg[i][j] ? -v[i] : v[i];
      o[j] = a;
    }
#pragma unroll
    for (int j = 0; j < A; ++j) v[j] = o[j];
  }
}

// NT threads per row, ROWS rows per workgroup
template <int A, int LOGP, int NT, int ROWS>
__global__ __launch_bounds__(NT * ROWS) void hadamard_rows_kernel(const float* __restrict__ Hin, int M, float qmax,
                                                                  int8_t* __restrict__ Q, uint16_t* __restrict__ Q16,
                                                                  float* __restrict__ scale, float* __restrict__ HR) {
  constexpr int P = 1 << LOGP, I = A * P;
  constexpr int kStride = P + 16;                      // of a block in LDS (floats): four blocks on different banks
  constexpr int L = P < 64 ? 8 : 16;                   // lanes per block in step 2
  constexpr int HI = P / (4 * L);                      // values of h
  constexpr int kItems = A * L, N2 = (kItems + NT - 1) / NT;
  extern __shared__ float rows_lds[];
  __shared__ float red[ROWS][NT / 64];
  const int sub = threadIdx.x / NT, tid = threadIdx.x - sub * NT;
  const int row = blockIdx.x * ROWS + sub;
  const bool real = row < M;
  const size_t base = (size_t)(real ? row : M - 1) * I;   // (rows past the end read the last one and store nothing)
  const float* src = Hin + base;
  float* lds = rows_lds + sub * (A * kStride);

  // ---- step 1 ----
  if constexpr (P < 64) {
    // A = 44, 32 positions: the two half wavefronts share the outputs of a position.  The core of H_44 is circulant
    // (chi(out - in) modulo 43), so the second half does the same sums on inputs that are renumbered by 22.
    static_assert(A == 44 || P >= 64, "two half wavefronts");
    constexpr int q = 43;
    const int b = tid & 31, h = tid >> 5;
    const float* s0 = src + b + (1 + 22 * h) * P;                    // w[i] = v[1 + (i + 22 h) mod 43], i < 21
    const float* s1 = src + b + (h ? 1 - 21 : 1) * P;                // ... and from 21 on
    float w[q];
#pragma unroll
    for (int i = 0; i < q; ++i) w[i] = i < 21 ? s0[i * P] : s1[i * P];
    const float v0 = src[b];
    float out0 = v0;
#pragma unroll
    for (int i = 0; i < q; ++i) out0 -= w[i];
    constexpr PaleySigns<44> sg{};
#pragma unroll
    for (int i = 0; i < 22; ++i) {
      float a = v0 + w[i];
#pragma unroll
      for (int j = 0; j < q; ++j)
        if (j != i) a += sg.neg[1 + j][1 + i] ? -w[j] : w[j];
      const int n = 1 + i + 22 * h;                                  // (22 + 21 is output 1 again: output 0 in its place)
      if (i == 21) a = h ? out0 : a;
      lds[(i == 21 && h ? 0 : n) * kStride + b] = a;
    }
  } else {
    float v[A];
#pragma unroll
    for (int a = 0; a < A; ++a) v[a] = src[a * P + tid];
    combine<A>(v);
#pragma unroll
    for (int a = 0; a < A; ++a) lds[a * kStride + tid] = v[a];
  }
  if constexpr (NT > 64) __syncthreads();
  else cq_wave_lds_fence();   // (a row is one wavefront's)

  // ---- step 2 ----
  const int l = tid & (L - 1);
  const int l0 = l & 1, l1 = (l >> 1) & 1, l2 = (l >> 2) & 1, l3 = (l >> 3) & 1;
  const float sign = (l0 ^ l1 ^ l2 ^ l3) ? -1.f : 1.f;               // product of the four below
  const float m1 = (l0 ^ l2) ? 1.f : -1.f, m2 = (l1 ^ l2) ? 1.f : -1.f, m4 = l2 ? 1.f : -1.f, m8 = l3 ? 1.f : -1.f;   // -s_j
  const int y = (l0 ^ l2) | ((l1 ^ l2) << 1) | ((l0 ^ l1 ^ l2) << 2) | (l3 << 3);
  const float norm = 1.f / sqrtf((float)I);
  float x[N2][HI][4];
  float amax = 0.f;
#pragma unroll
  for (int n = 0; n < N2; ++n) {
    const int item = tid + n * NT;
    const int a = (item < kItems ? item : 0) / L;
#pragma unroll
    for (int h = 0; h < HI; ++h) {
      const float4 t = *reinterpret_cast<const float4*>(lds + a * kStride + h * (4 * L) + l * 4);
      const float s0 = t.x + t.y, s1 = t.x - t.y, s2 = t.z + t.w, s3 = t.z - t.w;
      x[n][h][0] = s0 + s2; x[n][h][1] = s1 + s3; x[n][h][2] = s0 - s2; x[n][h][3] = s1 - s3;
    }
#pragma unroll
    for (int d = 1; d < HI; d <<= 1)
#pragma unroll
      for (int h = 0; h < HI; ++h)
        if (!(h & d))
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float u = x[n][h][j], w = x[n][h | d][j];
            x[n][h][j] = u + w;
            x[n][h | d][j] = u - w;
          }
#pragma unroll
    for (int h = 0; h < HI; ++h)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float u = x[n][h][j] * sign;
        u = fmaf(m1, lane_move<0xB1>(u), u);             // quad_perm 1 0 3 2
        u = fmaf(m2, lane_move<0x4E>(u), u);             // quad_perm 2 3 0 1
        u = fmaf(m4, lane_move<0x141>(u), u);            // row_half_mirror
        if constexpr (L == 16) u = fmaf(m8, lane_move<0x128>(u), u);   // row_ror 8
        u *= norm;
        x[n][h][j] = u;
        if (kItems % NT == 0 || item < kItems) amax = fmaxf(amax, fabsf(u));
      }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off));
  if constexpr (NT > 64) {
    if ((tid & 63) == 0) red[sub][tid >> 6] = amax;
    __syncthreads();
    amax = red[sub][0];
#pragma unroll
    for (int i = 1; i < NT / 64; ++i) amax = fmaxf(amax, red[sub][i]);
  }
  const float sc = amax == 0.f ? 1.f : amax / qmax;
  if (!real) return;
  if (tid == 0) scale[row] = sc;

  // ---- integer codes: round to nearest, ties to even ----
  const cq_quotient by(sc);
  auto codes = [&](auto fast) {
#pragma unroll
    for (int n = 0; n < N2; ++n) {
      const int item = tid + n * NT;
      if (kItems % NT != 0 && item >= kItems) break;
      const size_t at = base + (item / L) * P + y * 4;
#pragma unroll
      for (int h = 0; h < HI; ++h) {
        const float* u = x[n][h];
        const size_t e = at + h * (4 * L);
        if (HR) *reinterpret_cast<float4*>(HR + e) = make_float4(u[0], u[1], u[2], u[3]);
        float r[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) r[j] = fminf(fmaxf(rintf(by.get<decltype(fast)::value>(u[j])), -qmax), qmax);
        const uint32_t packed = ((uint32_t)(int)r[0] & 0xffu) | (((uint32_t)(int)r[1] & 0xffu) << 8) |
                                (((uint32_t)(int)r[2] & 0xffu) << 16) | (((uint32_t)(int)r[3] & 0xffu) << 24);
        if (Q) *reinterpret_cast<uint32_t*>(Q + e) = packed;
        if (Q16)  // the same codes as bf16 bit patterns (exact: small integers)
          *reinterpret_cast<uint2*>(Q16 + e) =
              make_uint2((__float_as_uint(r[0]) >> 16) | (__float_as_uint(r[1]) & 0xffff0000u),
                         (__float_as_uint(r[2]) >> 16) | (__float_as_uint(r[3]) & 0xffff0000u));
      }
    }
  };
  if (by.fast) codes(std::true_type{});
  else codes(std::false_type{});
}

// P threads take a row, a wavefront where P = 32; rows of one wavefront share a workgroup by four, of two by two
template <int A, int LOGP>
cq_status launch_rows(const float* Hin, int M, float qmax, int8_t* Q, uint16_t* Q16, float* scale, float* HR, hipStream_t s) {
  constexpr int NT = LOGP > 6 ? 1 << LOGP : 64, ROWS = NT == 64 ? 4 : NT == 128 ? 2 : 1;
  constexpr int lds = ROWS * A * ((1 << LOGP) + 16) * 4;
  auto kern = hadamard_rows_kernel<A, LOGP, NT, ROWS>;
  static std::atomic<bool> configured{false};
  const cq_status st = cq_configure_lds(kern, lds, configured, false);
  if (st != CQ_OK) return st;
  hipLaunchKernelGGL(kern, dim3((M + ROWS - 1) / ROWS), dim3(NT * ROWS), lds, s, Hin, M, qmax, Q, Q16, scale, HR);
  return cq_check_launch();
}

// Blocks of 2^logp values, A of them: in registers from 64 on (32 where 44 blocks make up for it) as far as a thread's values
// fit, which for a power of two takes 32 blocks from 8192 on; CQ_ERR_UNSUPPORTED: the general kernel.  Narrower rows leave
// a wavefront's lanes without work, 12288 would need 1024 threads for 12 blocks.  44 blocks of 64, a wavefront's work for
// each row, pay from 256 rows on (2816: 64 rows 7.8 / 8.2 us, 300 rows 9.3 / 8.7).
template <int A>
cq_status rows_by_block(int logp, const float* Hin, int M, float qmax, int8_t* Q, uint16_t* Q16, float* scale, float* HR,
                        hipStream_t s) {
  switch (logp) {
    case 5:
      if constexpr (A == 44) return launch_rows<A, 5>(Hin, M, qmax, Q, Q16, scale, HR, s);
      return CQ_ERR_UNSUPPORTED;
    case 6: return A == 44 && M < 256 ? CQ_ERR_UNSUPPORTED : launch_rows<A, 6>(Hin, M, qmax, Q, Q16, scale, HR, s);
    case 7: return launch_rows<A, 7>(Hin, M, qmax, Q, Q16, scale, HR, s);
    case 8: return launch_rows<A, 8>(Hin, M, qmax, Q, Q16, scale, HR, s);
    case 9:
      if constexpr (A == 16) return launch_rows<32, 8>(Hin, M, qmax, Q, Q16, scale, HR, s);
      else if constexpr (A * 512 <= kHadMaxI) return launch_rows<A, 9>(Hin, M, qmax, Q, Q16, scale, HR, s);
      return CQ_ERR_UNSUPPORTED;
    case 10:
      if constexpr (A == 16) return launch_rows<32, 9>(Hin, M, qmax, Q, Q16, scale, HR, s);
      return CQ_ERR_UNSUPPORTED;
    default: return CQ_ERR_UNSUPPORTED;
  }
}

// I = m * 2^k with m in {1, 12, 28, 44}; false if I has no such form
bool had_split(int I, int* m, int* p, int* k) {
  if (I <= 0) return false;
  int odd = I, twos = 0;
  while ((odd & 1) == 0) { odd >>= 1; ++twos; }
  if (odd == 1) { *m = 1; *p = I; *k = twos; return true; }
  if (odd != 3 && odd != 7 && odd != 11) return false;
  if (twos < 2) return false;
  *m = 4 * odd;
  *k = twos - 2;
  *p = 1 << *k;
  return true;
}

}  // namespace

bool cq_hadamard_supported(int I) {
  int m, p, k;
  return had_split(I, &m, &p, &k) && I % 4 == 0 && I <= kHadMaxI;
}

cq_status cq_hadamard_quant_launch(const float* Hin, int M, int I, int bits, int8_t* Q, uint16_t* Q16, float* scale,
                                   float* HR, hipStream_t s) {
  int m, p, k;
  if (!had_split(I, &m, &p, &k)) return CQ_ERR_SHAPE;
  if (M == 0) return CQ_OK;
  {
    static std::atomic<bool> c1{false}, c12{false}, c28{false}, c44{false};
    constexpr int kMaxLds = kHadMaxI * 4;
    if (cq_configure_lds(hadamard_quant_kernel<1>, kMaxLds, c1, false) != CQ_OK ||
        cq_configure_lds(hadamard_quant_kernel<12>, kMaxLds, c12, false) != CQ_OK ||
        cq_configure_lds(hadamard_quant_kernel<28>, kMaxLds, c28, false) != CQ_OK ||
        cq_configure_lds(hadamard_quant_kernel<44>, kMaxLds, c44, false) != CQ_OK)
      return CQ_ERR_HIP;
  }
  const float qmax = (float)((1 << (bits - 1)) - 1);
  const cq_status in_registers = m == 1    ? rows_by_block<16>(k - 4, Hin, M, qmax, Q, Q16, scale, HR, s)
                                 : m == 12 ? rows_by_block<12>(k, Hin, M, qmax, Q, Q16, scale, HR, s)
                                 : m == 28 ? rows_by_block<28>(k, Hin, M, qmax, Q, Q16, scale, HR, s)
                                           : rows_by_block<44>(k, Hin, M, qmax, Q, Q16, scale, HR, s);
  if (in_registers != CQ_ERR_UNSUPPORTED) return in_registers;
  const size_t lds = (size_t)I * 4;
  switch (m) {
    case 1:
      hipLaunchKernelGGL(hadamard_quant_kernel<1>, dim3(M), dim3(kHadThreads), lds, s, Hin, I, p, k, qmax, Q, Q16,
                         scale, HR);
      break;
    case 12:
      hipLaunchKernelGGL(hadamard_quant_kernel<12>, dim3(M), dim3(kHadThreads), lds, s, Hin, I, p, k, qmax, Q, Q16,
                         scale, HR);
      break;
    case 28:
      hipLaunchKernelGGL(hadamard_quant_kernel<28>, dim3(M), dim3(kHadThreads), lds, s, Hin, I, p, k, qmax, Q, Q16,
                         scale, HR);
      break;
    default:
      hipLaunchKernelGGL(hadamard_quant_kernel<44>, dim3(M), dim3(kHadThreads), lds, s, Hin, I, p, k, qmax, Q, Q16,
                         scale, HR);
      break;
  }
  return cq_check_launch();
}

extern "C" cq_status cq_hadamard_quant(const float* Hrows, int M, int I, int bits, float* HR_out, int8_t* Q_out,
                                       float* scale_out, cq_stream stream) {
  if (M < 0 || I <= 0) return CQ_ERR_SHAPE;
  if (!cq_hadamard_supported(I)) return CQ_ERR_SHAPE;
  if (bits != 4 && bits != 8) return CQ_ERR_UNSUPPORTED;
  if (M == 0) return CQ_OK;  // nothing to do (the pointers may be NULL)
  if (!Hrows || !Q_out || !scale_out) return CQ_ERR_NULL;
  return cq_hadamard_quant_launch(Hrows, M, I, bits, Q_out, nullptr, scale_out, HR_out, (hipStream_t)stream);
}
