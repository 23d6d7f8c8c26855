// a1 for prefill-sized batches: X_R = X R on the f16 matrix cores at (about) fp32 accuracy.
//
// Every fp32 operand is written as hi + 2^-11 lo with hi = f16(v) and lo = f16((v - hi) 2^11): v - hi is
// exact in fp32 and has at most 13 significant bits, so hi + 2^-11 lo differs from v by at most 2^-23 |v|.
// Products of two f16 numbers are exact in fp32, and the matrix cores accumulate in fp32, so
//     2^11 X R  =  Xh (2^11 Rh)  +  Xh Rl  +  Xl Rh  +  2^-11 Xl Rl
// evaluated without its last term (relative size 2^-22) is as accurate as an fp32 product, at three f16
// MFMAs per tile step instead of one fp32 MFMA step that is sixteen times slower.  All three products
// carry the same factor 2^11 and go into ONE accumulator (2^11 Rh is formed in registers from Rh: an
// exact exponent shift, |R| < 32 assumed -- R is orthogonal).  Rows of X are divided by a power of two
// first (exact) so that their largest entry lies in [1, 2): no f16 overflow or underflow whatever the
// scale of the activations.  R is split once, when the layer is set up, into the order the MFMA
// fragments are loaded in.
//
// Kernel: workgroup tile 256 output columns x 128 tokens (or 64), four wavefronts, each owning 64 columns (as
// MFMA "A" rows, two blocks of 32) and all the tokens (2 x 4 accumulator blocks of 32x32, or 2 x 2).  R fragments
// go from global memory (L2) straight into registers, one step (64 k) ahead
// (two steps ahead, with 64 more registers, was measured: no faster, so it is not their latency that bounds the loop); token tiles (both halves)
// arrive by direct global->LDS loads, four steps deep.
#include "cq_internal.h"
#include "cq_async.h"

namespace {

using namespace cq_async;

constexpr int kCols = 256;             // output columns per workgroup
constexpr int kTok = 128;              // tokens per workgroup (or, C = 2, 64)
constexpr int kStepK = 64;             // K per pipeline step (four MFMA sub-steps of 16)
constexpr int kStepBytes = kStepK * 2; // one token's share of a step and plane, in LDS and in memory
constexpr int kDepth = 4;                        // token tiles in LDS
constexpr int kOutStride = kCols * 4 + 16;       // epilogue staging row (64 tokens at a time)
// hi and lo tile of a step, kDepth of them: 128 KiB, or (C = 2) 64 KiB, of which the epilogue takes one more
constexpr int rot_lds_bytes(int C) {
  const int ring = kDepth * 2 * 32 * C * kStepBytes, out = 64 * kOutStride;
  return ring > out ? ring : out;
}
constexpr float kLoScale = 2048.f, kLoUnscale = 1.f / 2048.f;

__device__ __forceinline__ uint32_t f16_bits(float x) {
  const _Float16 h = (_Float16)x;
  return (uint32_t) __builtin_bit_cast(uint16_t, h);
}
__device__ __forceinline__ float f16_value(float x) { return (float)(_Float16)x; }

// R [K, N] fp32 -> fragments: block nb = n/32, sub-step j = k/16, plane p (0 hi, 1 lo): 1 KiB at
// ((nb*(K/16) + j)*2 + p)*1024 holding, for lane l, R[j*16 + (l/32)*8 + i][nb*32 + l%32], i = 0..7.
__global__ __launch_bounds__(256) void split_R_kernel(const float* __restrict__ R, int H, uint4* __restrict__ out) {
  const int nJ = H / 16;
  const size_t frag = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6);  // (nb, j)
  const int lane = threadIdx.x & 63;
  if (frag >= (size_t)(H / 32) * nJ) return;
  const int nb = (int)(frag / nJ), j = (int)(frag - (size_t)nb * nJ);
  const int n = nb * 32 + (lane & 31), k0 = j * 16 + (lane >> 5) * 8;
  uint32_t hi[4], lo[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float a = R[(size_t)(k0 + 2 * i) * H + n], b = R[(size_t)(k0 + 2 * i + 1) * H + n];
    const float ah = f16_value(a), bh = f16_value(b);
    hi[i] = f16_bits(ah) | (f16_bits(bh) << 16);
    lo[i] = f16_bits((a - ah) * kLoScale) | (f16_bits((b - bh) * kLoScale) << 16);
  }
  out[(frag * 2 + 0) * 64 + lane] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
  out[(frag * 2 + 1) * 64 + lane] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
}

// One workgroup per token: row maximum, power-of-two scale s (largest entry of x/s in [1, 2)), then the
// two f16 planes of x/s.  planes: hi [T, H], lo [T, H] (the latter times 2^11); row_pow2 [T] = s.
__global__ __launch_bounds__(256) void split_X_kernel(const float* __restrict__ X, int T, int H,
                                                      uint16_t* __restrict__ hi, uint16_t* __restrict__ lo,
                                                      float* __restrict__ row_pow2) {
  __shared__ float red[4];
  const int t = blockIdx.x, tid = threadIdx.x;
  const float* x = X + (size_t)t * H;
  float amax = 0.f;
  for (int c = tid * 4; c < H; c += 1024) {
    const float4 v = *reinterpret_cast<const float4*>(x + c);
    amax = fmaxf(amax, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off));
  if ((tid & 63) == 0) red[tid >> 6] = amax;
  __syncthreads();
  amax = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  // s = 2^floor(log2(amax)): the exponent field alone (1 for a zero or denormal maximum)
  const uint32_t ebits = __float_as_uint(amax) & 0x7f800000u;
  const float s = ebits == 0u ? 1.f : __uint_as_float(ebits);
  const float inv = 1.f / s;  // exact: a power of two
  if (tid == 0) row_pow2[t] = s;
  for (int c = tid * 4; c < H; c += 1024) {
    const float4 v = *reinterpret_cast<const float4*>(x + c);
    const float a[4] = {v.x * inv, v.y * inv, v.z * inv, v.w * inv};
    float h[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) h[i] = f16_value(a[i]);
    *reinterpret_cast<uint2*>(hi + (size_t)t * H + c) =
        make_uint2(f16_bits(h[0]) | (f16_bits(h[1]) << 16), f16_bits(h[2]) | (f16_bits(h[3]) << 16));
    *reinterpret_cast<uint2*>(lo + (size_t)t * H + c) =
        make_uint2(f16_bits((a[0] - h[0]) * kLoScale) | (f16_bits((a[1] - h[1]) * kLoScale) << 16),
                   f16_bits((a[2] - h[2]) * kLoScale) | (f16_bits((a[3] - h[3]) * kLoScale) << 16));
  }
}

struct RotArgs {
  const uint8_t* Rs;       // split R fragments
  const uint16_t* Xh;      // [T, K] f16
  const uint16_t* Xl;      // [T, K] f16 (times 2^11)
  const float* row_pow2;   // [T]
  float* XR;               // [T, N] fp32, or (K parts) partial sums [parts][T][N]
  int T, N, K;
  int row_tiles;           // N / 256
  int tok_tiles;           // ceil(T / 128), or of 64
  int ksteps;              // K steps (of 64) per K part, a multiple of four
  int n_work;              // token tiles x row tiles x K parts
};

// pairs of f16 times 2^11 (exact: an exponent shift)
typedef _Float16 cq_h2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pair_times_2048(uint32_t a) {
  const cq_h2 k = {(_Float16)2048.f, (_Float16)2048.f};
  const cq_h2 v = __builtin_bit_cast(cq_h2, a) * k;
  return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ cq_v4u times_2048(const cq_v4u a) {
  // (built in one piece: element-wise stores into an uninitialised vector were seen to compile into a
  // broadcast of element 0 here)
  const cq_v4u r = {pair_times_2048(a[0]), pair_times_2048(a[1]), pair_times_2048(a[2]), pair_times_2048(a[3])};
  return r;
}

__device__ __forceinline__ cq_v16f mfma_f16(const cq_v4u a, const cq_v4u b, cq_v16f c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(cq_v8f16, a), __builtin_bit_cast(cq_v8f16, b), c, 0,
                                                0, 0);
}

__device__ __forceinline__ cq_v4f mfma_f16_16(const cq_v4u a, const cq_v4u b, cq_v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(cq_v8f16, a), __builtin_bit_cast(cq_v8f16, b), c, 0, 0, 0);
}

// C: token blocks of 32.  TWICE: the two halves of the K range are summed apart and added at the end (an accumulator rounds
// at the size of its own partial sum: the result is as accurate as two parts').
template <int C, bool TWICE>
__global__ __launch_bounds__(256, 1) void rot_split_kernel(const RotArgs p) {
  constexpr int kC = C, kTok = 32 * C;
  constexpr int kPlaneBytes = kTok * kStepBytes, kStageBytes = 2 * kPlaneBytes;
  // XCD-aware remap of the linear workgroup id (ids go round-robin over the 8 XCDs): XCD x takes a
  // contiguous share of the work, so that neighbours in its L2 share token tiles and columns of R
  const int per = (p.n_work + 7) >> 3;
  const int work = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per || work >= p.n_work) return;
  // (the token tiles of a K part and a column tile follow each other: they share its piece of R)
  const int rest = work / p.tok_tiles, tile = work - rest * p.tok_tiles;
  const int kz = rest / p.row_tiles, rt = rest - kz * p.row_tiles;
  const int mrow0 = tile * kTok, mcnt = min(kTok, p.T - mrow0);

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r32 = lane & 31, g2 = lane >> 5;
  const int N = p.N, K = p.K;
  const int nS = p.ksteps, sb = kz * p.ksteps, nJ = K / 16;   // this workgroup's K steps: sb .. sb + nS - 1
  // this wavefront's two column blocks: nb0, nb0 + 1.  Fragment (rb, sub-step j, plane pl) of lane l is at
  // Rs + (((nb0 + rb)*nJ + j)*2 + pl)*1024 + 16 l: a uniform base, the lane offset, an immediate.
  const int nb0 = __builtin_amdgcn_readfirstlane((rt * kCols + wave * 64) / 32);
  const uint8_t* wbase = p.Rs + ((size_t)nb0 * nJ + (size_t)sb * 4) * 2048;
  const size_t rbstride = (size_t)nJ * 2048;
  const uint32_t lane16 = (uint32_t)lane * 16;

  // ---- token tiles: as in the codebook product's large-tile kernel (token-major rows of 128 bytes,
  // chunk c of token t at position c ^ ((t >> 1) & 7); one direct-to-LDS load moves 8 tokens x 128 bytes;
  // the swizzle is applied on the global side).  Wavefront w moves tokens [8Cw, 8Cw + 8C) of both planes:
  // 2 x C loads per step, C/2 of them per sub-step. ----
  uint32_t aoff[C];  // byte offset of this lane's 16 bytes of step 0 within a plane (T*K*2 < 2^32)
#pragma unroll
  for (int i = 0; i < C; ++i) {
    const int tok = wave * (8 * C) + i * 8 + (lane >> 3);
    const uint32_t row = (uint32_t)(mrow0 + min(tok, mcnt - 1));  // tokens past the end repeat the last row
    const int chunk = (lane & 7) ^ ((tok >> 1) & 7);
    aoff[i] = (row * (uint32_t)K + (uint32_t)chunk * 8) * 2;
  }
  const uint8_t* xh = reinterpret_cast<const uint8_t*>(p.Xh) + (size_t)sb * kStepBytes;
  const uint8_t* xl = reinterpret_cast<const uint8_t*>(p.Xl) + (size_t)sb * kStepBytes;
  const uint32_t lds_wave = __builtin_amdgcn_readfirstlane(wave * (8 * C) * kStepBytes);
  // a quarter of the wavefront's loads of step s: tokens 8Cw + 8jj .. +7 of both planes, or (C = 2) 8 tokens of one
  auto fetch_tile_part = [&](int s, int buf, int jj) {
    const size_t o = (size_t)s * kStepBytes;
    const int i = C == 4 ? jj : jj >> 1;
    if (C == 4 || (jj & 1) == 0) load_global_to_lds_s<0>(buf * kStageBytes + lds_wave + i * 1024, xh + o, aoff[i]);
    if (C == 4 || (jj & 1) == 1) load_global_to_lds_s<0>(buf * kStageBytes + kPlaneBytes + lds_wave + i * 1024, xl + o, aoff[i]);
  };
  // R fragments of sub-step jj of step s: [rb][plane]
  auto fetch_R = [&](cq_v4u (&w)[2][2], int s, int jj) {
    const uint8_t* src = wbase + (size_t)(s * 4 + jj) * 2048;
    load_global_async_s<0>(w[0][0], src, lane16);
    load_global_async_s<1024>(w[0][1], src, lane16);
    load_global_async_s<0>(w[1][0], src + rbstride, lane16);
    load_global_async_s<1024>(w[1][1], src + rbstride, lane16);
  };
  // token fragment: lane (token r32 of block cb, k group g2) wants chunk 2*jj + g2 of the step (the k
  // order of the R fragments), stored at position (2*jj + g2) ^ ((r32 >> 1) & 7) = (g2 ^ ..) ^ (2*jj)
  const uint32_t boff = (uint32_t)r32 * kStepBytes + ((uint32_t)(g2 ^ ((r32 >> 1) & 7)) << 4);
  // Eight address registers (sub-step x lower / upper pair of tile buffers), made opaque to the compiler;
  // buffer, plane and token block go into the instruction's offset field.  (Left to itself the compiler
  // keeps all 128 loop-invariant addresses in registers it does not have.)
  uint32_t bx[2][4];
#pragma unroll
  for (int jj = 0; jj < 4; ++jj) {
    bx[0][jj] = boff ^ ((uint32_t)jj << 5);
    bx[1][jj] = bx[0][jj] + 2 * kStageBytes;
    asm volatile("" : "+v"(bx[0][jj]), "+v"(bx[1][jj]));
  }
  auto read_b = [&](int buf, int plane, int jj, int cb) {
    return lds_read_u128(bx[buf >> 1][jj] + (uint32_t)((buf & 1) * kStageBytes + plane * kPlaneBytes + cb * 32 * kStepBytes));
  };

  cq_v16f acc[2][kC];  // 2^11 X R
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int cb = 0; cb < kC; ++cb)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[rb][cb][i] = 0.f;

  // Vector-memory operations per sub-step, in this order: 4 R fragment loads (sub-step jj of the NEXT
  // step, into the registers just consumed), then C/2 tile loads (part jj of the tile three steps ahead).
  // A fragment is therefore followed by C/2 + 3*(4 + C/2) younger operations when its sub-step comes round
  // (20 or 16), and the last part of the tile two steps ahead by the operations of the current step (24 or 20): those
  // are the two wait counts.  (A count is safe as long as at least that many younger operations exist.)
  constexpr int kPerSub = 4 + C / 2, kWaitR = C / 2 + 3 * kPerSub, kWaitTile = 4 * kPerSub;
  cq_v4u wq[4][2][2];
  // prologue, oldest first: tiles 0 and 1, the R fragments of step 0, tile 2
#pragma unroll
  for (int i = 0; i < 4; ++i) fetch_tile_part(0, 0, i);
#pragma unroll
  for (int i = 0; i < 4; ++i) fetch_tile_part(min(1, nS - 1), 1, i);
#pragma unroll
  for (int jj = 0; jj < 4; ++jj) fetch_R(wq[jj], 0, jj);
#pragma unroll
  for (int i = 0; i < 4; ++i) fetch_tile_part(min(2, nS - 1), 2, i);
  vm_wait<kWaitTile>(wq[0][0][0], wq[0][0][1], wq[0][1][0], wq[0][1][1]);  // tiles 0 and 1 have landed
  __syncthreads();

  cq_v4u bh[kC], bl[kC];
#pragma unroll
  for (int cb = 0; cb < kC; ++cb) {
    bh[cb] = read_b(0, 0, 0, cb);
    bl[cb] = read_b(0, 1, 0, cb);
  }

  cq_v16f first[TWICE ? 2 : 1][TWICE ? kC : 1];   // the first half's sums
  int s0 = 0;
  do {  // K is a multiple of 256: steps come in fours (no zero-trip path, accumulators stay in place)
#pragma unroll
    for (int par = 0; par < kDepth; ++par) {  // step s0 + par reads tile buffer par
      const int s = s0 + par;
      const int s_next = min(s + 1, nS - 1), s_tile = min(s + 3, nS - 1);
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        vm_wait<kWaitR>(wq[jj][0][0], wq[jj][0][1], wq[jj][1][0], wq[jj][1][1]);
        const cq_v4u ah0 = wq[jj][0][0], al0 = wq[jj][0][1], ah1 = wq[jj][1][0], al1 = wq[jj][1][1];
        const cq_v4u aH0 = times_2048(ah0), aH1 = times_2048(ah1);
        // next sub-step's token fragments: jj + 1 of this step, or the first of the next step
        const int nbuf = jj < 3 ? par : (par + 1) & (kDepth - 1), njj = (jj + 1) & 3;
        // three products per accumulator block, a whole round of blocks apart (no back-to-back dependence)
#pragma unroll
        for (int cb = 0; cb < kC; ++cb) {
          acc[0][cb] = mfma_f16(aH0, bh[cb], acc[0][cb]);
          acc[1][cb] = mfma_f16(aH1, bh[cb], acc[1][cb]);
        }
#pragma unroll
        for (int cb = 0; cb < kC; ++cb) {
          acc[0][cb] = mfma_f16(ah0, bl[cb], acc[0][cb]);
          acc[1][cb] = mfma_f16(ah1, bl[cb], acc[1][cb]);
          bl[cb] = read_b(nbuf, 1, njj, cb);
        }
#pragma unroll
        for (int cb = 0; cb < kC; ++cb) {
          acc[0][cb] = mfma_f16(al0, bh[cb], acc[0][cb]);
          acc[1][cb] = mfma_f16(al1, bh[cb], acc[1][cb]);
          bh[cb] = read_b(nbuf, 0, njj, cb);
        }
        __builtin_amdgcn_sched_barrier(0);
        // the consumed registers take the same sub-step of the next step; then this sub-step's tile part
        fetch_R(wq[jj], s_next, jj);
        fetch_tile_part(s_tile, (par + 3) & (kDepth - 1), jj);
        __builtin_amdgcn_sched_barrier(0);
      }
      vm_wait<kWaitTile>(wq[0][0][0], wq[0][0][1], wq[0][1][0], wq[0][1][1]);  // own share of the tile two steps ahead
      __syncthreads();
    }
    s0 += kDepth;
    if constexpr (TWICE) {
      if (s0 * 2 == nS)
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
          for (int cb = 0; cb < kC; ++cb) {
            first[rb][cb] = acc[rb][cb];
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[rb][cb][i] = 0.f;
          }
    }
  } while (s0 < nS);
  if constexpr (TWICE)
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int cb = 0; cb < kC; ++cb)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[rb][cb][i] += first[rb][cb][i];
  // Nothing of this workgroup may still be on its way into LDS when the tile buffers are reused, nor into
  // registers: the last (clamped, unused) fragment loads still target the ring, which therefore has to
  // stay allocated up to this wait -- it is named here so that the compiler cannot reuse it earlier.
  asm volatile("s_waitcnt vmcnt(0)"
               : "+v"(wq[0][0][0]), "+v"(wq[0][0][1]), "+v"(wq[0][1][0]), "+v"(wq[0][1][1]), "+v"(wq[1][0][0]),
                 "+v"(wq[1][0][1]), "+v"(wq[1][1][0]), "+v"(wq[1][1][1]), "+v"(wq[2][0][0]), "+v"(wq[2][0][1]),
                 "+v"(wq[2][1][0]), "+v"(wq[2][1][1]), "+v"(wq[3][0][0]), "+v"(wq[3][0][1]), "+v"(wq[3][1][0]),
                 "+v"(wq[3][1][1])
               :
               : "memory");

  // ---- epilogue: x = s_t 2^-11 acc; through LDS, 64 tokens at a time, so that stores are
  // row-contiguous (a lane holds 4 consecutive columns of ONE token per accumulator quad) ----
  typedef __attribute__((address_space(3))) cq_v4u lds_v4u;
#pragma unroll
  for (int pass = 0; pass < kC / 2; ++pass) {
    __syncthreads();  // the tile buffers (first pass) or the previous pass's rows are no longer read
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int cb = pass * 2 + half;
      const int tl = half * 32 + r32;
      const float sc = p.row_pow2[mrow0 + min(cb * 32 + r32, mcnt - 1)] * kLoUnscale;
#pragma unroll
      for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int vb = 0; vb < 4; ++vb) {
          // MFMA 32x32 output: register v holds row 8*(v/4) + 4*(lane/32) + v%4, column lane%32
          const int col = wave * 64 + rb * 32 + vb * 8 + g2 * 4;
          const uint32_t at = (uint32_t)tl * kOutStride + (uint32_t)col * 4;
          const cq_v4u o = {__float_as_uint(sc * acc[rb][cb][4 * vb]), __float_as_uint(sc * acc[rb][cb][4 * vb + 1]),
                            __float_as_uint(sc * acc[rb][cb][4 * vb + 2]), __float_as_uint(sc * acc[rb][cb][4 * vb + 3])};
          *reinterpret_cast<lds_v4u*>((uintptr_t)at) = o;
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < 64 * (kCols / 4) / 256; ++it) {
      const int i = it * 256 + tid;
      const int tl = i / (kCols / 4), pc = i - tl * (kCols / 4);
      const int tok = pass * 64 + tl;
      if (tok < mcnt) {
        const uint32_t at = (uint32_t)tl * kOutStride + (uint32_t)pc * 16;
        float* dst = p.XR + ((size_t)kz * p.T + mrow0 + tok) * N + (size_t)rt * kCols + pc * 4;
        *reinterpret_cast<cq_v4u*>(dst) = *reinterpret_cast<const lds_v4u*>((uintptr_t)at);
      }
    }
  }
}

// ---- few tokens ----------------------------------------------------------------------------------------------------
// Bound by reading R once.  The fp32 kernel's workgroups read pieces of 1 KiB, 16 KiB apart, and stay at 3.8 TB/s (64 MiB in
// 17 us, also without its matrix instructions; more loads in flight make it slower); the split copy lies in fragment order,
// so that a workgroup of one block of 32 columns reads one contiguous run.  Eight wavefronts share its K range (N sub-steps
// of 16 each), the activations of a wavefront's sub-steps live in its registers, split there: the power of two that a row is
// divided by is that of its largest entry in the wavefront's own slice of K, which can only be closer.
// TB: blocks of 32 tokens; 0: up to 16 tokens on the 16x16x32 shape, whose lanes (token l%16, k group l/16) all hold
// activations of their own (half the loads and conversions).  A pair of fragments becomes its two operands of 16 columns with
// one lane swap per pair of dwords; lane row g then carries sub-step g%2 of the pair, k group g/2.
// Xh Rh has an accumulator of its own and the two small products share another, so that the large one is rounded once per
// step and not three times: together with sums over the wavefronts in pairs the error of X_R falls from 2.1e-7 to 1.5e-7 at
// H = 4096 and from 1.5e-7 to 1.2e-7 at H = 1024, at the same time per call.
constexpr int kFewWaves = 8;
struct RotFewArgs {
  const uint8_t* Rs;
  const float* X;
  float* out;       // [parts][T][H], or X_R itself with one part
  int T, H, parts;
};

// the wavefronts' sums, `apart` entries from each other, in pairs (one after the other, the eight roundings were a third of
// the error; in float64 the layer took 0.2 us longer and the error was 4 % smaller)
__device__ __forceinline__ float4 few_sum(const float4* lds, int apart) {
  float4 v[kFewWaves];
#pragma unroll
  for (int w = 0; w < kFewWaves; ++w) v[w] = lds[w * apart];
#pragma unroll
  for (int d = 1; d < kFewWaves; d *= 2)
#pragma unroll
    for (int w = 0; w < kFewWaves; w += 2 * d) {
      v[w].x += v[w + d].x; v[w].y += v[w + d].y; v[w].z += v[w + d].z; v[w].w += v[w + d].w;
    }
  return v[0];
}

// x . R[:, column] over a wavefront's slice (k from 16 j0 on), from the planes of R in plain fp32: what a slice with an
// infinite entry gives.  Its planes are no numbers (inf - inf); the sum is +-Inf by the sign of x R, or NaN where infinities
// of both signs meet, a NaN is among them, or R is 0, as in an fp32 product.
__device__ __forceinline__ float few_fp32(const RotFewArgs& p, int nb, int j0, int count, int tok, int col) {
  const float* x = p.X + (size_t)tok * p.H + (size_t)j0 * 16;
  const _Float16* r = reinterpret_cast<const _Float16*>(p.Rs) + ((size_t)nb * (p.H / 16) + j0) * 1024 + col * 8;
  float s = 0.f;
#pragma unroll 1
  for (int k = 0; k < count; ++k) {
    const _Float16* e = r + (k >> 4) * 1024 + ((k >> 3) & 1) * 256 + (k & 7);
    s = fmaf(x[k], fmaf((float)e[512], kLoUnscale, (float)e[0]), s);
  }
  return s;
}

template <int N, int TB_>
__global__ __launch_bounds__(64 * kFewWaves, 1) void rot_few_kernel(const RotFewArgs p) {
  constexpr bool HALF = TB_ == 0;
  constexpr int TB = HALF ? 1 : TB_;
  constexpr int NX = HALF ? N / 2 : N;  // activation fragments of a lane
  constexpr int D = N < 8 ? N : 8;      // sub-steps of R in flight (2 KiB each)
  extern __shared__ float few_lds[];   // [wavefront][token block][quad of columns][lane] float4
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r32 = lane & 31, g2 = lane >> 5;
  const int nb = (int)blockIdx.x / p.parts, kz = (int)blockIdx.x - nb * p.parts;
  const int j0 = (kz * kFewWaves + wave) * N;           // this wavefront's first sub-step
  const uint4* frag = reinterpret_cast<const uint4*>(p.Rs) + ((size_t)nb * (p.H / 16) + j0) * 128 + lane;
  uint4 ring[D][2];
#pragma unroll
  for (int d = 0; d < D; ++d) {
    ring[d][0] = frag[(size_t)d * 128];
    ring[d][1] = frag[(size_t)d * 128 + 64];
  }
  // (the loads of R stay in front of the conversion of X, where the compiler leaves 4 of them otherwise: H = 4096, 8 and 16
  // tokens 44.5 -> 43.6 and 46.5 -> 45.5 us per layer, with sixteen in flight 45.3 and 47.6; the shorter slices gain nothing)
  if constexpr (HALF && N == 16) __builtin_amdgcn_sched_barrier(0);
  // this lane's activations: token r32 of every block, values 8 g2 .. + 7 of every sub-step, as f16 planes
  // (HALF: token lane%16, of every pair of sub-steps the values 8 (lane/32) .. + 7 of sub-step lane/16%2)
  cq_v4u xh[TB][NX], xl[TB][NX];
  const int tcol = HALF ? lane & 15 : r32;
  const int xoff = HALF ? ((lane >> 4) & 1) * 16 + g2 * 8 : g2 * 8;
  float pow2[TB];
#pragma unroll
  for (int tb = 0; tb < TB; ++tb) {
    const float* x = p.X + (size_t)min(tb * 32 + tcol, p.T - 1) * p.H + (size_t)j0 * 16 + xoff;   // (rows past the end are not stored)
    constexpr int kApart = HALF ? 32 : 16;
    float4 v[NX][2];
#pragma unroll
    for (int j = 0; j < NX; ++j) {
      v[j][0] = *reinterpret_cast<const float4*>(x + j * kApart);
      v[j][1] = *reinterpret_cast<const float4*>(x + j * kApart + 4);
    }
    float amax = 0.f;
#pragma unroll
    for (int j = 0; j < NX; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        amax = fmaxf(fmaxf(amax, fmaxf(fabsf(v[j][h].x), fabsf(v[j][h].y))), fmaxf(fabsf(v[j][h].z), fabsf(v[j][h].w)));
    amax = fmaxf(amax, __shfl_xor(amax, 32));
    if constexpr (HALF) amax = fmaxf(amax, __shfl_xor(amax, 16));
    // (a slice of subnormal numbers is divided by the smallest normal one: undivided, its planes would all be zero)
    const uint32_t ebits = max(__float_as_uint(amax) & 0x7f800000u, 0x00800000u);
    pow2[tb] = __uint_as_float(ebits);
    const float inv = ebits == 0x7f800000u ? 1.f : 1.f / pow2[tb];   // exact: a power of two
#pragma unroll
    for (int j = 0; j < NX; ++j) {
      const float a[8] = {v[j][0].x * inv, v[j][0].y * inv, v[j][0].z * inv, v[j][0].w * inv,
                          v[j][1].x * inv, v[j][1].y * inv, v[j][1].z * inv, v[j][1].w * inv};
      uint32_t hi[4], lo[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float h0 = f16_value(a[2 * i]), h1 = f16_value(a[2 * i + 1]);
        hi[i] = f16_bits(h0) | (f16_bits(h1) << 16);
        lo[i] = f16_bits((a[2 * i] - h0) * kLoScale) | (f16_bits((a[2 * i + 1] - h1) * kLoScale) << 16);
      }
      xh[tb][j] = cq_v4u{hi[0], hi[1], hi[2], hi[3]};
      xl[tb][j] = cq_v4u{lo[0], lo[1], lo[2], lo[3]};
    }
  }
  float4* lds = reinterpret_cast<float4*>(few_lds);
  if constexpr (HALF) {
    cq_v4f acc[2], low[2];   // columns 0..15 and 16..31
    acc[0] = acc[1] = low[0] = low[1] = cq_v4f{0.f, 0.f, 0.f, 0.f};
    typedef __attribute__((ext_vector_type(2))) unsigned pair_u32;
#pragma unroll
    for (int j = 0; j < N; j += 2) {
      cq_v4u r[2][2];   // [plane][column half]
#pragma unroll
      for (int pl = 0; pl < 2; ++pl) {
        const cq_v4u f0 = __builtin_bit_cast(cq_v4u, ring[j % D][pl]), f1 = __builtin_bit_cast(cq_v4u, ring[(j + 1) % D][pl]);
        const pair_u32 w0 = __builtin_amdgcn_permlane16_swap(f0[0], f1[0], false, false);
        const pair_u32 w1 = __builtin_amdgcn_permlane16_swap(f0[1], f1[1], false, false);
        const pair_u32 w2 = __builtin_amdgcn_permlane16_swap(f0[2], f1[2], false, false);
        const pair_u32 w3 = __builtin_amdgcn_permlane16_swap(f0[3], f1[3], false, false);
        r[pl][0] = cq_v4u{w0[0], w1[0], w2[0], w3[0]};
        r[pl][1] = cq_v4u{w0[1], w1[1], w2[1], w3[1]};
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
        if (j + i + D < N) {
          ring[(j + i) % D][0] = frag[(size_t)(j + i + D) * 128];
          ring[(j + i) % D][1] = frag[(size_t)(j + i + D) * 128 + 64];
        }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        acc[h] = mfma_f16_16(r[0][h], xh[0][j / 2], acc[h]);
        low[h] = mfma_f16_16(r[1][h], xh[0][j / 2], low[h]);
        low[h] = mfma_f16_16(r[0][h], xl[0][j / 2], low[h]);
      }
    }
    // MFMA 16x16 output: register v of a lane holds column (of R) 4*(lane/16) + v, token lane%16
    auto val = [&](float a, float l) { return pow2[0] * fmaf(l, kLoUnscale, a); };
    if (__float_as_uint(pow2[0]) != 0x7f800000u) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
        lds[(wave * 2 + h) * 64 + lane] = make_float4(val(acc[h][0], low[h][0]), val(acc[h][1], low[h][1]),
                                                      val(acc[h][2], low[h][2]), val(acc[h][3], low[h][3]));
    } else {
#pragma unroll 1
      for (int i = 0; i < 8; ++i)
        few_lds[((wave * 2 + (i >> 2)) * 64 + lane) * 4 + (i & 3)] =
            few_fp32(p, nb, j0, N * 16, min(tcol, p.T - 1), (i >> 2) * 16 + (lane >> 4) * 4 + (i & 3));
    }
    __syncthreads();
    if (tid >= 128) return;
    if (tcol < p.T)
      *reinterpret_cast<float4*>(p.out + ((size_t)kz * p.T + tcol) * p.H + nb * 32 + wave * 16 + (lane >> 4) * 4) =
          few_sum(lds + tid, 128);
    return;
  }
  cq_v16f acc[TB], low[TB];
#pragma unroll
  for (int tb = 0; tb < TB; ++tb)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[tb][i] = low[tb][i] = 0.f;
#pragma unroll
  for (int j = 0; j < N && !HALF; ++j) {
    const cq_v4u rh = __builtin_bit_cast(cq_v4u, ring[j % D][0]), rl = __builtin_bit_cast(cq_v4u, ring[j % D][1]);
    if (j + D < N) {
      ring[j % D][0] = frag[(size_t)(j + D) * 128];
      ring[j % D][1] = frag[(size_t)(j + D) * 128 + 64];
    }
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
      acc[tb] = mfma_f16(rh, xh[tb][j % NX], acc[tb]);
      low[tb] = mfma_f16(rl, xh[tb][j % NX], low[tb]);
      low[tb] = mfma_f16(rh, xl[tb][j % NX], low[tb]);
    }
  }
  // MFMA 32x32 output: register v of a lane holds column (of R) 8*(v/4) + 4*(lane/32) + v%4, token lane%32
#pragma unroll
  for (int tb = 0; tb < TB; ++tb) {
    auto val = [&](int i) { return pow2[tb] * fmaf(low[tb][i], kLoUnscale, acc[tb][i]); };
    if (__float_as_uint(pow2[tb]) != 0x7f800000u) {
#pragma unroll
      for (int vb = 0; vb < 4; ++vb)
        lds[((wave * TB + tb) * 4 + vb) * 64 + lane] = make_float4(val(4 * vb), val(4 * vb + 1), val(4 * vb + 2), val(4 * vb + 3));
    } else {
#pragma unroll 1
      for (int i = 0; i < 16; ++i)
        few_lds[(((wave * TB + tb) * 4 + (i >> 2)) * 64 + lane) * 4 + (i & 3)] =
            few_fp32(p, nb, j0, N * 16, min(tb * 32 + r32, p.T - 1), (i >> 2) * 8 + g2 * 4 + (i & 3));
    }
  }
  __syncthreads();
#pragma unroll
  for (int i0 = 0; i0 < TB * 256; i0 += 64 * kFewWaves) {   // the wavefronts' sums, in their order
    const int i = i0 + tid;
    if (i >= TB * 256) break;
    const int tok = (i >> 8) * 32 + r32, vb = (i >> 6) & 3;
    if (tok < p.T)
      *reinterpret_cast<float4*>(p.out + ((size_t)kz * p.T + tok) * p.H + nb * 32 + vb * 8 + g2 * 4) =
          few_sum(lds + i, TB * 256);
  }
}

template <int N, int TB>
cq_status launch_few(const RotFewArgs& a, hipStream_t s) {
  constexpr int lds = kFewWaves * (TB == 0 ? 2048 : TB * 4096);
  static std::atomic<bool> configured{false};
  const cq_status st = cq_configure_lds(rot_few_kernel<N, TB>, lds, configured, false);
  if (st != CQ_OK) return st;
  hipLaunchKernelGGL((rot_few_kernel<N, TB>), dim3((unsigned)(a.H / 32 * a.parts)), dim3(64 * kFewWaves), lds, s, a);
  return cq_check_launch();
}

template <int N>
cq_status launch_few_tokens(const RotFewArgs& a, hipStream_t s) {
  if (a.T <= 16) return launch_few<N, 0>(a, s);
  if (a.T <= 32) return launch_few<N, 1>(a, s);
  if constexpr (N == 4) return launch_few<N, 2>(a, s);   // (more tokens: few_steps gives 4)
  return CQ_ERR_UNSUPPORTED;
}

}  // namespace

// Sub-steps of 16 k per wavefront of the kernel for few tokens, 0: not taken.  Layer of 8 small experts, fp32 kernel / this
// one, us at 1, 16 and 32 tokens: H = 1024 26.4 / 25.7, 27.4 / 26.9, 29.9 / 29.7; 2048 30.0 / 28.0, 32.3 / 30.0, 35.0 / 32.5;
// 3072 38.7 / 36.0, 43.4 / 42.0, 50.0 / 47.4; 4096 45.6 / 41.1, 49.7 / 46.0, 53.8 / 51.2.  Wider ones keep the fp32 operands: from
// 6144 on they lose (61.9 / 64.0, 67.5 / 71.8, 80.3 / 86.7; 8192 86 / 86, 91 / 95, 116 / 123), and between them the gain is 3 % and
// not at every width (4608 50.0 / 47.7, 55.7 / 53.4, 69.2 / 69.1; 5120 52.5 / 52.1, 58.4 / 59.7; 5632 56.4 / 54.6, 63.2 / 60.5).
// 33 and 64 tokens: H = 1024 31.1 / 32.2, 34.1 / 35.2; 1536 35.5 / 34.2, 40.2 / 36.8; 2560 51.4 / 48.4, 59.6 / 54.6; 4096
// 170.8 / 171.2 at 40 tokens of the Mixtral shape.  Whole layers at 1 and 16 tokens: Mixtral shape 72.8 / 67.5, 149.7 / 144.0; DeepSeek-V2-Lite shape
// 46.9 / 42.9, 85.3 / 80.0.
// Error of X_R against float64, 2-norm (and largest, of the row's maximum), fp32 kernel / this one: H = 1024 1.6e-7 / 1.2e-7
// (6.4e-7 / 4.0e-7), 2048 2.2e-7 .. 2.9e-7 / 1.2e-7 (1.1e-6 / 4.3e-7), 3072 2.5e-7 .. 3.2e-7 / 1.3e-7 (1.6e-6 / 4.0e-7), 4096
// 2.9e-7 .. 4.2e-7 / 1.5e-7 (1.5e-6 / 5.0e-7), and smaller at every width and batch.  8-bit codes that lie on the other side
// of a rounding tie than float64's, over 49 million of them at all widths: 452 / 213.  Which code of which call that is
// depends on the inputs: a single call can be further from float64 on either path.
static int few_steps(int T, int H) {
  if (H % 512 != 0 || H < 1024 || H > 4096 || T > 64) return 0;
  if (T > 32) return H >= 1536 && H < 3072 ? 4 : 0;   // (a wavefront holds the activations of T tokens x 16 n values)
  const int blocks = H / 32;
  for (int n = 16; n > 4; n /= 2)
    if (H % (16 * kFewWaves * n) == 0 && blocks * (H / (16 * kFewWaves * n)) >= 192) return n;
  return 4;
}
int cq_rotate_few_parts(int T, int H) {
  const int n = few_steps(T, H);
  return n ? H / (16 * kFewWaves * n) : 0;
}
cq_status cq_rotate_few_launch(const float* X, const void* R_split, int T, int H, float* out, hipStream_t s) {
  const RotFewArgs a = {(const uint8_t*)R_split, X, out, T, H, cq_rotate_few_parts(T, H)};
  switch (few_steps(T, H)) {
    case 16: return launch_few_tokens<16>(a, s);
    case 8: return launch_few_tokens<8>(a, s);
    case 4: return launch_few_tokens<4>(a, s);
    default: return CQ_ERR_UNSUPPORTED;
  }
}

bool cq_rotate_split_supported(int T, int H) {
  // whole column tiles and K steps in fours; enough tokens to fill tiles; 32-bit byte offsets into a plane
  return H % 256 == 0 && H >= 256 && T >= 256 && (long)T * H * 2 < (1L << 32);
}

// K parts of the layer's rotation: the tiles of 128 tokens x 256 columns are cut along K until they fill the chip, in
// parts of whole rounds of the pipeline (four steps, 256 k) that are powers of two, whose partial sums [parts][T][H] the
// quantization adds in a fixed order.  (T = 512, H = 4096: 64 tiles, one K loop of 64 steps on a quarter of the chip
// took 124 us, in four parts 52 us; T = 77: 43 us on the fp32 matrix cores, 23 us in 16 parts.)  The sum over K in parts
// is also the more accurate one: an accumulator rounds at the size of its own partial sum.  The partial sums lie where the
// layer keeps other things later.
// A launch in parts takes tiles of 64 tokens in half as many parts (narrow_parts), each of which sums the halves of its K
// range apart, so that the result is as accurate: the same products per workgroup, half the partial sums, which are written
// once and read again by the next launch, and less padding.  The launch alone is shorter only where its padding or its
// number of workgroups was worse (a workgroup's fragments of R serve half the tokens, and the second sum leaves a
// compute unit's registers to one workgroup), what is always shorter is the next launch, which reads half the sums.  This
// launch + the next one, us, tiles of 128 / 64 tokens, everything else the same: H = 4096, 128 tokens 25.2 + 9.6 / 19.2 + 9.5,
// 192 37.5 + 9.2 / 25.0 + 9.1, 384 61.4 + 11.3 / 40.0 + 11.3, 600 68.3 + 19.3 / 71.6 + 13.8, 1024 84.5 + 22.1 / 90.2 + 16.9;
// H = 2048, 129 16.4 + 12.5 / 11.1 + 12.9, 512 19.8 + 17.5 / 17.9 + 15.1, 1024 28.9 + 18.9 / 28.6 + 16.6, 2048 49.8 + 28.1 /
// 51.3 + 23.3; H = 1024, 1024 20.1 + 12.2 / 16.0 + 12.9, 4096 30.8 + 22.8 / 28.7 + 18.1.  Error of X_R against float64 over 37
// sizes the same or smaller (H = 4096, 128 tokens, where the parts did not all fit, 2.7e-7 / 2.0e-7, 77 tokens 2.09e-7 / 2.04e-7).
//
// Whether the layer's rotation takes this path: uncut from 48 tiles on, cut into parts where these make at least 44
// workgroups -- from 64 tokens on, or, narrower than 3072 columns, from a second tile of tokens, and narrower than 2048 from
// 513 tokens on.  A workgroup's K loop takes about 1.7 us per step, so a width whose K steps do not divide by 8 (an odd
// multiple of 256) stays with the fp32 kernel until it has tiles enough uncut.  Rotation and quantization, fp32 kernel
// against this one, us (workgroups of this one): H = 4096, 64 tokens 49 / 38 (256), 129..160 86 / 52; H = 3072, 96 tokens
// 40 / 40 (48), 160 59 / 42; H = 2048, 128 tokens 28 / 29 (64), 160 34 / 30 (128); H = 3840 (one part), 128 tokens 53 / 117
// (15), 256 87 / 117 (30), 300 147 / 121 (45); H = 2304 (one part), 512 tokens 72 / 80 (36), 640 95 / 81 (45); H = 2560 (two),
// 256 tokens 49 / 53 (40), 300 62 / 55 (60); H = 1024, 400 tokens 26 / 28 (64), 513 28 / 29 (80), 769 33 / 30.
// Error of X_R against float64, fp32 kernel / this path, 2-norm (and largest, of the row's maximum): H = 4096, 64 .. 256
// tokens 3.9e-7 .. 6.0e-7 / 1.9e-7 .. 2.1e-7 (1.1e-6 .. 2.2e-6 / 5.3e-7 .. 6.4e-7); H = 2048, 129 .. 600 tokens 3.2e-7 ..
// 4.7e-7 / 2.3e-7 .. 2.7e-7 (9.8e-7 .. 1.8e-6 / 6.4e-7 .. 1.1e-6).
size_t cq_rotate_split_partials_bytes(int parts, int T, int H) {
  return parts > 1 ? cq_align_up((size_t)parts * T * H * sizeof(float), 256) : 0;
}

namespace {
// full_parts: parts that fill the chip
constexpr int kFewest = 44;   // fewest workgroups of a launch in parts
long tiles(int T, int H) { return (long)((T + kTok - 1) / kTok) * (H / kCols); }
int full_parts(int T, int H) {
  int parts = 1;
  while (tiles(T, H) * parts * 2 <= 256 && (H / kStepK) % (parts * 2 * kDepth) == 0) parts *= 2;
  return parts;
}
// Launches in parts take tiles of 64 tokens, in half as many parts if these still fill the chip (they are never more).  0:
// tiles of 128 are faster.  Half as many parts of twice the tiles read R twice as often, which a wide R, far larger than the
// caches, does not give back beyond a few tiles of tokens.  Layers of 8 experts with I = 512, us, tiles of 128 / 64: H = 5120,
// 128 tokens 138 / 122, 320 172 / 168, 384 179 / 179, 512 233 / 245, 700 274 / 281; 6144, 128 157 / 141, 192 175 / 175, 256 187 /
// 193, 448 270 / 282; 7168, 128 186 / 173, 140 200 / 207, 384 300 / 321; 8192, 100 213 / 203, 140 233 / 242, 384 345 / 365;
// 4096, 256 tokens 124 / 122, 512 163 / 162, 700 216 / 215, 960 255 / 257, 1024 253 / 256 (two of the 8 experts per token: 900
// 189 / 186, 960 191 / 187, 1024 194 / 195); narrower always less.
// Where the parts stay as many the tiles only lose padding: 6144, 270 tokens 232 / 199.
int narrow_parts(int T, int H, int parts) {
  const long all = (long)((T + 63) / 64) * (H / kCols);
  if (all * parts <= 256 && all * (parts / 2) < 192) return parts;
  return H <= 3072 || T <= (H <= 4096 ? 960 : H <= 5120 ? 384 : 128) ? parts / 2 : 0;
}
bool preferred(int T, int H) {
  if (cq_rotate_split_always(T, H)) return true;
  if (H % kCols != 0 || H < 1024 || (long)T * H < (1L << 18) || (long)T * H * 2 >= (1L << 32)) return false;
  if (T < (H >= 3072 ? 64 : H >= 2048 ? kTok + 1 : 513)) return false;
  return tiles(T, H) * full_parts(T, H) >= kFewest;
}
}  // namespace

// (The parts fall as T grows, and the bytes with them: each number of parts counts with the largest T that has it.)
size_t cq_rotate_split_bytes_upto(int T, int H) {
  size_t most = 0;
  if (H % kCols != 0 || T < 64) return 0;
  for (int parts = 1; parts <= 256; parts *= 2) {
    const long last = 256 / (parts * (long)(H / kCols)) * kTok;
    const int t = parts > 1 && last < T ? (int)last : T;
    if (!preferred(t, H)) continue;   // (then no smaller batch of as many parts is, either)
    const size_t n = cq_rotate_split_workspace_bytes(t, H) + cq_rotate_split_partials_bytes(full_parts(t, H), t, H);
    if (n > most) most = n;
  }
  return most;
}

int cq_rotate_split_parts(int T, int H, size_t available, bool* narrow) {
  *narrow = false;
  if (!preferred(T, H)) return 0;
  const size_t fixed = cq_rotate_split_workspace_bytes(T, H);
  if (fixed > available) return 0;
  int parts = full_parts(T, H);
  while (parts > 1 && fixed + cq_rotate_split_partials_bytes(parts, T, H) > available) parts /= 2;
  if (!cq_rotate_split_always(T, H) && tiles(T, H) * parts < kFewest) return 0;
  const int halved = parts > 1 ? narrow_parts(T, H, parts) : 0;
  *narrow = halved > 0;
  return *narrow ? halved : parts;
}

bool cq_rotate_split_always(int T, int H) {
  return cq_rotate_split_supported(T, H) && tiles(T, H) >= 48;
}

extern "C" size_t cq_rotate_quant_split_workspace_bytes(int T, int H) {
  return T > 0 && H > 0 ? cq_rotate_split_workspace_bytes(T, H) : 0;
}

extern "C" cq_status cq_rotate_quant_split(const float* X, const void* R_split, int T, int H, int act_bits,
                                           float* XR_out, int8_t* Q_out, float* scale_out, void* workspace,
                                           size_t workspace_bytes, cq_stream stream) {
  if (!X || !R_split || !XR_out || !Q_out || !scale_out) return CQ_ERR_NULL;
  if (T <= 0 || H <= 0) return CQ_ERR_SHAPE;
  if (!cq_rotate_split_supported(T, H)) return CQ_ERR_SHAPE;
  if (act_bits != 4 && act_bits != 8) return CQ_ERR_UNSUPPORTED;
  if (!workspace || workspace_bytes < cq_rotate_split_workspace_bytes(T, H)) return CQ_ERR_WORKSPACE;
  const cq_status st = cq_rotate_split_launch(X, R_split, T, H, 1, false, XR_out, workspace, (hipStream_t)stream);
  if (st != CQ_OK) return st;
  return cq_quantize_launch(XR_out, 1, T, H, act_bits, XR_out, Q_out, nullptr, scale_out, nullptr, (hipStream_t)stream);
}

extern "C" size_t cq_rotation_split_bytes(int H) {
  return H > 0 && H % 32 == 0 ? (size_t)H * H * 4 : 0;  // two f16 planes
}

extern "C" cq_status cq_rotation_split(const float* R, int H, void* out, size_t out_bytes, cq_stream stream) {
  if (!R || !out) return CQ_ERR_NULL;
  if (H <= 0 || H % 32 != 0) return CQ_ERR_SHAPE;
  if (out_bytes < cq_rotation_split_bytes(H)) return CQ_ERR_WORKSPACE;
  const size_t frags = (size_t)(H / 32) * (H / 16);
  hipLaunchKernelGGL(split_R_kernel, dim3((unsigned)((frags + 3) / 4)), dim3(256), 0, (hipStream_t)stream, R, H,
                     (uint4*)out);
  return cq_check_launch();
}

size_t cq_rotate_split_workspace_bytes(int T, int H) {
  return cq_align_up((size_t)T * sizeof(float), 256) + 2 * cq_align_up((size_t)T * H * 2, 256);
}

// X_R = X R from the split R; XR_out [T, H] fp32.  workspace: cq_rotate_split_workspace_bytes(T, H).
// parts > 1: XR_out receives partial sums [parts][T][H].  narrow: tiles of 64 tokens.
cq_status cq_rotate_split_launch(const float* X, const void* R_split, int T, int H, int parts, bool narrow, float* XR_out,
                                 void* workspace, hipStream_t s) {
  const int tok = narrow ? 64 : kTok;
  const bool twice = narrow && H / kStepK / parts % (2 * kDepth) == 0;
  auto kern = !narrow ? rot_split_kernel<4, false> : twice ? rot_split_kernel<2, true> : rot_split_kernel<2, false>;
  static std::atomic<bool> configured[3] = {{false}, {false}, {false}};
  const int lds = rot_lds_bytes(narrow ? 2 : 4);
  const cq_status cst = cq_configure_lds(kern, lds, configured[narrow + twice], true);
  if (cst != CQ_OK) return cst;
  char* ws = (char*)workspace;
  float* row_pow2 = (float*)ws;
  uint16_t* Xh = (uint16_t*)(ws + cq_align_up((size_t)T * sizeof(float), 256));
  uint16_t* Xl = (uint16_t*)((char*)Xh + cq_align_up((size_t)T * H * 2, 256));
  hipLaunchKernelGGL(split_X_kernel, dim3(T), dim3(256), 0, s, X, T, H, Xh, Xl, row_pow2);
  RotArgs a;
  a.Rs = (const uint8_t*)R_split;
  a.Xh = Xh;
  a.Xl = Xl;
  a.row_pow2 = row_pow2;
  a.XR = XR_out;
  a.T = T;
  a.N = H;
  a.K = H;
  a.row_tiles = H / kCols;
  a.tok_tiles = (T + tok - 1) / tok;
  a.ksteps = H / kStepK / parts;
  a.n_work = a.tok_tiles * a.row_tiles * parts;
  const int per = (a.n_work + 7) / 8;
  hipLaunchKernelGGL(kern, dim3(per * 8), dim3(256), lds, s, a);
  return cq_check_launch();
}
