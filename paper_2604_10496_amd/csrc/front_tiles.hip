// a2 + a3 + a4 in two launches for batches of many tokens: the first adds up the K parts of the rotation and multiplies the
// rows by the router matrix while they are in LDS, the second quantizes the rows and selects every token's experts.
//
// The separate launches (quantization, a product with K-split partial logits, top-k) read the rows three times and wait for
// each other twice.  The codes need a row's maximum and the selection all of a row's logits, so one wait stays; it lies where
// nothing but the rows, the partial logits of 256 columns each and their maxima crosses it.
// A workgroup of the first launch has 32 tokens x 256 columns, so that the router matrix, which all of them read from L2, is
// read once per 32 tokens (a workgroup of front_rows.hip per 1 or 2).  fp32 MFMA of 16 tokens x 16 experts; a lane's four k of
// a 16-byte load go to four MFMAs, the same ones for both operands.  2048 tokens of width 2048, 128 experts, from a rotation in
// one part: 36.0 us in the three separate launches, 29.9 in these two (on another card 19.2 + 12.2); the product's share is 7.5
// of the first one, the rest loads that wait for one another.  (With two parts of the rotation to add up, when the first one
// took 24 us: four wavefronts with 16 columns' loads each in flight and both blocks of experts in turn 28.7.)
// All sums have a fixed order: parts ascending; a partial logit in the order of the MFMAs (of up to 32 experts: in eighths of
// the columns, added in pairs); 256-column blocks ascending.
#include "cq_internal.h"
#include "cq_quotient.h"
#include "cq_route.h"

#include <type_traits>

namespace {

constexpr int kTokens = 32;      // of a workgroup
constexpr int kColumns = 256;    // ... of the rows
constexpr int kStride = kColumns + 4;   // floats: the 16 rows of a fragment read hit 16 different groups of four banks
constexpr int kMaxE = 128;

struct FrontTilesArgs {
  const float* part;     // [ksplit][T][H]
  int ksplit, in_place;  // in_place: the rows are X_R already
  int T, H, E, top_k;
  float qmax;
  const float* Wr;
  const float* bias;
  float* XR;
  float* lp;             // [H / 256][T][E] partial logits
  float* amax;           // [H / 256][T] maxima of 256 columns
  int8_t* Q;
  uint16_t* Q16;
  float* scale;
  float* logits;
  int32_t* ids;
  float* w;
};

constexpr int kWaves = 8;
// How the wavefronts share the product: all columns of one block of 16 experts each, with both halves of the tokens (more
// than 64 experts) or one of them (up to 64), or an eighth of the columns each (up to 32 experts).
enum { kBlockBoth, kBlockHalf, kByColumns };

template <int SHARE>
__global__ __launch_bounds__(64 * kWaves, 4) void logits_tiles_kernel(const FrontTilesArgs p) {
  __shared__ float xs[kTokens * kStride];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15, g = lane >> 4;
  const int t0 = blockIdx.x * kTokens, c0 = blockIdx.y * kColumns;
  const int nb = (p.E + 15) >> 4;          // blocks of 16 experts
  constexpr bool kCols = SHARE == kByColumns;
  const int block = SHARE == kBlockBoth ? wave : wave & 3;   // (kByColumns: both blocks)
  // the router rows' loads, 16 columns of a block each: the first eight in front of everything else
  constexpr int kSteps = kCols ? 4 : kColumns / 16, kRing = kCols ? 4 : 8;
  float4 b[kRing];
  auto load_b = [&](int s) {
    const int e = min((kCols ? s >> 1 : block) * 16 + j, p.E - 1);
    const int col = c0 + (kCols ? wave * 32 + (s & 1) * 16 : s * 16);
    b[s % kRing] = *reinterpret_cast<const float4*>(p.Wr + (size_t)e * p.H + col + 4 * g);
  };
#pragma unroll
  for (int s = 0; s < kRing; ++s) load_b(s);
  // ---- a wavefront's four rows: sums of the parts, X_R, maxima ----
  constexpr int kRows = kTokens / kWaves;
  float4 v[kRows];
  const float* src[kRows];
#pragma unroll
  for (int i = 0; i < kRows; ++i) {        // (a token past the end is the last one again; nothing of it is stored)
    src[i] = p.part + (size_t)min(t0 + wave * kRows + i, p.T - 1) * p.H + c0 + lane * 4;
    v[i] = *reinterpret_cast<const float4*>(src[i]);
  }
  constexpr int kAtOnce = 3;               // parts whose loads are in flight together
  for (int z0 = 1; z0 < p.ksplit; z0 += kAtOnce) {
    float4 q[kAtOnce][kRows];
#pragma unroll
    for (int z = 0; z < kAtOnce; ++z)
#pragma unroll
      for (int i = 0; i < kRows; ++i)
        q[z][i] = *reinterpret_cast<const float4*>(src[i] + (size_t)min(z0 + z, p.ksplit - 1) * p.T * p.H);
#pragma unroll
    for (int z = 0; z < kAtOnce; ++z)
      if (z0 + z < p.ksplit)
#pragma unroll
        for (int i = 0; i < kRows; ++i) { v[i].x += q[z][i].x; v[i].y += q[z][i].y; v[i].z += q[z][i].z; v[i].w += q[z][i].w; }
  }
  float m[kRows];
#pragma unroll
  for (int i = 0; i < kRows; ++i) {
    const int r = wave * kRows + i;
    if (!p.in_place && t0 + r < p.T) *reinterpret_cast<float4*>(p.XR + (size_t)(t0 + r) * p.H + c0 + lane * 4) = v[i];
    *reinterpret_cast<float4*>(xs + r * kStride + lane * 4) = v[i];
    m[i] = fmaxf(fmaxf(fmaxf(0.f, fabsf(v[i].x)), fabsf(v[i].y)), fmaxf(fabsf(v[i].z), fabsf(v[i].w)));
  }
  // four maxima over 64 lanes: two exchanges halve the number of rows a lane has, four more finish its one row
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const bool up = lane & 32;
    m[i] = fmaxf(up ? m[i + 2] : m[i], __shfl_xor(up ? m[i] : m[i + 2], 32));
  }
  {
    const bool up = lane & 16;
    m[0] = fmaxf(up ? m[1] : m[0], __shfl_xor(up ? m[0] : m[1], 16));
  }
#pragma unroll
  for (int off = 8; off > 0; off >>= 1) m[0] = fmaxf(m[0], __shfl_xor(m[0], off));
  {
    const int t = t0 + wave * kRows + ((lane >> 5) & 1) * 2 + ((lane >> 4) & 1);
    if ((lane & 15) == 0 && t < p.T) p.amax[(size_t)blockIdx.y * p.T + t] = m[0];
  }
  __syncthreads();
  // ---- partial logits ----
  // (four accumulators, one per component of the loads: sixteen products one after the other in each, no result that the
  // next MFMA waits for, and a smaller error than one chain of 64)
  auto product = [&](cq_v4f (&acc)[4], int h, int s, int col) {
    const float4 x = *reinterpret_cast<const float4*>(xs + (16 * h + j) * kStride + col + 4 * g);
    const float4 w = b[s % kRing];
    acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.x, w.x, acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.y, w.y, acc[1], 0, 0, 0);
    acc[2] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.z, w.z, acc[2], 0, 0, 0);
    acc[3] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.w, w.w, acc[3], 0, 0, 0);
  };
  auto total = [](const cq_v4f (&a)[4], int i) { return (a[0][i] + a[1][i]) + (a[2][i] + a[3][i]); };
  // (of an MFMA's result a lane has expert j of tokens 4g .. 4g+3)
  auto store = [&](int h, int i, int e, float x) {
    const int t = t0 + 16 * h + 4 * g + i;
    if (t < p.T && e < p.E) p.lp[((size_t)blockIdx.y * p.T + t) * p.E + e] = x;
  };
  if constexpr (kCols) {
    cq_v4f acc[2][2][4] = {};
#pragma unroll
    for (int s = 0; s < kSteps; ++s)
#pragma unroll
      for (int h = 0; h < 2; ++h) product(acc[s >> 1][h], h, s, wave * 32 + (s & 1) * 16);
    __syncthreads();   // (the rows have been read: their place takes the wavefronts' sums)
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < 4; ++i) xs[(wave * 16 + k * 8 + h * 4 + i) * 64 + lane] = total(acc[k][h], i);
    __syncthreads();
    // a wavefront adds up two of the sixteen values of a lane
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int at = wave * 2 + u;         // (k, h, i) as stored
      float x[kWaves];
#pragma unroll
      for (int z = 0; z < kWaves; ++z) x[z] = xs[(z * 16 + at) * 64 + lane];
      store((at >> 2) & 1, at & 3, (at >> 3) * 16 + j, ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7])));
    }
  } else {
    constexpr int kHalves = SHARE == kBlockBoth ? 2 : 1;
    if (block >= nb) return;
    const int h0 = SHARE == kBlockBoth ? 0 : wave >> 2;
    cq_v4f acc[kHalves][4] = {};
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
#pragma unroll
      for (int h = 0; h < kHalves; ++h) product(acc[h], h0 + h, s, s * 16);
      if (s + kRing < kSteps) load_b(s + kRing);
    }
#pragma unroll
    for (int h = 0; h < kHalves; ++h)
#pragma unroll
      for (int i = 0; i < 4; ++i) store(h0 + h, i, block * 16 + j, total(acc[h], i));
  }
}

// One workgroup per token: codes of the row, whose maximum is known, and (first wavefront) the token's experts.
// NV: groups of four columns per thread; NSLOT: experts per lane.
template <int NV, int NSLOT>
__global__ __launch_bounds__(256) void quantize_topk_kernel(const FrontTilesArgs p) {
  __shared__ int s_id[64];
  __shared__ float s_val[64];
  const int t = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int nc = p.H / kColumns;
  float4 v[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = min((i * 256 + tid) * 4, p.H - 4);   // (columns past the end: the last ones again, not kept)
    v[i] = *reinterpret_cast<const float4*>(p.XR + (size_t)t * p.H + c);
  }
  float amax = p.amax[(size_t)min(lane, nc - 1) * p.T + t];   // (at most 32 blocks)
  if (tid < 64) {
    float val[NSLOT];
#pragma unroll
    for (int s = 0; s < NSLOT; ++s) {
      const int e = s * 64 + lane;
      val[s] = 0.f;
      if (e < p.E) {
        const float* src = p.lp + (size_t)t * p.E + e;
        float x = src[0];
        constexpr int kAtOnce = NV >= 4 ? 15 : 7;
        for (int z0 = 1; z0 < nc; z0 += kAtOnce) {
          float q[kAtOnce];
#pragma unroll
          for (int i = 0; i < kAtOnce; ++i) q[i] = src[(size_t)min(z0 + i, nc - 1) * p.T * p.E];
#pragma unroll
          for (int i = 0; i < kAtOnce; ++i)
            if (z0 + i < nc) x += q[i];
        }
        if (p.bias) x += p.bias[e];
        p.logits[(size_t)t * p.E + e] = x;
        val[s] = x;
      }
    }
    const size_t o = (size_t)t * p.top_k;
    if constexpr (NSLOT == 1) cq_route::wave_topk_regs(val[0], p.E, p.top_k, lane, p.ids + o, p.w + o);
    else cq_route::wave_topk_regs2(val, p.E, p.top_k, lane, s_id, s_val, p.ids + o, p.w + o);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off));
  const float s = amax == 0.f ? 1.f : amax / p.qmax;
  if (tid == 0) p.scale[t] = s;
  const cq_quotient by(s);
  auto codes = [&](auto fast) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int c = (i * 256 + tid) * 4;
      if (c >= p.H) break;
      const float r0 = fminf(fmaxf(rintf(by.get<decltype(fast)::value>(v[i].x)), -p.qmax), p.qmax);
      const float r1 = fminf(fmaxf(rintf(by.get<decltype(fast)::value>(v[i].y)), -p.qmax), p.qmax);
      const float r2 = fminf(fmaxf(rintf(by.get<decltype(fast)::value>(v[i].z)), -p.qmax), p.qmax);
      const float r3 = fminf(fmaxf(rintf(by.get<decltype(fast)::value>(v[i].w)), -p.qmax), p.qmax);
      *reinterpret_cast<uint32_t*>(p.Q + (size_t)t * p.H + c) =
          ((uint32_t)(int)r0 & 0xffu) | (((uint32_t)(int)r1 & 0xffu) << 8) | (((uint32_t)(int)r2 & 0xffu) << 16) |
          (((uint32_t)(int)r3 & 0xffu) << 24);
      if (p.Q16)  // the same codes as bf16 bit patterns (exact: small integers)
        *reinterpret_cast<uint2*>(p.Q16 + (size_t)t * p.H + c) =
            make_uint2((__float_as_uint(r0) >> 16) | (__float_as_uint(r1) & 0xffff0000u),
                       (__float_as_uint(r2) >> 16) | (__float_as_uint(r3) & 0xffff0000u));
    }
  };
  if (by.fast) codes(std::true_type{});
  else codes(std::false_type{});
}

template <int NV>
void launch_second(const FrontTilesArgs& a, hipStream_t s) {
  if (a.E <= 64) hipLaunchKernelGGL((quantize_topk_kernel<NV, 1>), dim3(a.T), dim3(256), 0, s, a);
  else hipLaunchKernelGGL((quantize_topk_kernel<NV, 2>), dim3(a.T), dim3(256), 0, s, a);
}

}  // namespace

// From 64 tokens on where front_rows.hip does not take the batch: more than 512 tokens, H > 4096 or small router matrices.  us
// per layer (I = 512, everything else the same) in separate launches / so: 128 experts of width 2048, 600 tokens 149.0 / 137.7,
// 1024 179.6 / 167.2, 2048 282.5 / 276.8; 64 of 2048, 600 112.1 / 106.4, 2048 228.4 / 220.4; 33 of 768, 64 50.2 / 46.0, 1500
// 87.6 / 82.2; 32 of 2048, 600 97.9 / 91.9, 2048 179.3 / 171.5; 32 of 4096, 2048 407.4 / 394.3; 20 of 8192, 200 221.0 / 206.0, 1000
// 567.1 / 560.2; 16 of 1024, 600 69.7 / 65.8, 4096 153.7 / 152.7; 16 of 4096, 600 178.3 / 176.5, 2048 369.3 / 368.2.  Up to 8 experts,
// whose separate product is the cheapest: 8 of 1024, 600 67.7 / 64.2, 1024 75.6 / 76.2, 4096 112.2 / 111.1; 8 of 2048, 600
// 93.1 / 93.3, 1500 120.3 / 118.6, 3000 182.1 / 180.3, 4096 222.0 / 225.4; 8 of 4096, 600 163.0 / 161.2, 1024 196.4 / 195.2, 2048
// 307.1 / 309.3, 4096 567.3 / 567.8.  From 2^21 values on these are within 1.5 % of each other either way, and come here for the
// logits' accuracy (below).  Up to 512 tokens front_rows.hip is as fast or faster: 64 experts of width 2048 200 tokens 150.4 /
// 153.2, 400 tokens 171.7 / 171.2.
// The logits' error against float64 (2-norm, with that of X_R) is smaller than the separate product's: 3.4e-7 / 3.1e-7 at 600
// tokens of 64 and 128 experts; 8 experts, 6.5e-7 / 5.2e-7 at 4096 tokens of width 2048, 8.3e-7 / 7.3e-7 at 2048 and 9.1e-7 / 7.2e-7 at
// 4096 tokens of width 4096; 2.5e-7 / 2.2e-7 at 600 of width 1024.
bool cq_front_tiles_supported(int T, int H, int E, int top_k) {
  return T >= 64 && H % kColumns == 0 && H <= 32 * kColumns && E <= kMaxE && top_k <= 64;
}

size_t cq_front_tiles_bytes(int T, int H, int E) {
  return cq_align_up((size_t)(H / kColumns) * T * E * 4, 256) + (size_t)(H / kColumns) * T * 4;
}

cq_status cq_front_tiles_launch(const float* partials, int ksplit, int T, int H, int act_bits, const float* Wr, const float* bias,
                                int E, float* XR, int8_t* Q, uint16_t* Q16, float* scale, float* logits, int top_k,
                                int32_t* topk_ids, float* topk_w, void* workspace, hipStream_t s) {
  float* lp = (float*)workspace;
  float* amax = (float*)((char*)workspace + cq_align_up((size_t)(H / kColumns) * T * E * 4, 256));
  const FrontTilesArgs a = {partials, ksplit, partials == XR && ksplit == 1 ? 1 : 0, T, H, E, top_k,
                            (float)((1 << (act_bits - 1)) - 1), Wr, bias, XR, lp, amax, Q, Q16, scale, logits, topk_ids, topk_w};
  const dim3 grid((T + kTokens - 1) / kTokens, H / kColumns);
  auto first = E <= 32 ? logits_tiles_kernel<kByColumns> : E <= 64 ? logits_tiles_kernel<kBlockHalf> : logits_tiles_kernel<kBlockBoth>;
  hipLaunchKernelGGL(first, grid, dim3(64 * kWaves), 0, s, a);
  const cq_status st = cq_check_launch();
  if (st != CQ_OK) return st;
  if (H <= 1024) launch_second<1>(a, s);
  else if (H <= 2048) launch_second<2>(a, s);
  else if (H <= 4096) launch_second<4>(a, s);
  else launch_second<8>(a, s);
  return cq_check_launch();
}
