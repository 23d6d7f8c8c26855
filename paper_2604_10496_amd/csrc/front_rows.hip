// a2 + a3 + a4 in one launch: the K parts of the rotation are added up, the rows are quantized, the router logits are formed
// from the rows while they are in LDS, and every token's experts are selected.
//
// One workgroup of 16 wavefronts takes TPW tokens.  Separate launches (quantization, a K-split product with partial logits,
// top-k over them) read the rows again and wait for each other; what bounds this one is the router matrix, which every
// workgroup reads from L2 (64 bytes per clock and compute unit), so the tokens of a workgroup share each of its loads.
// (Requesting the first of them in front of the partial sums gained nothing; eight wavefronts instead of sixteen left too
// little in flight: 82.1 against 81.6 us at 16 tokens of 64 experts, 64.4 against 58.9 at 8 tokens of 128.)  A wavefront takes every sixteenth expert; its lanes run over the row.
// All sums have a fixed order: parts ascending; a logit over the lane's columns ascending, then a tree over the lanes.
#include "cq_internal.h"
#include "cq_quotient.h"
#include "cq_route.h"

#include <type_traits>

namespace {

constexpr int kRowsWaves = 16, kRowsThreads = 64 * kRowsWaves;
constexpr int kRowsMaxE = 128;

struct FrontRowsArgs {
  const float* part;      // [ksplit][T][H]
  int ksplit, in_place;   // in_place: the rows are X_R already
  int T, H;
  float qmax;
  const float* Wr;
  const float* bias;
  int E, top_k;
  float* XR;
  int8_t* Q;              // NULL: the rows have been quantized before
  uint16_t* Q16;
  float* scale;
  float* logits;
  int32_t* ids;
  float* w;
};

constexpr int EB = 2;   // experts of a wavefront at a time

template <int TPW>
__global__ __launch_bounds__(kRowsThreads) void front_rows_kernel(const FrontRowsArgs p) {
  extern __shared__ float4 rows[];          // [TPW][H / 4]
  __shared__ float red[TPW][kRowsWaves];
  __shared__ float s_logit[TPW][kRowsMaxE];
  __shared__ int s_id[TPW][64];
  __shared__ float s_val[TPW][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int t0 = blockIdx.x * TPW, H4 = p.H >> 2;
  // a thread has four columns of every token
  const bool mine = tid < H4;
  float4 v[TPW];
#pragma unroll
  for (int k = 0; k < TPW; ++k) {
    const int t = min(t0 + k, p.T - 1);     // (a token past the end is the last one again; nothing of it is stored)
    const float4* src = reinterpret_cast<const float4*>(p.part + (size_t)t * p.H) + min(tid, H4 - 1);
    const size_t stride = (size_t)p.T * H4;
    float4 x = src[0];
    constexpr int kAtOnce = 3;
    for (int z0 = 1; z0 < p.ksplit; z0 += kAtOnce) {
      float4 q[kAtOnce];
#pragma unroll
      for (int z = 0; z < kAtOnce; ++z) q[z] = src[(size_t)min(z0 + z, p.ksplit - 1) * stride];
#pragma unroll
      for (int z = 0; z < kAtOnce; ++z)
        if (z0 + z < p.ksplit) { x.x += q[z].x; x.y += q[z].y; x.z += q[z].z; x.w += q[z].w; }
    }
    v[k] = x;
  }
#pragma unroll
  for (int k = 0; k < TPW; ++k) {
    const float4 x = v[k];
    float amax = 0.f;
    if (mine) {
      rows[k * H4 + tid] = x;
      if (!p.in_place && t0 + k < p.T) reinterpret_cast<float4*>(p.XR + (size_t)(t0 + k) * p.H)[tid] = x;
      amax = fmaxf(fmaxf(fabsf(x.x), fabsf(x.y)), fmaxf(fabsf(x.z), fabsf(x.w)));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off));
    if (lane == 0) red[k][wave] = amax;
  }
  __syncthreads();

  // ---- integer codes: round to nearest, ties to even ----
  if (p.Q) {
#pragma unroll
    for (int k = 0; k < TPW; ++k) {
      if (t0 + k >= p.T) break;
      float amax = red[k][0];
#pragma unroll
      for (int i = 1; i < kRowsWaves; ++i) amax = fmaxf(amax, red[k][i]);
      const float s = amax == 0.f ? 1.f : amax / p.qmax;
      if (tid == 0) p.scale[t0 + k] = s;
      const cq_quotient by(s);
      auto codes = [&](auto fast) {
        const float r0 = fminf(fmaxf(rintf(by.get<decltype(fast)::value>(v[k].x)), -p.qmax), p.qmax);
        const float r1 = fminf(fmaxf(rintf(by.get<decltype(fast)::value>(v[k].y)), -p.qmax), p.qmax);
        const float r2 = fminf(fmaxf(rintf(by.get<decltype(fast)::value>(v[k].z)), -p.qmax), p.qmax);
        const float r3 = fminf(fmaxf(rintf(by.get<decltype(fast)::value>(v[k].w)), -p.qmax), p.qmax);
        reinterpret_cast<uint32_t*>(p.Q + (size_t)(t0 + k) * p.H)[tid] =
            ((uint32_t)(int)r0 & 0xffu) | (((uint32_t)(int)r1 & 0xffu) << 8) | (((uint32_t)(int)r2 & 0xffu) << 16) |
            (((uint32_t)(int)r3 & 0xffu) << 24);
        if (p.Q16)  // the same codes as bf16 bit patterns (exact: small integers)
          reinterpret_cast<uint2*>(p.Q16 + (size_t)(t0 + k) * p.H)[tid] =
              make_uint2((__float_as_uint(r0) >> 16) | (__float_as_uint(r1) & 0xffff0000u),
                         (__float_as_uint(r2) >> 16) | (__float_as_uint(r3) & 0xffff0000u));
      };
      if (!mine) continue;
      if (by.fast) codes(std::true_type{});
      else codes(std::false_type{});
    }
  }

  // ---- router logits: experts wave, wave + 16, ... ----
  for (int e0 = wave; e0 < p.E; e0 += kRowsWaves * EB) {
    const float4* wr[EB];
    float sum[EB][TPW];
#pragma unroll
    for (int u = 0; u < EB; ++u) {
      wr[u] = reinterpret_cast<const float4*>(p.Wr + (size_t)min(e0 + kRowsWaves * u, p.E - 1) * p.H);
#pragma unroll
      for (int k = 0; k < TPW; ++k) sum[u][k] = 0.f;
    }
    constexpr int kAhead = 8;   // loads of a lane per expert in flight
    for (int c0 = lane; c0 < H4; c0 += 64 * kAhead) {
      float4 b[kAhead][EB];
#pragma unroll
      for (int i = 0; i < kAhead; ++i)
#pragma unroll
        for (int u = 0; u < EB; ++u) b[i][u] = wr[u][min(c0 + 64 * i, H4 - 1)];
#pragma unroll
      for (int i = 0; i < kAhead; ++i) {
        if (c0 + 64 * i < H4) {
#pragma unroll
          for (int k = 0; k < TPW; ++k) {
            const float4 x = rows[k * H4 + c0 + 64 * i];
#pragma unroll
            for (int u = 0; u < EB; ++u)
              sum[u][k] = fmaf(x.w, b[i][u].w, fmaf(x.z, b[i][u].z, fmaf(x.y, b[i][u].y, fmaf(x.x, b[i][u].x, sum[u][k]))));
          }
        }
      }
    }
#pragma unroll
    for (int u = 0; u < EB; ++u)
#pragma unroll
      for (int k = 0; k < TPW; ++k) {
        float x = sum[u][k];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
        const int e = e0 + kRowsWaves * u;
        if (lane == 0 && e < p.E) {
          if (p.bias) x += p.bias[e];
          s_logit[k][e] = x;
        }
      }
  }
  __syncthreads();

  // ---- one wavefront per token selects its experts ----
  if (wave < TPW && t0 + wave < p.T) {
    const int t = t0 + wave;
    float val[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int e = s * 64 + lane;
      val[s] = e < p.E ? s_logit[wave][e] : 0.f;
      if (e < p.E) p.logits[(size_t)t * p.E + e] = val[s];
    }
    const size_t o = (size_t)t * p.top_k;
    if (p.E <= 64) cq_route::wave_topk_regs(val[0], p.E, p.top_k, lane, p.ids + o, p.w + o);
    else cq_route::wave_topk_regs2(val, p.E, p.top_k, lane, s_id[wave], s_val[wave], p.ids + o, p.w + o);
  }
}

template <int TPW>
cq_status launch_front_rows(const FrontRowsArgs& a, hipStream_t s) {
  hipLaunchKernelGGL((front_rows_kernel<TPW>), dim3((a.T + TPW - 1) / TPW), dim3(kRowsThreads), (size_t)TPW * a.H * 4, s, a);
  return cq_check_launch();
}

}  // namespace

// Batches that make about one round of workgroups, of one token up to 256 and of two up to 512; us per layer in separate
// launches (quantization, logits, top-k; the rotation and the grouping as they are) and so: DeepSeek-V2-Lite shape (64
// experts) 16 tokens 80.5 / 81.6, 32 tokens 100.3 / 98.7, 64 tokens 114.4 / 108.2, 128 tokens 137.3 / 130.4, 256 tokens
// 166.5 / 161.5, 512 tokens (two) 200.0 / 196.5, 1024 tokens (two) 269.6 / 275.2, (four) 270.6; Qwen3 shape (128 experts) 16
// tokens 60.8 / 64.8, 64 tokens 92.5 / 84.9, 128 tokens 116.8 / 106.7, 300 tokens (two) 140.9 / 137.3, 600 tokens 184 / 196;
// Mixtral shape (8 experts), 512 tokens 526 / 522.  Not where the router matrix is so small that its product is not what the
// launches wait for (4 experts of width 256, 512 tokens 41.8 / 43.8).
// With fewer than 64 tokens not where a workgroup has a router matrix of more than 1 MiB to read for its one token: 128
// experts of width 4096 32 and 63 tokens 104.5 / 109.0 and 119.7 / 121.9 (64 tokens 137.2 / 121.6), of width 3072 33 tokens
// 93.4 / 98.8; 128 of width 2048 75.4 / 71.0, 64 of width 4096 90.3 / 88.2 (48 tokens).  Behind the Hadamard rotation, whose
// rows are quantized already, not with more than 64 experts either: 128 of width 2048, 33 tokens 61.7 / 62.7 (64 tokens 71.5 /
// 65.7), 64 of width 4096 48 tokens 2 % less.
bool cq_front_rows_supported(int T, int H, int E, int top_k, bool quantized) {
  if (T < 32 || T > 512 || H % 64 != 0 || H > 4 * kRowsThreads || E > kRowsMaxE || top_k > 64) return false;
  if (T < 64 && ((long)E * H > (1L << 18) || (quantized && (T == 32 || E > 64)))) return false;
  return (long)E * H >= (1L << 15);
}

cq_status cq_front_rows_launch(const float* partials, int ksplit, int T, int H, int act_bits, const float* Wr, const float* bias,
                               int E, float* XR, int8_t* Q, uint16_t* Q16, float* scale, float* logits, int top_k,
                               int32_t* topk_ids, float* topk_w, hipStream_t s) {
  const FrontRowsArgs a = {partials, ksplit, partials == XR && ksplit == 1 ? 1 : 0, T, H, (float)((1 << (act_bits - 1)) - 1),
                           Wr, bias, E, top_k, XR, Q, Q16, scale, logits, topk_ids, topk_w};
  return T <= 256 ? launch_front_rows<1>(a, s) : launch_front_rows<2>(a, s);
}
