// a6 / a7 for groups with many tokens (prefill regime, bound by the matrix cores).
//
// Workgroup tile: 256 weight rows x CT tokens (CT = 256, 128, 96, 64 or 32), four wavefronts, each owning 64 rows
// and ALL the tile's tokens (accumulators 2 x CT/32 MFMA blocks of 32x32).  Consequences:
//   * every wavefront decodes only its own rows, straight into MFMA A-operand registers: the decoded
//     weights never touch LDS, and no weight is decoded twice;
//   * a lane owns one row of each of its two 32-row blocks for the whole K loop, so the two 16-entry
//     centroid tables it needs are loop invariant and live in registers.  Decoding is pure vector ALU:
//     nibbles become byte selectors, v_perm_b32 picks the low and the high bytes of the centroids out
//     of register-resident byte tables (two 8-entry halves, xored: cq_decode.h), one or two more perm levels
//     interleave the bytes into bf16/f16 pairs.
//     About 1.3 ALU operations per MFMA at 256 tokens, mostly hidden behind the matrix pipe (with two wavefronts on a
//     SIMD v_perm_b32 and the other three-operand operations take 4.4 clocks, two-operand ones 2.7, an MFMA about 8 of the
//     issue beside six or more of them: 168 operations per step and wavefront).  What the launches wait for is power: the
//     clock falls from 2.3 GHz for 64 workgroups to 1.5..1.9 for 512, four wavefronts per SIMD instead of two (32 rows
//     each) take fewer clocks and the same time, and activations of zero 10 to 21 % less of it;
//     With block-wise tables (one per group of g weights along K, g a multiple of 512) the two tables are
//     replaced every g/64 steps; the raw tables of the next group are requested one group ahead;
//   * LDS holds only the activation tiles.  They arrive by direct global->LDS loads (no staging
//     registers, no ds_write), four tiles deep, and each wavefront reads a tile once per K step.
// The activation operand is 16-bit (bf16 integer codes or f16 rows); other kinds are converted by a
// small pre-pass.  The token tiles are derived in the kernel from the group offsets (groups are ragged and their sizes
// are only known on the device); the work index is remapped so that tiles sharing activations run on
// the same XCD (L2).
#include <type_traits>

#include "cq_internal.h"
#include "cq_async.h"
#include "cq_decode.h"
#include "cq_route.h"

namespace {

constexpr int kLargeRows = 256;  // weight rows per workgroup
constexpr int kStepK = 64;       // K per pipeline step
constexpr int kStepBytes = kStepK * 2;  // one token's share of a step in LDS and in global memory
// tokens of the tiles of the three widths: whole tiles (one workgroup per compute unit), half tiles (two)
template <bool HALF>
struct tile_widths {
  static constexpr int w0 = HALF ? 128 : 256, w1 = HALF ? 96 : 128, w2 = 64;
};
constexpr int kAtOnce[2] = {256, 512};   // workgroups that the chip runs at a time
constexpr int kNextTableBytes = 2048;  // block-wise tables: raw next tables of a wavefront's 64 rows (x 4 wavefronts x 2)

struct LargeArgs {
  const uint8_t* idx;
  const uint16_t* cent;
  int prepacked;
  int N, K;
  const uint16_t* A;           // [rows, K] bf16 or f16
  const int32_t* a_gather;     // sorted row -> row of A, or NULL
  const float* row_scale;
  const int32_t* scale_gather; // sorted row -> entry of row_scale, or NULL
  void* out;
  int out_ld;
  const int32_t* group_offsets;   // [G + 1]
  int G;
  int small_max;          // groups with at most this many rows are left to the streaming kernel
  int row_tiles;          // N / 256
  int nblk;               // centroid tables per weight row (1: one table over all of K)
  int gsteps;             // K steps per table (block-wise tables: group size / 64, a multiple of 8)
  // K split (block-wise tables, plain products of few rows): workgroups with blockIdx.y = z take the K steps
  // [z * ksteps, (z+1) * ksteps), a whole number of table groups, and store fp32 partial sums at
  // out + z * part_stride elements; ksteps covers all of K when there is no split
  int ksteps;
  size_t part_stride;
  // K split of the tiles of a plain fp32 product with a long K (tail_part != NULL): the tiles of the two narrow widths
  // w1 and w2, which come last, are cut into kS1 parts in {1, 2, 4} (tile_map); split z > 0 of the j-th w1-token
  // (w2-token) tile stores its partial sums at rows j*w1 (tail_rows1 + j*w2) of slice z-1 of tail_part,
  // [kS1-1][tail_rows][N] fp32 -- or, when the launch has fewer rows than such slots (tail_abs), at the tile's own sorted
  // rows; the widest tiles then come in kS0 parts.  tail_sum_kernel adds the slices to `out` in the order z = 1, 2, ...
  float* tail_part;
  int w0, w1, w2;     // the three widths of the launch
  int at_once;        // workgroups of it that the chip runs at a time
  int tail_rows1;     // rows reserved for the w1-token tiles (capacity of that list * w1)
  int tail_rows;      // rows per slice
  int tail_abs;       // 1: a slice has M_total rows and a tile stores at its own sorted rows (fewer rows than slots)
};

#ifndef CQ_TAIL_SPLIT_MAX
#define CQ_TAIL_SPLIT_MAX 4
#endif
constexpr int kTailSplitMax = CQ_TAIL_SPLIT_MAX;   // most K parts a narrow tile is cut into (1: never)
constexpr int kTailMinSteps = 128;   // K steps (of 64) from which the narrow tiles of a plain product may be split

__device__ __forceinline__ uint32_t f32_to_f16_sat(float x) {
  x = fminf(fmaxf(x, -65504.f), 65504.f);
  const _Float16 h = (_Float16)x;
  return (uint32_t) __builtin_bit_cast(uint16_t, h);
}
__device__ __forceinline__ uint32_t code_bf16(int c) { return __float_as_uint((float)c) >> 16; }

template <bool F16>
__device__ __forceinline__ cq_v16f mfma_large(const cq_v4u a, const cq_v4u b, cq_v16f c) {
  if constexpr (F16)
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(cq_v8f16, a), __builtin_bit_cast(cq_v8f16, b), c,
                                                  0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(cq_v8bf16, a),
                                                   __builtin_bit_cast(cq_v8bf16, b), c, 0, 0, 0);
}

using namespace cq_async;

// LDS row stride (bytes) of the epilogue's staging tile of 64 tokens x the workgroup's output columns
constexpr int epilogue_row_stride(int epi, int outk) {
  const int esize = outk == CQ_OUT_F16 ? 2 : 4;
  const int row = (epi == CQ_EPI_SWIGLU ? kLargeRows / 2 : kLargeRows) * esize;
  const int quad = (epi == CQ_EPI_SWIGLU ? 2 : 4) * esize;
  return row + (quad == 16 ? 16 : 8);
}

// One tile: 128 * RB weight rows (row tile rt of that height) x up to 32*C tokens (rows mrow0 .. mrow0+mcnt-1 of group
// grp); each wavefront owns RB blocks of 32 rows.
// F16: the activations are f16 (else bf16); C = CT/32 token blocks (8, 4, 3, 2 or 1); D = depth of the load
// pipeline in K steps (a power of two; narrow tiles spend less matrix time per step and need more).
// BLK: block-wise centroid tables (p.nblk per row, each serving p.gsteps K steps).  PRE: the indices are the
// prepacked copy (whose nibble arrangement decodes with four operations fewer per 8 weights).
// kz / kS: this workgroup takes part kz of kS equal parts of K (narrow tiles of a plain fp32 product; 0 / 1
// otherwise) and, for kz > 0, stores at row tail_row0 of slice kz-1 of p.tail_part instead of p.out.
template <bool F16, int EPI, int OUTK, int C, int D, bool BLK, bool PRE, bool A32 = false, int RB = 2>
__device__ __forceinline__ void large_tile(const LargeArgs& p, const int grp_, const int mrow0_, const int mcnt_,
                                           const int rt_, const int kz_ = 0, const int kS_ = 1, const int tail_row0 = 0) {
  // (uniform, but derived per work item: kept in scalar registers from here on)
  const int grp = __builtin_amdgcn_readfirstlane(grp_), mrow0 = __builtin_amdgcn_readfirstlane(mrow0_);
  const int mcnt = __builtin_amdgcn_readfirstlane(mcnt_), rt = __builtin_amdgcn_readfirstlane(rt_);
  const int kz = __builtin_amdgcn_readfirstlane(kz_), kS = __builtin_amdgcn_readfirstlane(kS_);
  constexpr bool kTail = !BLK && EPI == CQ_EPI_NONE && OUTK == CQ_OUT_F32;
  constexpr int CT = 32 * C;
  constexpr int kRows = 128 * RB;
  static_assert(RB == 2 || (RB == 1 && !BLK), "tiles of 128 rows have one table per row");
  constexpr uint32_t kBufBytes = CT * kStepBytes;  // one activation tile: CT tokens x 128 bytes

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: what depends on it stays scalar
  const int r32 = lane & 31, g2 = lane >> 5;
  const int N = p.N, K = p.K;
  const size_t rowbytes = (size_t)K >> 1;
  const int n0 = rt * kRows + wave * (32 * RB);  // this wavefront's rows
  // index loads: a uniform base per row block and step, plus this lane's offset of its 16 bytes (of row r32 of the block)
  const uint8_t* wp0 = p.idx + ((size_t)grp * N + n0) * rowbytes;
  const uint8_t* wp1 = wp0 + 32 * rowbytes;
  const uint32_t woff = PRE ? (uint32_t)lane * 16u : (uint32_t)r32 * (uint32_t)rowbytes + (uint32_t)g2 * 16u;
  constexpr int sstride = PRE ? 1024 : 32;
  // this workgroup's K range: steps [sb, sb + nS) (all of K unless the launch splits K)
  int sb = BLK ? (int)blockIdx.y * p.ksteps : 0;
  int nS = BLK ? min(p.ksteps, K / kStepK - sb) : K / kStepK;
  if constexpr (kTail) {
    if (kS > 1) {   // equal parts of an even number of steps (the last one takes what is left: at least two)
      const int per = ((nS + kS - 1) / kS + 1) & ~1;
      sb = kz * per;
      nS = min(per, nS - sb);
    }
  }
  if constexpr (BLK || kTail) {
    wp0 += (size_t)sb * sstride;
    wp1 += (size_t)sb * sstride;
  }

  const int nblk = BLK ? p.nblk : 1;
  const uint16_t* cgrp = p.cent + (size_t)grp * N * nblk * CQ_N_CENTROIDS;   // this group's tables (uniform)
  const int blk0 = BLK ? sb / p.gsteps : 0;                                     // first table group of the K range
  const uint32_t crow_off = ((uint32_t)(n0 + r32) * nblk + blk0) * (CQ_N_CENTROIDS * 2);  // row r32's first table, bytes
  const uint32_t crow_skip = 32u * nblk * (CQ_N_CENTROIDS * 2);                // from row r32 to row 32 + r32
  RowTable tab[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
    tab[rb] = make_row_table<F16>(
        reinterpret_cast<const uint16_t*>(reinterpret_cast<const uint8_t*>(cgrp) + crow_off + rb * crow_skip));
  // Block-wise tables: the raw centroids of the next group of weights wait in LDS above the activation
  // tiles, 2 KiB per wavefront and parity of the group (two direct-to-LDS loads: lane (r32, g2) moves half
  // g2 of the 32-byte table of row r32, then of row 32 + r32), and become register tables when that group
  // starts.  Nothing but one byte offset per lane stays in registers meanwhile.
  int blk_next = 1;            // group (counted from the range's first) whose tables were requested last
  int switch_at = p.gsteps;    // first K step of that group
  const uint32_t tbl_lds = __builtin_amdgcn_readfirstlane(D * kBufBytes + wave * kNextTableBytes);  // above the ring
  auto fetch_tables = [&](int b) {
    // (clamped to the row's last table)
    const uint8_t* src = reinterpret_cast<const uint8_t*>(cgrp) + (size_t)min(b, nblk - 1 - blk0) * (CQ_N_CENTROIDS * 2);
    const uint32_t at = tbl_lds + (b & 1) * (4 * kNextTableBytes);
    const uint32_t lane_off = crow_off + g2 * 16;
    load_global_to_lds_s<0>(at, src, lane_off);
    load_global_to_lds_s<0>(at + 1024, src, lane_off + crow_skip);
  };

  // ---- activation tiles ----
  // LDS tile: token-major, 128 bytes (8 chunks of 8 k) per token; chunk c of token t sits at position
  // c ^ ((t >> 1) & 7) of the token's row.  With that swizzle the 16 lanes of one phase of a fragment
  // read (16 consecutive tokens, same chunk) hit 16 different 16-byte bank groups.
  // Transfer: one direct-to-LDS load moves 8 tokens x 128 bytes (8 lanes per token: whole contiguous
  // row segments on the global side, 1 KiB contiguous in LDS).  The swizzle is applied on the global
  // side: lane (token, position) fetches chunk position ^ ((token >> 1) & 7).  Wavefront w moves
  // tokens [w*CT/4, (w+1)*CT/4) of every step: C loads.
  // Tokens past the end of the tile load the tile's last row instead (no branches in the pipeline);
  // a token is one output column, and those columns are never stored.
  // (A32: the launcher knows that every row's byte offset fits 32 bits; the address arithmetic is then scalar)
  const uint8_t* ap[A32 ? 1 : C];
  uint32_t aoff[A32 ? C : 1];
  const uint8_t* const abase = reinterpret_cast<const uint8_t*>(p.A) + (size_t)sb * kStepK * 2;
#pragma unroll
  for (int i = 0; i < C; ++i) {
    const int tok = wave * (CT / 4) + i * 8 + (lane >> 3);
    const int m = mrow0 + min(tok, mcnt - 1);
    const size_t row = (size_t)(p.a_gather ? p.a_gather[m] : m);
    const int chunk = (lane & 7) ^ ((tok >> 1) & 7);
    if constexpr (A32) aoff[i] = (uint32_t)((row * (size_t)K + chunk * 8) * 2);
    else ap[i] = abase + (row * (size_t)K + chunk * 8) * 2;
  }
  const uint32_t lds_wave = __builtin_amdgcn_readfirstlane(wave * (CT / 4) * kStepBytes);
  // this wavefront's loads i0 .. i0+n-1 of the activations of step s into tile `buf`
  auto fetch_tile = [&](int s, int buf, int i0, int n) {
    const size_t o = (size_t)s * kStepBytes;
#pragma unroll
    for (int i = 0; i < C; ++i)
      if (i >= i0 && i < i0 + n) {
        if constexpr (A32) load_global_to_lds_s<0>(buf * kBufBytes + lds_wave + i * 1024, abase + o, aoff[i]);
        else load_global_to_lds(buf * kBufBytes + lds_wave + i * 1024, ap[i] + o);
      }
  };
  auto fetch_weights = [&](cq_v4u (&w)[RB], int s) {
    const size_t o = (size_t)s * sstride;
    load_global_async_s<0>(w[0], wp0 + o, woff);
    if constexpr (RB == 2) load_global_async_s<0>(w[1], wp1 + o, woff);
  };
  // fragment read: lane (token r32 of block cb, k group g2) wants chunk g2*4 + jj of sub-step jj
  const uint32_t boff = (uint32_t)r32 * kStepBytes + ((uint32_t)((g2 * 4) ^ ((r32 >> 1) & 7)) << 4);
  // One address register per sub-step (and per 64 KiB of tiles), opaque to the compiler; buffer and token block go into
  // the instruction's offset field.  (Left to itself the compiler keeps up to 48 loop-invariant addresses in registers,
  // which half tiles do not have: 13 to 28 spilled.)
  constexpr int kBufSets = (int)((D * kBufBytes + 65535) / 65536), kSetBufs = D / kBufSets;
  uint32_t bx[kBufSets][4];
#pragma unroll
  for (int jj = 0; jj < 4; ++jj)
#pragma unroll
    for (int i = 0; i < kBufSets; ++i) {
      bx[i][jj] = (boff ^ ((uint32_t)jj << 4)) + i * kSetBufs * kBufBytes;
      asm volatile("" : "+v"(bx[i][jj]));
    }
  auto read_b = [&](int buf, int jj, int cb) {
    return lds_read_u128(bx[buf / kSetBufs][jj] + (uint32_t)(buf % kSetBufs) * kBufBytes + cb * 32 * kStepBytes);
  };

  cq_v16f acc[RB][C];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int cb = 0; cb < C; ++cb)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[rb][cb][i] = 0.f;

  // Pipeline: at the start of step s the weights and the activation tile of step s+D-1 are requested
  // (weights: ring of D register pairs; tiles: ring of D LDS buffers, tile s in buffer s%D).  At the
  // end of step s every wavefront waits for its own share of tile s+2 (the loads of the D-3 steps
  // requested after it may stay in flight), then the workgroup barrier publishes it; the last sub-step
  // of step s+1 already reads from it.  The barrier also retires tile s, which the requests of step
  // s+1 overwrite.  Loads thus have D-2 full steps to arrive (two steps = about 2 us for 256 tokens).
  // vector-memory loads a wavefront issues per step: the wait counts below depend on it
  constexpr int kPerStep = C + RB;  // C tile loads + RB weight loads
  constexpr int kInFlight = (D - 3) * kPerStep;
  static_assert(D >= 4 && (D & (D - 1)) == 0 && kInFlight < 64, "ring depth / vmcnt range");
  static_assert(2 * kPerStep > 2 && kInFlight + kPerStep + 2 < 64,
                "the waits of D - 1 steps retire the table loads before they are used");
  cq_v4u wq[D][RB];
#pragma unroll
  for (int i = 0; i < D - 1; ++i) {
    // (block-wise tables: the first request for tables sits where the loop's requests will sit, in front
    // of the last step requested ahead -- the wait counts below are the same in every pass)
    if constexpr (BLK) {
      if (i == D - 2) fetch_tables(1);
    }
    fetch_weights(wq[i], min(i, nS - 1));
    fetch_tile(min(i, nS - 1), i, 0, C);
  }
  if constexpr (RB == 2) vm_wait<kInFlight>(wq[0][0], wq[0][1], wq[1][0], wq[1][1]);
  else vm_wait<kInFlight>(wq[0][0], wq[1][0]);
  __syncthreads();

  // Software pipeline over the 16-wide K sub-steps.  While the matrix cores work through the 2*C MFMAs
  // of one sub-step, the vector ALU decodes the A fragments of the next one and LDS delivers its B
  // fragments (a wavefront issues in order, so the pipes only overlap if their instructions alternate;
  // the group barriers below ask the scheduler for exactly that).
  // The B fragments live in one register set: as soon as the two MFMAs of a token block are issued,
  // its registers take the block's fragment of the next sub-step (a full sub-step of slack).
  // vector ALU operations per MFMA that the scheduler is asked for: in half tiles a decode8 call per C MFMAs and row block.  (Whole
  // tiles have no second workgroup on the compute unit whose products could run under the decoding: four per MFMA also
  // where the tile is narrow; block-wise tables, gate/up + down at 96 tokens 350 -> 344 us, at 200 tokens 400 -> 396.)
  constexpr int kValu = !A32 || C >= 8 ? 4 : C == 4 ? 6 : C == 1 ? 21 : 12;
  cq_v4u af[2][RB];
  cq_v4u bfr[C];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) af[0][rb] = decode8<PRE>(wq[0][rb][0], tab[rb]);
#pragma unroll
  for (int cb = 0; cb < C; ++cb) bfr[cb] = read_b(0, 0, cb);

  int s0 = 0;
  do {  // at least two steps exist (no zero-trip path: the accumulators stay in their AGPRs throughout)
#pragma unroll
    for (int par = 0; par < D; ++par) {  // step s0 + par uses weights wq[par] and tile buffer par
      if (par > 0 && (par & 1) == 0 && s0 + par >= nS) break;  // K is a multiple of 128: steps come in pairs
      const int s3 = min(s0 + par + D - 1, nS - 1);
      fetch_weights(wq[(par + D - 1) & (D - 1)], s3);
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const int cur = jj & 1, nxt = cur ^ 1;
        if constexpr (BLK) {
          if (par == D - 1 && jj == 3) {
            // A group of weights ends with this step (groups are whole multiples of D steps, so only here;
            // the branch sits at a sub-step boundary, where the instruction scheduler is fenced anyway).
            // Its successor's tables were requested at least D steps ago and have arrived: the waits since
            // left fewer loads outstanding than were issued after that request.  The wait below never
            // stalls (no more than that many loads are ever outstanding); it orders the LDS reads behind
            // the arrival.
            if (s0 + D == switch_at) {
              asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kInFlight + kPerStep + 2) : "memory");
              const uint32_t at = tbl_lds + (blk_next & 1) * (4 * kNextTableBytes) + r32 * 16;
              const cq_v4u a0 = lds_read_u128(at), a1 = lds_read_u128(at + 512);
              const cq_v4u b0 = lds_read_u128(at + 1024), b1 = lds_read_u128(at + 1536);
              uint32_t r0[8] = {a0[0], a0[1], a0[2], a0[3], a1[0], a1[1], a1[2], a1[3]};
              uint32_t r1[8] = {b0[0], b0[1], b0[2], b0[3], b1[0], b1[1], b1[2], b1[3]};
              tab[0] = make_row_table<F16>(r0);
              tab[1] = make_row_table<F16>(r1);
              ++blk_next;
              switch_at += p.gsteps;
            }
            // The tables of the group after the current one are requested in EVERY pass (again, if they
            // were requested before: 2 KiB per wavefront from L2, the same bytes to the same place), so
            // that the number of loads in flight, and with it every wait count, is a compile-time constant.
            fetch_tables(blk_next);
          }
        }
        // the C tile loads are spread over the step: no LDS write bursts
        if constexpr (C >= 4) fetch_tile(s3, (par + D - 1) & (D - 1), jj * (C / 4), C / 4);
        else if (jj < C) fetch_tile(s3, (par + D - 1) & (D - 1), jj, 1);
        // next sub-step: jj + 1 of this step, or the first one of the next step
        const int nbuf = jj < 3 ? par : (par + 1) & (D - 1), njj = (jj + 1) & 3;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) af[nxt][rb] = decode8<PRE>(wq[nbuf][rb][njj], tab[rb]);
#pragma unroll
        for (int cb = 0; cb < C; ++cb) {
          const cq_v4u b = bfr[cb];
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) acc[rb][cb] = mfma_large<F16>(af[cur][rb], b, acc[rb][cb]);
          bfr[cb] = read_b(nbuf, njj, cb);
        }
#pragma unroll
        for (int i = 0; i < RB * C; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                   // one MFMA
          __builtin_amdgcn_sched_group_barrier(0x002, kValu, 0);               // vector ALU operations
          if (i % RB == RB - 1) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // one LDS read
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      // (block-wise tables: the two table requests of a pass's last step are younger than what the waits
      // of that step and of the next D - 4 steps are for, and may stay in flight as well)
      // (par is a constant once the loop is unrolled: no branch is left here)
      if constexpr (RB == 1)
        vm_wait<kInFlight>(wq[(par + 2) & (D - 1)][0]);
      else if (BLK && (par == D - 1 || par <= D - 5))
        vm_wait<kInFlight + 2>(wq[(par + 2) & (D - 1)][0], wq[(par + 2) & (D - 1)][1]);
      else
        vm_wait<kInFlight>(wq[(par + 2) & (D - 1)][0], wq[(par + 2) & (D - 1)][1]);
      __syncthreads();
    }
    s0 += D;
  } while (s0 < nS);
  // Nothing of this workgroup may still be on its way into LDS when the loop is left, nor into registers: the last (clamped,
  // unused) loads of weights still target the ring, which therefore has to stay allocated up to this wait -- its entries are
  // named here and behind it, so that the compiler cannot reuse them earlier.  (What is on its way after the last step, an odd
  // one of the ring, was requested in the last D - 3 steps: with four entries, an even one.)
  asm volatile("s_waitcnt vmcnt(0)" : "+v"(wq[0][0])::"memory");
#pragma unroll
  for (int i = 0; i < D; i += D == 4 ? 2 : 1)
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) asm volatile("" : "+v"(wq[i][rb]));

  // ---- epilogue: per-token scale, optional SiLU(gate)*up, store ----
  // A lane holds 4 consecutive outputs of ONE token per accumulator quad, so storing from registers
  // would touch 64 different cache lines per instruction.  Instead the tile goes through LDS (free
  // now) 64 tokens at a time: row-major [token][this workgroup's columns] with a padded row stride
  // (conflict-free writes), then the workgroup streams whole rows out, neighbouring lanes writing
  // neighbouring bytes.
  constexpr int kOutCols = EPI == CQ_EPI_SWIGLU ? kRows / 2 : kRows;
  constexpr int kEsize = OUTK == CQ_OUT_F16 ? 2 : 4;
  constexpr int kRowBytes = kOutCols * kEsize;                    // 128 .. 1024
  constexpr int kQuadBytes = (EPI == CQ_EPI_SWIGLU ? 2 : 4) * kEsize;  // what one accumulator quad becomes
  constexpr int kRowStride = kRowBytes + (kQuadBytes == 16 ? 16 : 8);
  constexpr int kPiece = kRowStride % 16 == 0 ? 16 : 8;           // bytes per lane when streaming out
  constexpr int kPiecesPerRow = kRowBytes / kPiece;
  static_assert(kRowStride <= epilogue_row_stride(EPI, OUTK), "the launcher sizes LDS for tiles of 256 rows");
  const size_t out_col0 = (size_t)rt * kOutCols;
  typedef __attribute__((address_space(3))) uint32_t lds_u32;
  typedef __attribute__((address_space(3))) cq_v4u lds_v4u;
  typedef __attribute__((__vector_size__(2 * sizeof(uint32_t)))) uint32_t v2u;
  typedef __attribute__((address_space(3))) v2u lds_v2u;
#pragma unroll
  for (int pass = 0; pass < (C + 1) / 2; ++pass) {
    __syncthreads();  // the tile buffers (first pass) or the previous pass's rows are no longer read
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int cb = pass * 2 + half;
      if (cb >= C) break;
      const int tl = half * 32 + r32;  // token within the pass
      float sc = 1.f;
      if (p.row_scale) {
        const int m = mrow0 + min(cb * 32 + r32, mcnt - 1);
        sc = p.row_scale[p.scale_gather ? p.scale_gather[m] : m];
      }
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
        for (int vb = 0; vb < 4; ++vb) {
          // MFMA 32x32 output: register v holds row 8*(v/4) + 4*(lane/32) + v%4, column lane%32
          const int quad = (wave * (32 * RB) + rb * 32 + vb * 8 + g2 * 4) >> 2;  // which 4 weight rows of the tile
          const uint32_t at = (uint32_t)tl * kRowStride + (uint32_t)quad * kQuadBytes;
          const float x0 = sc * acc[rb][cb][4 * vb], x1 = sc * acc[rb][cb][4 * vb + 1];
          const float x2 = sc * acc[rb][cb][4 * vb + 2], x3 = sc * acc[rb][cb][4 * vb + 3];
          if constexpr (EPI == CQ_EPI_SWIGLU) {
            const float h0 = x0 * __builtin_amdgcn_rcpf(1.f + __expf(-x0)) * x1;
            const float h1 = x2 * __builtin_amdgcn_rcpf(1.f + __expf(-x2)) * x3;
            if constexpr (OUTK == CQ_OUT_F16)
              *reinterpret_cast<lds_u32*>((uintptr_t)at) = f32_to_f16_sat(h0) | (f32_to_f16_sat(h1) << 16);
            else
              *reinterpret_cast<lds_v2u*>((uintptr_t)at) = v2u{__float_as_uint(h0), __float_as_uint(h1)};
          } else {
            if constexpr (OUTK == CQ_OUT_F16)
              *reinterpret_cast<lds_v2u*>((uintptr_t)at) = v2u{f32_to_f16_sat(x0) | (f32_to_f16_sat(x1) << 16),
                                                                f32_to_f16_sat(x2) | (f32_to_f16_sat(x3) << 16)};
            else
              *reinterpret_cast<lds_v4u*>((uintptr_t)at) =
                  cq_v4u{__float_as_uint(x0), __float_as_uint(x1), __float_as_uint(x2), __float_as_uint(x3)};
          }
        }
      }
    }
    __syncthreads();
    // stream the 64 rows out: piece i of the pass = (token i / kPiecesPerRow, piece i % kPiecesPerRow)
#pragma unroll
    for (int it = 0; it < 64 * kPiecesPerRow / 256; ++it) {
      const int i = it * 256 + tid;
      const int tl = i / kPiecesPerRow, pc = i - tl * kPiecesPerRow;
      const int tok = pass * 64 + tl;
      if (tok < mcnt) {
        const uint32_t at = (uint32_t)tl * kRowStride + (uint32_t)pc * kPiece;
        char* dst = reinterpret_cast<char*>(p.out) + ((size_t)(mrow0 + tok) * p.out_ld + out_col0) * kEsize + (size_t)pc * kPiece;
        if constexpr (BLK) dst += (size_t)blockIdx.y * p.part_stride * kEsize;
        if constexpr (kTail) {
          if (kz > 0)
            dst = reinterpret_cast<char*>(p.tail_part) +
                  (((size_t)(kz - 1) * p.tail_rows + tail_row0 + tok) * p.out_ld + out_col0) * kEsize + (size_t)pc * kPiece;
        }
        if constexpr (kPiece == 16)
          *reinterpret_cast<cq_v4u*>(dst) = *reinterpret_cast<const lds_v4u*>((uintptr_t)at);
        else
          *reinterpret_cast<v2u*>(dst) = *reinterpret_cast<const lds_v2u*>((uintptr_t)at);
      }
    }
  }
}

// The launch's token tiles, derived by every wavefront from the group offsets (a launch that built lists of them cost 5
// us, twice per layer): a group with more than small_max rows is cut into tiles of w0 (while more than w1 rows remain),
// then one of w1 or (up to w2 rows left) w2.  List 0 holds the w0-wide tiles, lists 1 and 2 the last tiles of the groups,
// each in group order.  Lane l looks at group 64 r + l in round r; the offsets of the first two rounds stay in registers,
// those of further ones are loaded again when a tile is looked up.  All members but the lane's own group are uniform.
struct tile_map {
  int n0, n1, n2;           // tiles per list
  int kS0, kS1;             // K parts of a tile of list 0, and of lists 1 and 2
  int from[2], to[2];       // offsets of the lane's groups of rounds 0 and 1
  int base, m0, a, last, incl;   // this batch of 64: the lane's group: first row, whole tiles, rows left; tiles up to it
  uint64_t m1, m2;          // ... its groups whose last tile is in list 1, 2

  __device__ __forceinline__ void round(const LargeArgs& p, int f, int t) {
    m0 = f;
    const int me = t - f > p.small_max ? t - f : 0;
    a = me / p.w0;
    last = me - a * p.w0;
    if (last > p.w1) { ++a; last -= p.w0; }   // (negative: the last whole tile is not full)
    m1 = __ballot(last > p.w2);
    m2 = __ballot(last > 0 && last <= p.w2);
    incl = cq_route::wave_scan(a);
  }
  __device__ __forceinline__ void load(const LargeArgs& p, int lane, int at, int& f, int& t) {
    const int g = at + lane;
    f = g < p.G ? p.group_offsets[g] : 0;
    t = g < p.G ? p.group_offsets[g + 1] : 0;
  }
  __device__ __forceinline__ void add() {
    n0 += __builtin_amdgcn_readlane(incl, 63);
    n1 += __popcll(m1);
    n2 += __popcll(m2);
  }
  __device__ __forceinline__ void init(const LargeArgs& p, int lane) {
    n0 = n1 = n2 = 0;
    load(p, lane, 0, from[0], to[0]);
    load(p, lane, 64, from[1], to[1]);
    for (base = 128; base < p.G; base += 64) {
      int f, t;
      load(p, lane, base, f, t);
      round(p, f, t);
      add();
    }
    if (p.G > 64) {
      round(p, from[1], to[1]);
      add();
    }
    round(p, from[0], to[0]);
    add();
    base = 0;
    // K parts: the narrow tiles come last; when there are fewer of them than the chip runs at a time, the end of the
    // launch runs on a part of it for the length of a whole K loop -- parts of K on more workgroups shorten it.  A launch
    // of few tiles in all (tail_abs: any tile can have partial sums) leaves most of the chip idle for a whole K loop
    // otherwise.
    kS0 = kS1 = 1;
    if (p.tail_part) {
      const int narrow = (n1 + n2) * p.row_tiles, all = narrow + n0 * p.row_tiles;
      while (kS1 < kTailSplitMax && narrow > 0 && narrow * kS1 * 2 <= p.at_once) kS1 *= 2;
      while (p.tail_abs && kS0 < kTailSplitMax && n0 > 0 && all * kS0 * 2 <= p.at_once) kS0 *= 2;
    }
  }
  // group, first sorted row and row count of tile t of a list (t < the list's n)
  __device__ __forceinline__ void find(const LargeArgs& p, int lane, int list, int t, int& grp, int& row0, int& cnt) {
    for (;;) {
      const int here = list == 0 ? __builtin_amdgcn_readlane(incl, 63) : __popcll(list == 1 ? m1 : m2);
      if (t < here) break;
      t -= here;
      base += 64;
      int f = from[1], u = to[1];
      if (base > 64) load(p, lane, base, f, u);
      round(p, f, u);
    }
    int src, i;
    if (list == 0) {
      src = __ffsll((long long)__ballot(incl > t)) - 1;
      i = t - (__builtin_amdgcn_readlane(incl, src) - __builtin_amdgcn_readlane(a, src));
    } else {
      src = cq_route::nth_set_lane(list == 1 ? m1 : m2, t, lane);
      i = __builtin_amdgcn_readlane(a, src);
    }
    const int whole = __builtin_amdgcn_readlane(a, src), rest = __builtin_amdgcn_readlane(last, src);
    grp = base + src;
    row0 = __builtin_amdgcn_readlane(m0, src) + i * p.w0;
    cnt = min(p.w0, whole * p.w0 + rest - i * p.w0);
  }
};

// How many of an XCD's last tiles are cut into two of 128 rows (all: its tiles of the launch, last: those of list 2).
// An XCD has 32 compute units, and one that runs a single workgroup does 0.84 of the work of two: what counts is how many
// tiles the busiest unit gets, all / 32 rounded up.  Up to half a round too many, 16 tiles in halves save half a tile's time
// (groups x 2048 x 2048 of 60 rows, us, whole / halves: 36 groups, i.e. tiles per XCD, 39.1 / 32.4, 48 41.1 / 35.3, 66
// 58.9 / 51.4, 80 62.2 / 55.2, 112 83.8 / 76.5); any more, and the halves themselves begin another round (52: 41.5 / 48.4,
// 64: 45.2 / 52.0, 96: 64.9 / 69.9).  A launch that leaves units idle takes all of them in halves, while none gets a half
// besides a whole tile (8 23.0 / 16.7, 16 25.0 / 18.5, 24 26.0 / 24.9, 32 28.7 / 27.4).  With 8, 24 or 32 halves instead of
// 16 the launches of more than a round take the same or longer.
constexpr int kHalvedMax = 32;
__device__ __forceinline__ int halved_tiles(int all, int last) {
  if (all <= 32) return all + last <= 32 || last == all ? last : 0;
  const int over = all & 31;
  return over > 0 && over <= 16 && last >= over ? min(16, last) : 0;
}

// The same for whole tiles, one workgroup per compute unit: where up to half a round of the widest ones is too many (s0 on an
// XCD), these come in halves, which all run at once.  Groups of 512 rows x 2048 x 4096, us, whole / halves: s0 = 34 198.5 /
// 171.0, 40 198.5 / 174.0, 48 215.7 / 196.6, 66 319.5 / 292.5, 80 337.7 / 317.7, 112 454 / 439; one group of 8448 to 9216 rows x
// 4096 x 14336 (66 to 72) 1001..1007 / 914..922.  Beyond ten rounds no difference (28672 x 4096, 462 to 504: 1624..1745 / 1608..1749).
constexpr int kHalvedWholeMax = 16;
__device__ __forceinline__ int halved_whole_tiles(int s0) {
  const int over = s0 & 31;
  return s0 > 32 && over <= kHalvedWholeMax ? over : 0;
}

// Work items = (token tile, row tile, K part); tiles of the three widths in ONE launch so that the short lists do not
// leave most of the chip idle.  Two forms:
//   * whole tiles, 256 / 128 / 64 tokens, one workgroup per compute unit (all 512 registers of a lane, four or eight
//     activation tiles in LDS): a decoded weight serves up to 256 tokens.  Bound by the matrix cores and by power; the
//     last ones of 256 tokens may come in two halves of 128 weight rows (halved_whole_tiles);
//   * half tiles, 128 / 96 / 64 (or 32) tokens (HALF), 256 registers and at most half the LDS, so that TWO workgroups share a
//     compute unit and one's barriers, waits, decoding and epilogue run under the other's matrix work.
//     The last tiles of list 2 may come in two halves of 128 weight rows (halved_tiles).
//     gate/up + down of the Mixtral shape at 128 rows per group 314 + 172 -> 275 + 148 us, of DeepSeek-V2-Lite's at
//     48 rows per group (two launches before, of the streaming kernel and of whole tiles) 203 -> 134 us.
// cq_gemm_uses_half_tiles has the rule between the two.
// XCD-aware remap of the linear workgroup id (ids go round-robin over the 8 XCDs): XCD x takes a contiguous share of
// each list (neighbours share activations in its L2; equal mix on every XCD), the widest tiles first.  The grid is
// sized for the worst case; the lists are usually much shorter.
template <bool F16, int EPI, int OUTK, bool BLK, bool PRE, bool HALF>
__global__ __launch_bounds__(256, HALF ? 2 : 1) void gemm_large_kernel(const LargeArgs p) {
  using W = tile_widths<HALF>;
  constexpr int kDeep = HALF ? 4 : 8;   // pipeline depth of the narrower tiles: less matrix time per step, needs more
  const int lane = threadIdx.x & 63, xcd = blockIdx.x & 7;
  int slot = blockIdx.x >> 3;
  tile_map map;
  map.init(p, lane);
  const int row_tiles = p.row_tiles;
  // work item `slot` of this XCD's share of a list: its tile, row tile and K part
  int grp, row0, cnt, tile, rt, kz;
  auto item = [&](int list, int kS) {
    const int n = (list == 0 ? map.n0 : list == 1 ? map.n1 : map.n2) * row_tiles * kS;
    const int work = xcd * ((n + 7) >> 3) + slot;
    if (work >= n) return false;
    const int per_tile = row_tiles * kS;
    tile = work / per_tile;
    const int rest = work - tile * per_tile;
    rt = rest / kS;
    kz = rest - rt * kS;
    map.find(p, lane, list, tile, grp, row0, cnt);
    return true;
  };
  const int s0 = (map.n0 * row_tiles * map.kS0 + 7) >> 3, s1 = (map.n1 * row_tiles * map.kS1 + 7) >> 3,
            s2 = (map.n2 * row_tiles * map.kS1 + 7) >> 3;
  const int over = !HALF && !BLK && map.kS0 == 1 ? halved_whole_tiles(s0) : 0;
  if (slot < s0 - over) {
    if (item(0, map.kS0)) large_tile<F16, EPI, OUTK, W::w0 / 32, 4, BLK, PRE, HALF>(p, grp, row0, cnt, rt, kz, map.kS0, row0);
    return;
  }
  if (slot < s0 + over) {
    if constexpr (!HALF && !BLK) {
      const int part0 = (slot - (s0 - over)) & 1;
      slot = s0 - over + ((slot - (s0 - over)) >> 1);
      if (item(0, 1)) large_tile<F16, EPI, OUTK, W::w0 / 32, 4, BLK, PRE, HALF, 1>(p, grp, row0, cnt, 2 * rt + part0, 0, 1, row0);
    }
    return;
  }
  slot -= s0 + over;
  if (slot < s1) {
    if (item(1, map.kS1))
      large_tile<F16, EPI, OUTK, W::w1 / 32, kDeep, BLK, PRE, HALF>(p, grp, row0, cnt, rt, kz, map.kS1,
                                                                    p.tail_abs ? row0 : tile * W::w1);
    return;
  }
  slot -= s1;
  // the last tiles of the launch, cut into halves
  const int halves = HALF ? halved_tiles(s0 + s1 + s2, s2) : 0;
  const bool cut = slot >= s2 - halves;
  const int part = cut ? (slot - (s2 - halves)) & 1 : 0;
  if (cut) slot = s2 - halves + ((slot - (s2 - halves)) >> 1);
  if (slot >= s2 || !item(2, map.kS1)) return;
  const int tail_row = p.tail_abs ? row0 : p.tail_rows1 + tile * W::w2;
  if constexpr (HALF) {
    // (up to 32 rows: decoding a tile's weights takes longer than the products of 64 tokens, but those cost power, which is
    // what a full launch is bound by; 66 groups of 20 rows x 2816 x 2048 60.5 -> 57.0 us, x 2048 x 1408 42.8 -> 41.1.  Rows
    // of zeros in place of the missing ones, in wider tiles, gained 2 % at 33 of 64 rows and lost 1 % at 46 and 64)
    if (cut) {
      if (cnt <= 32) large_tile<F16, EPI, OUTK, 1, kDeep, BLK, PRE, HALF, 1>(p, grp, row0, cnt, 2 * rt + part, kz, map.kS1, tail_row);
      else large_tile<F16, EPI, OUTK, 2, kDeep, BLK, PRE, HALF, 1>(p, grp, row0, cnt, 2 * rt + part, kz, map.kS1, tail_row);
      return;
    }
    if (cnt <= 32) {
      large_tile<F16, EPI, OUTK, 1, kDeep, BLK, PRE, HALF>(p, grp, row0, cnt, rt, kz, map.kS1, tail_row);
      return;
    }
  }
  large_tile<F16, EPI, OUTK, W::w2 / 32, kDeep, BLK, PRE, HALF>(p, grp, row0, cnt, rt, kz, map.kS1, tail_row);
}

// out[row] += slice 0 + slice 1 + ... of the tiles' K parts, in that order (see LargeArgs::tail_part).
// blockIdx.y: entry of the w1-token list, of the w2-token list, then (launches of few tiles) of the widest list;
// blockIdx.x: 1024 columns; blockIdx.z: 8 rows.
constexpr int kTailSumRows = 8;
__global__ __launch_bounds__(256) void tail_sum_kernel(const LargeArgs p, int cap1) {
  const int list = (int)blockIdx.y < cap1 ? 1 : (int)blockIdx.y < 2 * cap1 ? 2 : 0;
  const int j = (int)blockIdx.y - (list == 0 ? 2 : list - 1) * cap1;
  const int lane = threadIdx.x & 63;
  tile_map map;
  map.init(p, lane);
  const int kS = list == 0 ? map.kS0 : map.kS1;
  if (kS <= 1 || j >= (list == 0 ? map.n0 : list == 1 ? map.n1 : map.n2)) return;
  int grp, mrow0, mcnt;
  map.find(p, lane, list, j, grp, mrow0, mcnt);
  const int row0 = p.tail_abs ? mrow0 : list == 2 ? p.tail_rows1 + j * p.w2 : j * p.w1;
  const int c = (blockIdx.x * 256 + threadIdx.x) * 4;
  const int r0 = blockIdx.z * kTailSumRows;
  if (c >= p.N || r0 >= mcnt) return;
  float* out = reinterpret_cast<float*>(p.out);
  float4 acc[kTailSumRows], part[kTailSumRows][kTailSplitMax > 1 ? kTailSplitMax - 1 : 1];
#pragma unroll
  for (int i = 0; i < kTailSumRows; ++i) {   // all loads first (rows past the tile's end read its last row)
    const int r = min(r0 + i, mcnt - 1);
    acc[i] = *reinterpret_cast<const float4*>(out + (size_t)(mrow0 + r) * p.N + c);
#pragma unroll
    for (int z = 1; z < kTailSplitMax; ++z)
      if (z < kS)
        part[i][z - 1] = *reinterpret_cast<const float4*>(p.tail_part + ((size_t)(z - 1) * p.tail_rows + row0 + r) * p.N + c);
  }
#pragma unroll
  for (int i = 0; i < kTailSumRows; ++i) {
    if (r0 + i >= mcnt) break;
#pragma unroll
    for (int z = 1; z < kTailSplitMax; ++z)
      if (z < kS) {
        acc[i].x += part[i][z - 1].x; acc[i].y += part[i][z - 1].y;
        acc[i].z += part[i][z - 1].z; acc[i].w += part[i][z - 1].w;
      }
    *reinterpret_cast<float4*>(out + (size_t)(mrow0 + r0 + i) * p.N + c) = acc[i];
  }
}

// Narrow tiles alone, for launches in which no group has more than 64 (C = 2) or 32 (C = 1) rows (block-wise
// tables at decode sizes): few accumulators and at most half the LDS, so two workgroups share a compute
// unit.  The list of 64-token tiles holds one entry per non-empty group in such a launch.
// (pipeline depth: 8 steps for 32-token tiles; 4 for 64-token tiles, whose accumulators leave no room for the
// register ring of 8 -- with 8 the bf16 instantiations spilled one or two registers, which kernels with
// asynchronous register loads must not do)
constexpr int narrow_depth(int C) { return C >= 2 ? 4 : 8; }
template <bool F16, int EPI, int OUTK, bool BLK, bool PRE, int C>
__global__ __launch_bounds__(256, 2) void gemm_narrow_kernel(const LargeArgs p) {
  const int lane = threadIdx.x & 63;
  tile_map map;
  map.init(p, lane);
  const int n2 = map.n2 * p.row_tiles;
  const int per = (n2 + 7) >> 3;
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  if (slot >= per) return;
  const int work = xcd * per + slot;
  if (work >= n2) return;
  const int tile = work / p.row_tiles, rt = work - tile * p.row_tiles;
  int grp, row0, cnt;
  map.find(p, lane, 2, tile, grp, row0, cnt);
  large_tile<F16, EPI, OUTK, C, narrow_depth(C), BLK, PRE>(p, grp, row0, cnt, rt);
}

// Pre-pass for activation kinds the main kernel does not read: sorted row m of the result is row
// src(m) of A as bf16 (exact for integer codes) or f16 (saturating, from fp32).  8 values per thread.
template <int AK>
__global__ __launch_bounds__(256) void convert_rows_kernel(const void* __restrict__ A, const int32_t* __restrict__ gather,
                                                           int M, int K, uint16_t* __restrict__ out) {
  const int cpr = K >> 3;  // 8-value chunks per row
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (size_t)M * cpr) return;
  const int m = (int)(i / cpr), c = (int)(i - (size_t)m * cpr);
  const size_t src = (size_t)(gather ? gather[m] : m) * K + (size_t)c * 8;
  uint32_t o[4];
  if constexpr (AK == CQ_A_INT8_CODES) {
    const uint2 raw = *reinterpret_cast<const uint2*>(reinterpret_cast<const int8_t*>(A) + src);
    const uint32_t rw[2] = {raw.x, raw.y};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int b0 = (int)(int8_t)(rw[h] & 0xff), b1 = (int)(int8_t)((rw[h] >> 8) & 0xff);
      const int b2 = (int)(int8_t)((rw[h] >> 16) & 0xff), b3 = (int)(int8_t)(rw[h] >> 24);
      o[2 * h] = code_bf16(b0) | (code_bf16(b1) << 16);
      o[2 * h + 1] = code_bf16(b2) | (code_bf16(b3) << 16);
    }
  } else {
    const float4 f0 = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(A) + src);
    const float4 f1 = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(A) + src + 4);
    o[0] = f32_to_f16_sat(f0.x) | (f32_to_f16_sat(f0.y) << 16);
    o[1] = f32_to_f16_sat(f0.z) | (f32_to_f16_sat(f0.w) << 16);
    o[2] = f32_to_f16_sat(f1.x) | (f32_to_f16_sat(f1.y) << 16);
    o[3] = f32_to_f16_sat(f1.z) | (f32_to_f16_sat(f1.w) << 16);
  }
  *reinterpret_cast<uint4*>(out + (size_t)m * K + (size_t)c * 8) = make_uint4(o[0], o[1], o[2], o[3]);
}

template <bool F16, int EPI, int OUTK, bool BLK, bool PRE, int C>
cq_status launch_narrow(const LargeArgs& a, int max1, hipStream_t s) {
  auto kern = gemm_narrow_kernel<F16, EPI, OUTK, BLK, PRE, C>;
  constexpr int lds_epi = 64 * epilogue_row_stride(EPI, OUTK);
  constexpr int lds_loop = narrow_depth(C) * 32 * C * kStepBytes + (BLK ? 8 * kNextTableBytes : 0);
  constexpr int lds = lds_loop > lds_epi ? lds_loop : lds_epi;
  static_assert(2 * lds <= 160 * 1024, "two workgroups per compute unit");
  static std::atomic<bool> configured{false};
  const cq_status st = cq_configure_lds(kern, lds, configured, true);
  if (st != CQ_OK) return st;
  const long grid = (((long)max1 * a.row_tiles + 7) / 8) * 8;
  if (grid <= 0) return CQ_OK;
  const int total = a.K / kStepK;
  hipLaunchKernelGGL(kern, dim3((unsigned)grid, (unsigned)((total + a.ksteps - 1) / a.ksteps)), dim3(256), lds, s, a);
  return cq_check_launch();
}

// narrow: 64 or 32 when the caller knows that no group has more rows than that (block-wise tables), kHalf: half tiles,
// else 0
constexpr int kHalf = -1;
template <bool F16, int EPI, int OUTK, bool BLK, bool PRE, bool HALF>
cq_status launch_tiles(LargeArgs a, int max0, int max1, hipStream_t s) {
  auto kern = gemm_large_kernel<F16, EPI, OUTK, BLK, PRE, HALF>;
  constexpr int lds_epi = 64 * epilogue_row_stride(EPI, OUTK);
  constexpr int lds_loop = 4 * tile_widths<HALF>::w0 * kStepBytes + (BLK ? 8 * kNextTableBytes : 0);
  constexpr int lds = lds_loop > lds_epi ? lds_loop : lds_epi;
  static_assert((HALF ? 2 : 1) * lds <= 160 * 1024, "workgroups per compute unit");
  static_assert(HALF || 8 * tile_widths<HALF>::w1 * kStepBytes <= 4 * tile_widths<HALF>::w0 * kStepBytes, "deep rings fit");
  static std::atomic<bool> configured{false};
  const cq_status st = cq_configure_lds(kern, lds, configured, true);
  if (st != CQ_OK) return st;
  // worst case of the kernel's per-XCD shares (a group ends in at most one tile of a narrow width, but the
  // two lists round up separately): ceil(n0/8) + ceil(n1/8) + ceil(n2/8) slots on each of 8 XCDs
  const long w0 = (long)max0 * a.row_tiles * (a.tail_part && a.tail_abs ? kTailSplitMax : 1),
             w1 = (long)max1 * a.row_tiles * (a.tail_part ? kTailSplitMax : 1);   // (narrow tiles may come in K parts)
  const long grid = ((w0 + 7) / 8 + (w1 + 7) / 8 + 1 + (HALF ? kHalvedMax : BLK ? 0 : kHalvedWholeMax)) * 8;
  if (grid <= 0) return CQ_OK;
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(256), lds, s, a);
  return cq_check_launch();
}

template <bool F16, int EPI, int OUTK, bool BLK, bool PRE>
cq_status launch_both(LargeArgs a, int max0, int max1, int narrow, hipStream_t s) {
  if constexpr (BLK) {
    if (narrow == 32) return launch_narrow<F16, EPI, OUTK, BLK, PRE, 1>(a, max1, s);
    if (narrow == 64) return launch_narrow<F16, EPI, OUTK, BLK, PRE, 2>(a, max1, s);
  } else {
    if (narrow == kHalf) return launch_tiles<F16, EPI, OUTK, BLK, PRE, true>(a, max0, max1, s);
  }
  return launch_tiles<F16, EPI, OUTK, BLK, PRE, false>(a, max0, max1, s);
}

template <bool F16, bool BLK, bool PRE>
cq_status dispatch_large_pre(const LargeArgs& a, int epilogue, int out_kind, int max0, int max1, int narrow, hipStream_t s) {
  if (epilogue == CQ_EPI_SWIGLU)
    return out_kind == CQ_OUT_F16
               ? launch_both<F16, CQ_EPI_SWIGLU, CQ_OUT_F16, BLK, PRE>(a, max0, max1, narrow, s)
               : launch_both<F16, CQ_EPI_SWIGLU, CQ_OUT_F32, BLK, PRE>(a, max0, max1, narrow, s);
  return out_kind == CQ_OUT_F16
             ? launch_both<F16, CQ_EPI_NONE, CQ_OUT_F16, BLK, PRE>(a, max0, max1, narrow, s)
             : launch_both<F16, CQ_EPI_NONE, CQ_OUT_F32, BLK, PRE>(a, max0, max1, narrow, s);
}

template <bool F16, bool BLK>
cq_status dispatch_large_blk(const LargeArgs& a, int epilogue, int out_kind, int max0, int max1, int narrow, hipStream_t s) {
  return a.prepacked
             ? dispatch_large_pre<F16, BLK, true>(a, epilogue, out_kind, max0, max1, narrow, s)
             : dispatch_large_pre<F16, BLK, false>(a, epilogue, out_kind, max0, max1, narrow, s);
}

// The two-workgroup kernel for 64-token tiles exists for block-wise tables only (the streaming kernel takes
// the small groups otherwise).
template <bool F16>
cq_status dispatch_large(const LargeArgs& a, int epilogue, int out_kind, int max0, int max1, int narrow, hipStream_t s) {
  return a.nblk > 1
             ? dispatch_large_blk<F16, true>(a, epilogue, out_kind, max0, max1, narrow, s)
             : dispatch_large_blk<F16, false>(a, epilogue, out_kind, max0, max1, narrow == kHalf ? kHalf : 0, s);
}

// Upper bounds on the tile counts for M_total rows in G groups (host side; sizes on the device vary).
void tile_caps(int G, int M_total, int* cap0, int* cap1) {
  *cap0 = M_total / (tile_widths<true>::w1 + 1) + 1;   // every widest tile covers more than w1 rows (96, or 128)
  *cap1 = G < M_total ? G : M_total;  // at most one per group
  if (*cap1 < 1) *cap1 = 1;
}

}  // namespace

// The tiles of a plain fp32 product with a long K may be cut into K parts (LargeArgs::tail_part).
bool cq_gemm_large_tail_split(const cq_codebook_weights* W, int epilogue, int out_kind) {
  return epilogue == CQ_EPI_NONE && out_kind == CQ_OUT_F32 && cq_tables_per_row(W) == 1 &&
         W->K / kStepK >= kTailMinSteps;
}

// Whole or half tiles.  The weights are decoded once per tile of tokens: with a long K (prologue and epilogue do not
// count) and several 256-token tiles per group, whole tiles save more than two workgroups per compute unit gain
// (Mixtral shape, K = 4096 and 14336: 1645 us per layer on half tiles against 1604 at 512 rows per group, 961 against
// 983 at 256, 622 against 691 at 128; K = 2048 / 1408 and 2048 / 768: 823 against 888 at 496 rows per group, 618 against
// 674 at 256).  Launches whose half tiles all run at once, one per compute unit, take these: whole tiles would leave half of the
// units idle.  Beyond, some units get two, while the whole tiles still have one each.  us, whole / half tiles, rows x N x K:
// one group of 1124 x 4096 x 4096 83 / 53, 1892 83 / 64, 2148 84 / 94, 2660 90 / 97, 3140 100 / 100; four of 921 x 2048 x 7168
// 133 / 104, 1177 141 / 158; 8 uneven ones, mean 460 x 2048 x 7168 134 / 112, 524 136 / 151; 16, mean 518 x 1024 x 2560 58 / 60.
// A group leaves up to a tile of fewer rows, which costs less: of 504 launches of 2 to 32 groups, even and uneven, all were
// faster on half tiles up to 122 * 256 rows x row tiles (by 13 % and more), of 144 from 125 to 128 * 256 29 were slower, by up to 12 %.
// Half tiles address the rows of A with 32-bit byte offsets.
// a_rows: number of rows of A, 0 if unknown.
bool cq_gemm_uses_half_tiles(const cq_codebook_weights* W, int M_total, long a_rows) {
  if (cq_tables_per_row(W) > 1 || a_rows <= 0 || a_rows * W->K * 2 >= (1L << 32)) return false;
  if (W->K <= 2048 || M_total < 384L * W->G) return true;
  const long row_tiles = W->N / kLargeRows;
  return W->G == 1 ? (M_total + 127L) / 128 * row_tiles <= 256 : M_total * row_tiles <= 122L * 256;
}

namespace {
// rows of a slice of partial sums: a slot per possible narrow tile (w1 + w2 rows per group), or the launch's own
// rows when those are fewer
int tail_slice_rows(int G, int M_total, bool half, bool* absolute) {
  int c0, c1;
  tile_caps(G, M_total, &c0, &c1);
  const int slots = c1 * (half ? tile_widths<true>::w1 + tile_widths<true>::w2 : tile_widths<false>::w1 + tile_widths<false>::w2);
  *absolute = M_total < slots;
  return *absolute ? M_total : slots;
}
// partial sums of those K parts: [kTailSplitMax - 1][rows of a slice][N] fp32
size_t tail_part_bytes(int G, int M_total, int N, bool half) {
  bool absolute;
  const int rows = tail_slice_rows(G, M_total, half, &absolute);
  return cq_align_up((size_t)(kTailSplitMax - 1) * rows * N * sizeof(float), 256);
}
}  // namespace

// (tail_N > 0: a plain fp32 product of N columns whose K is long enough) the partial sums of the tiles' K parts, plus (with_conversion) room for the activations as 16-bit rows [M_total, K]
size_t cq_gemm_large_workspace_bytes(int G, int M_total, int K, bool with_conversion, int tail_N) {
  size_t n = 0;
  if (tail_N > 0 && K / kStepK >= kTailMinSteps) n += tail_part_bytes(G, M_total, tail_N, false);   // (whole tiles have the more slots)
  if (with_conversion) n += cq_align_up((size_t)M_total * K * sizeof(uint16_t), 256);
  return n;
}

// A list of the tiles.  The kernel derives them itself; the size queries have always counted the list, and go on to: what
// a batch's workspace serves must not depend on how its launches find their tiles.
size_t cq_gemm_tile_list_bytes(int G, int M_total) {
  const long whole = M_total / 129 + 1, narrow = G < M_total ? G : M_total;
  return cq_align_up(256 + ((size_t)(whole + 2 * narrow) * 4 + (size_t)G) * sizeof(int32_t), 256);
}

bool cq_gemm_large_supported(const cq_codebook_weights* W) {
  if (W->N % kLargeRows != 0 || W->K % (2 * kStepK) != 0) return false;
  // block-wise tables change between two passes of the unrolled pipeline (8 steps of 64)
  // (and the kernel addresses a group's tables with 32-bit byte offsets)
  const int nblk = cq_tables_per_row(W);
  return nblk == 1 || (W->group_k % (8 * kStepK) == 0 && (long)W->N * nblk * (CQ_N_CENTROIDS * 2) < (1L << 31));
}

cq_status cq_gemm_large_launch(const cq_codebook_weights* W, const void* A, int a_kind, const float* row_scale,
                               const int32_t* row_gather, const int32_t* group_offsets, int M_total, int small_max,
                               int epilogue, void* out, int out_kind, void* workspace, hipStream_t s, bool half) {
  int cap0, cap1;
  tile_caps(W->G, M_total, &cap0, &cap1);
  LargeArgs a;
  a.idx = W->prepacked ? (const uint8_t*)W->prepacked : W->idx;
  a.cent = W->cent;
  a.prepacked = W->prepacked ? 1 : 0;
  a.N = W->N;
  a.K = W->K;
  a.A = (const uint16_t*)A;
  a.a_gather = row_gather;
  a.row_scale = row_scale;
  a.scale_gather = row_gather;
  a.out = out;
  a.out_ld = epilogue == CQ_EPI_SWIGLU ? W->N / 2 : W->N;
  a.group_offsets = group_offsets;
  a.G = W->G;
  a.small_max = small_max;
  a.at_once = kAtOnce[half];
  a.row_tiles = W->N / kLargeRows;
  a.nblk = cq_tables_per_row(W);
  a.gsteps = a.nblk > 1 ? W->group_k / kStepK : W->K / kStepK;
  {
    int ksplit;
    cq_gemm_split_plan(W, M_total, epilogue, &ksplit, &a.ksteps);  // a split is planned for 64-token launches only
    a.part_stride = ksplit > 1 ? (size_t)M_total * W->N : 0;
  }
  // workspace: the partial sums of the tiles' K parts (if the launch may split them), then the 16-bit copy of the rows
  size_t ws_off = 0;
  const bool tail = cq_gemm_large_tail_split(W, epilogue, out_kind);
  a.tail_part = nullptr;
  a.w0 = half ? tile_widths<true>::w0 : tile_widths<false>::w0;
  a.w1 = half ? tile_widths<true>::w1 : tile_widths<false>::w1;
  a.w2 = tile_widths<true>::w2;
  a.tail_rows1 = cap1 * a.w1;
  {
    bool absolute;
    a.tail_rows = tail_slice_rows(W->G, M_total, half, &absolute);
    a.tail_abs = absolute ? 1 : 0;
  }
  if (tail) {
    a.tail_part = (float*)((char*)workspace + ws_off);
    ws_off += tail_part_bytes(W->G, M_total, W->N, half);
  }
  if (a_kind == CQ_A_INT8_CODES || a_kind == CQ_A_F32) {
    // 16-bit copy of the rows in sorted order (the gather is applied here)
    uint16_t* A16 = (uint16_t*)((char*)workspace + ws_off);
    const size_t chunks = (size_t)M_total * (W->K / 8);
    const unsigned blocks = (unsigned)((chunks + 255) / 256);
    if (a_kind == CQ_A_INT8_CODES)
      hipLaunchKernelGGL(convert_rows_kernel<CQ_A_INT8_CODES>, dim3(blocks), dim3(256), 0, s, A, row_gather, M_total,
                         W->K, A16);
    else
      hipLaunchKernelGGL(convert_rows_kernel<CQ_A_F32>, dim3(blocks), dim3(256), 0, s, A, row_gather, M_total, W->K,
                         A16);
    a.A = A16;
    a.a_gather = nullptr;
  }
  const bool f16 = a_kind == CQ_A_F16 || a_kind == CQ_A_F32;
  // with so few rows in all, every group has at most that many: one narrow tile each
  const int narrow = half ? kHalf : M_total <= 32 ? 32 : M_total <= 64 ? 64 : 0;
  // (for the grid: every widest tile of a launch of whole tiles covers more than 128 rows)
  const int max0 = half ? cap0 : M_total / (tile_widths<false>::w1 + 1) + 1;
  const cq_status st = f16 ? dispatch_large<true>(a, epilogue, out_kind, max0, cap1, narrow, s)
                           : dispatch_large<false>(a, epilogue, out_kind, max0, cap1, narrow, s);
  if (st != CQ_OK || !tail) return st;
  // (a launch of a few dozen workgroups that return at once when nothing is split)
  hipLaunchKernelGGL(tail_sum_kernel, dim3((W->N / 4 + 255) / 256, 2 * cap1 + (a.tail_abs ? cap0 : 0), (half ? tile_widths<true>::w0 : tile_widths<false>::w0) / kTailSumRows),
                     dim3(256), 0, s, a, cap1);
  return cq_check_launch();
}
