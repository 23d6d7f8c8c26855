// a6 / a7, streaming kernel: planning (K ranges, workgroups per group, which kernel takes which groups), the
// internal launcher and the entry point cq_codebook_grouped_gemm.  The kernel itself is in codebook_gemm_small.h.
#include "codebook_gemm_small.h"

namespace {

// out[m, :] = sum over the K splits of partials[s][m, :] in the order s = 0, 1, ... for the rows of the
// groups the streaming kernel handled (at most max_rows rows); other rows are left alone.
template <int OUTK>
__global__ __launch_bounds__(256) void sum_partials_kernel(const float* __restrict__ partials, size_t part_stride,
                                                           int ksplit, const int32_t* __restrict__ group_offsets,
                                                           int max_rows, int N, void* __restrict__ out) {
  const int grp = blockIdx.y;
  const int m0 = group_offsets[grp], Me = group_offsets[grp + 1] - m0;
  if (Me <= 0 || Me > max_rows) return;
  const int c = (blockIdx.x * 256 + threadIdx.x) * 4;
  if (c >= N) return;
  for (int m = m0 + blockIdx.z; m < m0 + Me; m += gridDim.z) {   // (blockIdx.z: rows of the group in parallel)
    const size_t at = (size_t)m * N + c;
    float4 acc = *reinterpret_cast<const float4*>(partials + at);
    for (int q = 1; q < ksplit; ++q) {
      const float4 v = *reinterpret_cast<const float4*>(partials + (size_t)q * part_stride + at);
      acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
    }
    if constexpr (OUTK == CQ_OUT_F16)
      *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(out) + at) =
          make_uint2(f32_to_f16_bits_sat(acc.x) | (f32_to_f16_bits_sat(acc.y) << 16),
                     f32_to_f16_bits_sat(acc.z) | (f32_to_f16_bits_sat(acc.w) << 16));
    else
      *reinterpret_cast<float4*>(reinterpret_cast<float*>(out) + at) = acc;
  }
}

// upper bound on the rows of a group
int row_bound(int M_total, int max_group_rows) {
  return max_group_rows > 0 && max_group_rows < M_total ? max_group_rows : M_total;
}

// Batches a little too large for one pass: where few groups have more rows, a second pass over their indices on
// workgroups of its own is cheaper than the large-tile launch behind a streaming launch (and the launches that add up
// both kinds' partial sums).  With groups of at most 128 rows and fewer than 28 rows per group on average (23
// with block-wise tables, in passes of 16 rows): us per layer of the Mixtral shape, two launches against passes: 33 tokens
// 174 / 169, 77 tokens 207 / 192, 110 tokens 291 / 254; block-wise tables (large tiles against passes) 40 tokens
// 347 / 232, 79 tokens 369 / 325, 92 tokens 359 / 340, 104 tokens 363 / 359, 111 tokens 362 / 377 (from 24 rows per
// group on the partial sums of wider layers no longer fit into the library's own array, which held these batches).
// Short K (2048 and less), where the large tiles took the small groups as well: 8 rows cost a tile what 64 do, so a group that
// fits one pass is cheaper streamed (66 groups x 2816 x 2048: 8 rows 60 / 46 us, 32 rows 62 / 58; two passes 110), whole
// layers of the DeepSeek-V2-Lite shape on tiles and in passes: 33 tokens 126 / 106, 64 tokens 140 / 123, 128 tokens
// 151 / 144 (256: 167 / 178).
// But a unit of 64 weight rows costs a workgroup about 1.2 us + 0.5 us per 1024 of K (its table, and eight wavefronts' sums
// to add up), a tile of 256 of them 2 us + 9.5 us per 1024 of K in a round of 512: the shorter K, the fewer units may come
// one after the other on a workgroup.  Up to (K + 64) / 256 of them passes are still the cheaper (tiles / passes, us: K = 256 4 groups
// x 2048 of 56 rows 6.3 / 5.5, 53 of them in one group 6.9 / 7.3, 8 x 8192 of 112 rows 7.0 / 10.4; K = 512 8 x 2048 of 112
// rows 8.6 / 5.9, 8 x 8192 9.7 / 11.1, 64 x 2048 of 384 rows 17.7 / 23.3; K = 768 16 x 2048 of 96 rows 10.9 / 8.3, 128 x 2048
// of 264 uneven rows 21.6 / 26.7; K = 1024 8 x 4096 of 112 rows 13.3 / 9.7, 32 x 4096 of 256 rows 26.8 / 27.5).  K = 2048 always gains (DeepSeek-V2-Lite shape 33 and 128 tokens 55.6 / 45.6 and 61.2 / 58.8,
// Qwen3 shape 64 and 128 tokens 37.8 / 30.0 and 41.5 / 37.3), from 1408 on where the tiles make more than a round even if
// some groups are empty (64 x 4096 x 1408 of 256 even and uneven rows 60.7 / 50.0 and 47.6 / 48.4), not where they make one:
// 66 x 2048 x 1408, DeepSeek-V2-Lite shape, 33, 64 and 128 tokens 30.2 / 32.0, 32.8 / 40.0 and 36.1 / 41.8.
bool short_k_in_passes(const cq_codebook_weights* W, int M_total) {
  const long groups = W->G < M_total ? W->G : M_total;
  if (W->K >= 2048 || (W->K >= 1408 && groups * (W->N / 256) > 640)) return true;
  return W->K >= 256 && (groups + M_total / cq_route::kPassRows) * (W->N / 64) <= W->K + 64;
}
long rows_in_passes(const cq_codebook_weights* W) { return (cq_tables_per_row(W) > 1 ? 23L : 28L) * W->G; }
bool streams_in_passes(const cq_codebook_weights* W, int M_total, int max_group_rows) {
  if (W->K <= 2048 && (cq_tables_per_row(W) > 1 || !short_k_in_passes(W, M_total))) return false;
  return row_bound(M_total, max_group_rows) <= 128 && (long)M_total < rows_in_passes(W);
}

// Whether a K range of ksteps steps runs the streaming kernel's pipelined unit loop: 8 or 7 steps for every wavefront,
// or (one table per row) up to 4 with empty ones in between.
bool pipelined(int ksteps, bool blockwise) {
  return ksteps == 8 * kWaves || (!blockwise && (ksteps == 7 * kWaves || ksteps <= 4 * kWaves));
}

}  // namespace


// K split of the streaming kernel.  One workgroup keeps the activations of its K range in LDS for all
// its 64-row units; with few tokens (the decode regime) a long K (the down projection) is therefore cut
// into ranges of at most 4096 that different workgroups stream, and their partial sums are added in a
// fixed order afterwards.  Plain products only (a nonlinear epilogue needs the whole sum).
// Block-wise tables on the streaming kernel's pipelined loop: tables of 1024 weights (two K steps per wavefront
// and table), up to 32 rows (more where streams_in_passes says so; in passes either way), and K ranges of whole
// tables that give every wavefront exactly 8 steps (4096 weights) or 4 (2048); a nonlinear epilogue needs all of K in one
// range.
bool cq_gemm_blockwise_streams(const cq_codebook_weights* W, int M_total, int epilogue, int max_group_rows) {
  if (kWaves != 8 || cq_is_w2(W) || W->group_k != 1024 || W->K % 2048 != 0) return false;
  if (row_bound(M_total, max_group_rows) > 32 && !streams_in_passes(W, M_total, max_group_rows)) return false;
  return epilogue == CQ_EPI_NONE || W->K == 4096;
}

namespace {
// Block-wise tables on the large-tile kernel, one workgroup per 256 rows and group of tokens.  With at most 64 rows in all
// (one 64-token tile per group) and a short N there are too few of those to fill the chip, so K is cut into ranges of whole
// table groups, up to about two workgroups per compute unit.
void blockwise_tile_plan(const cq_codebook_weights* W, int M_total, int epilogue, int* ksplit, int* ksteps) {
  *ksplit = 1;
  *ksteps = W->K / 64;
  if (epilogue != CQ_EPI_NONE || M_total > 64 || !cq_gemm_large_supported(W)) return;
  const int nblk = cq_tables_per_row(W);
  const long wgs = (long)(W->G < M_total ? W->G : M_total) * (W->N / 256);
  long want = wgs > 0 ? 512 / wgs : 1;
  if (want > nblk) want = nblk;
  if (want <= 1) return;
  const int per = (nblk + (int)want - 1) / (int)want;   // table groups per range
  *ksteps = per * (W->group_k / 64);
  *ksplit = (nblk + per - 1) / per;
}

size_t partials_bytes(const cq_codebook_weights* W, int M_total, int ksplit) {
  return ksplit > 1 ? cq_align_up((size_t)ksplit * M_total * W->N * sizeof(float), 256) : 0;
}
}  // namespace

void cq_gemm_split_plan(const cq_codebook_weights* W, int M_total, int epilogue, int* ksplit, int* ksteps,
                        int max_group_rows) {
  const int nS = W->K / 64;
  *ksplit = 1;
  *ksteps = nS;
  const int nblk = cq_tables_per_row(W);
  if (nblk > 1 && cq_gemm_blockwise_streams(W, M_total, epilogue, max_group_rows)) {
    *ksteps = W->K % 4096 == 0 ? 64 : 32;
    *ksplit = nS / *ksteps;
    return;
  }
  if (nblk > 1) return blockwise_tile_plan(W, M_total, epilogue, ksplit, ksteps);
  if (epilogue != CQ_EPI_NONE || M_total > 256 || nS <= 64) return;
  const int want = (nS + 63) / 64;
  const int per = ((nS + want - 1) / want + kWaves - 1) / kWaves * kWaves;  // whole rounds of the wavefronts
  *ksteps = per;
  *ksplit = (nS + per - 1) / per;
}

size_t cq_gemm_partials_bytes(const cq_codebook_weights* W, int M_total, int epilogue, int max_group_rows) {
  if (cq_is_w2(W)) return epilogue == CQ_EPI_NONE ? cq_gemm_w2_partials_bytes(W, M_total) : 0;
  int ksplit, ksteps;
  cq_gemm_split_plan(W, M_total, epilogue, &ksplit, &ksteps, max_group_rows);
  return partials_bytes(W, M_total, ksplit);
}

// The grouping by expert can be folded into a launch when every workgroup of it runs the pipelined unit loop
// (at most 32 rows per group, a K range that it takes) and one lane per assignment
// suffices: at most 32 tokens (a group has at most one row per token), at most 64 assignments and experts.
bool cq_gemm_can_fuse_route(const cq_codebook_weights* W, int T, int E, int S, int top_k, int epilogue) {
  if (kWaves != 8) return false;
  if (T < 1 || T > 32 || top_k < 1 || T * top_k > 64 || E < 1 || E > 64 || S < 0 || W->G != E + S) return false;
  // (the 2-bit kernel takes every group of a launch it supports: its workgroups all derive their rows alike)
  if (cq_is_w2(W)) return cq_gemm_w2_supported(W, CQ_A_INT8_CODES, epilogue);
  const int M_total = T * (top_k + S);
  if (cq_tables_per_row(W) > 1 && !cq_gemm_blockwise_streams(W, M_total, epilogue, T)) return false;
  if (cq_gemm_uses_large_tiles(W, M_total, epilogue, T)) return false;
  int ksplit, ksteps;
  cq_gemm_split_plan(W, M_total, epilogue, &ksplit, &ksteps, T);
  return ksplit == 1 && pipelined(ksteps, cq_tables_per_row(W) > 1);
}

cq_status cq_gemm_codebook_launch(const cq_codebook_weights* W, const void* A, int a_kind, const float* row_scale,
                                  const int32_t* row_gather, const int32_t* group_offsets, int M_total,
                                  int epilogue, void* out, int out_kind, void* workspace, hipStream_t s,
                                  int* ksplit_left, const cq_route_fuse* route, int max_group_rows, long a_rows) {
  if (route && !cq_gemm_can_fuse_route(W, route->T, route->E, route->S, route->top_k, epilogue))
    return CQ_ERR_UNSUPPORTED;
  if (cq_is_w2(W))
    return cq_gemm_w2_launch(W, A, a_kind, row_scale, row_gather, group_offsets, M_total, epilogue, out, out_kind,
                             workspace, s, ksplit_left, route);
  if (ksplit_left) *ksplit_left = 1;
  GemmArgs a;
  a.route = route ? *route : cq_route_fuse{nullptr, 0, 0, 0, 0, nullptr, nullptr, nullptr, nullptr};
  a.idx = W->prepacked ? (const uint8_t*)W->prepacked : W->idx;
  a.cent = W->cent;
  a.prepacked = W->prepacked ? 1 : 0;
  a.N = W->N;
  a.K = W->K;
  a.A = A;
  a.row_scale = row_scale;
  a.row_gather = row_gather;
  a.group_offsets = group_offsets;
  a.out = out;
  a.out_ld = epilogue == CQ_EPI_SWIGLU ? W->N / 2 : W->N;
  {
    // about one workgroup per compute unit: the per-workgroup prologue (activation staging, first
    // table, ring fill) is paid once and there is no partially filled last round of workgroups
    cq_gemm_split_plan(W, M_total, epilogue, &a.ksplit, &a.ksteps, max_group_rows);
    a.partials = (float*)workspace;  // partial sums first, then the large-tile kernel's
    a.part_stride = (size_t)M_total * W->N;
    // The kernel itself divides these workgroups among the groups that have rows (cq_route::pick_group).  Up to 32
    // such groups share one round of them evenly enough; with more, the whole number of workgroups per group can
    // leave a good part of the chip idle (129 groups: one workgroup each on 256 compute units), so the grid has room
    // for two or four rounds of which the kernel uses what is cheapest.
    const bool large_too = cq_gemm_uses_large_tiles(W, M_total, epilogue, max_group_rows);
    const int pass_rows = cq_tables_per_row(W) > 1 && a.ksteps == 8 * kWaves ? kBlockwisePassRows : cq_route::kPassRows;
    const int n_max = (W->G < M_total ? W->G : M_total) + M_total / pass_rows;   // passes over groups with rows
    // Where the pipelined loop is not available (other K), a group of 17..32 rows runs the plain loop on one
    // set of workgroups, several times slower per unit than the small groups around it: many short workgroups
    // then, so that the compute units the small groups leave early take the rest of the big ones.
    const int target = row_bound(M_total, max_group_rows) > 16 && !pipelined(a.ksteps, cq_tables_per_row(W) > 1) ? 1024 : 256;
    a.G = W->G;
    a.slots = target / a.ksplit > 1 ? target / a.ksplit : 1;
    a.rounds = target != 256 || (n_max <= 32 && !large_too) ? 1 : n_max <= 256 ? 2 : 4;
    a.grid = a.slots * a.rounds > n_max ? a.slots * a.rounds : n_max;
  }
  // Groups of up to 32 rows go to the streaming kernel above; larger ones to the large-tile kernel (when
  // the row count allows its 256-row tiles), which derives its token tiles from the group offsets.  Block-wise tables
  // go to the large-tile kernel with every group, except tables of 1024 weights at decode sizes, which the
  // streaming kernel's pipelined loop takes (cq_gemm_blockwise_streams).
  const bool bw_streams = cq_gemm_blockwise_streams(W, M_total, epilogue, max_group_rows) && cq_tables_per_row(W) > 1;
  const bool blockwise = cq_tables_per_row(W) > 1 && !bw_streams;
  const bool large = cq_gemm_uses_large_tiles(W, M_total, epilogue, max_group_rows);
  if (blockwise && !large) return CQ_ERR_UNSUPPORTED;
  // (the converted copy of A, and rows that are not gathered, are M_total)
  const bool converts = a_kind == CQ_A_INT8_CODES || a_kind == CQ_A_F32;
  const bool half = large && cq_gemm_uses_half_tiles(W, M_total, converts || !row_gather ? M_total : a_rows);
  // Where large tiles run anyway, they take the small groups as well and the streaming launch falls away if that is the
  // cheaper: with a short K always where the batch does not stream in passes (gate/up + down at 40 tokens, before they did:
  // DeepSeek-V2-Lite shape 92 us against 105 us in two launches, Qwen3 shape 46 against 78), with a long one from 28 rows per
  // group on (Mixtral shape at 64 tokens 245 against 172 us, at 96 tokens 241 against 246, at 128 tokens the whole layer 290
  // against 302).
  const bool no_small = blockwise || (half && (W->K <= 2048 || (long)M_total >= 28L * W->G)) ||
                        (large && !half && (long)M_total >= 384L * W->G);
  const int small_max = no_small ? 0 : kSmallMaxRows;
  const int qt = bw_streams ? W->group_k / 512 : 0;
  a.max_rows = large ? small_max : 0x7fffffff;
  void* large_ws = (char*)workspace + cq_gemm_partials_bytes(W, M_total, epilogue, max_group_rows);
  cq_status st;
  if (blockwise) {
    // (with a K split the kernel stores fp32 partial sums, per split, where the streaming kernel would)
    st = cq_gemm_large_launch(W, A, a_kind, row_scale, row_gather, group_offsets, M_total, small_max, epilogue,
                              a.ksplit > 1 ? (void*)a.partials : out, a.ksplit > 1 ? CQ_OUT_F32 : out_kind, large_ws, s, false);
    if (st != CQ_OK || a.ksplit == 1) return st;
    if (ksplit_left) {
      *ksplit_left = a.ksplit;  // the caller adds the partial sums itself
      return st;
    }
    const dim3 grid((W->N / 4 + 255) / 256, W->G, 16);   // (z: up to 16 rows of a group at a time)
    if (out_kind == CQ_OUT_F16)
      hipLaunchKernelGGL(sum_partials_kernel<CQ_OUT_F16>, grid, dim3(256), 0, s, a.partials, a.part_stride, a.ksplit,
                         group_offsets, 0x7fffffff, W->N, out);
    else
      hipLaunchKernelGGL(sum_partials_kernel<CQ_OUT_F32>, grid, dim3(256), 0, s, a.partials, a.part_stride, a.ksplit,
                         group_offsets, 0x7fffffff, W->N, out);
    return cq_check_launch();
  }
  if (no_small)
    return cq_gemm_large_launch(W, A, a_kind, row_scale, row_gather, group_offsets, M_total, 0, epilogue, out, out_kind,
                                large_ws, s, half);
  switch (a_kind) {
    case CQ_A_INT8_CODES: st = cq_gemm_small_dispatch_int8(a, qt, epilogue, out_kind, s); break;
    case CQ_A_F16: st = cq_gemm_small_dispatch_f16(a, qt, epilogue, out_kind, s); break;
    case CQ_A_BF16: st = cq_gemm_small_dispatch_bf16(a, qt, epilogue, out_kind, s); break;
    default: st = cq_gemm_small_dispatch_f32(a, qt, epilogue, out_kind, s); break;
  }
  if (st != CQ_OK) return st;
  if (a.ksplit > 1) {
    if (ksplit_left && !large) {
      *ksplit_left = a.ksplit;  // the caller adds the partial sums itself (they are all there is)
    } else {
      const dim3 grid((W->N / 4 + 255) / 256, W->G, 16);   // (z: up to 16 rows of a group at a time)
      if (out_kind == CQ_OUT_F16)
        hipLaunchKernelGGL(sum_partials_kernel<CQ_OUT_F16>, grid, dim3(256), 0, s, a.partials, a.part_stride, a.ksplit,
                           group_offsets, a.max_rows, W->N, out);
      else
        hipLaunchKernelGGL(sum_partials_kernel<CQ_OUT_F32>, grid, dim3(256), 0, s, a.partials, a.part_stride, a.ksplit,
                           group_offsets, a.max_rows, W->N, out);
      st = cq_check_launch();
      if (st != CQ_OK) return st;
    }
  }
  if (!large) return st;
  return cq_gemm_large_launch(W, A, a_kind, row_scale, row_gather, group_offsets, M_total, kSmallMaxRows, epilogue,
                              out, out_kind, large_ws, s, half);
}


bool cq_gemm_can_use_large_tiles(const cq_codebook_weights* W, int M_total, int max_group_rows) {
  // no group can have more rows than the streaming kernel takes: nothing for the large tiles to do
  if (cq_tables_per_row(W) == 1 && max_group_rows > 0 && max_group_rows <= kSmallMaxRows) return false;
  return !cq_is_w2(W) && cq_gemm_large_supported(W) && (M_total > kSmallMaxRows || cq_tables_per_row(W) > 1);
}

bool cq_gemm_uses_large_tiles(const cq_codebook_weights* W, int M_total, int epilogue, int max_group_rows) {
  if (cq_tables_per_row(W) > 1 && cq_gemm_blockwise_streams(W, M_total, epilogue, max_group_rows)) return false;
  if (cq_tables_per_row(W) == 1 && !cq_is_w2(W) && streams_in_passes(W, M_total, max_group_rows)) {
    int ksplit, ksteps;
    cq_gemm_split_plan(W, M_total, epilogue, &ksplit, &ksteps, max_group_rows);
    if (pipelined(ksteps, false)) return false;
  }
  return cq_gemm_can_use_large_tiles(W, M_total, max_group_rows);
}

size_t cq_gemm_product_bytes(const cq_codebook_weights* W, int M_total, int epilogue, int rows_per_token, bool with_conversion) {
  const bool layer = rows_per_token > 0;
  const int per = layer ? rows_per_token : 1, units = M_total / per;   // tokens, or single rows
  const bool one_table = cq_tables_per_row(W) == 1;
  auto stream_bytes = [&](int u) { return cq_gemm_partials_bytes(W, u * per, epilogue, layer ? u : 0); };
  auto tile_bytes = [&](int u) -> size_t {
    if (!cq_gemm_can_use_large_tiles(W, u * per, layer ? u : 0)) return 0;
    return cq_gemm_tile_list_bytes(W->G, u * per) + cq_gemm_large_workspace_bytes(W->G, u * per, W->K, with_conversion, W->N);
  };
  size_t most = 0;
  auto take = [&](size_t n) { if (n > most) most = n; };
  if (one_table) {   // a launch of both kernels; the streaming one's partial sums end with the batches of up to 256 rows
    take(stream_bytes(units) + tile_bytes(units));
    const int last = cq_is_w2(W) ? units : 256 / per;
    if (last > 0 && last < units) take(stream_bytes(last) + tile_bytes(last));
    return most;
  }
  // block-wise tables: everything streams (up to 32 rows a group, and in passes), or everything is on large tiles, whose
  // partial sums end with the launches of up to 64 rows
  take(stream_bytes(units < kSmallMaxRows ? units : kSmallMaxRows));
  long last = (rows_in_passes(W) - 1) / per;   // the most tokens that stream in passes
  if (last > 128) last = 128;
  if (last > units) last = units;
  if (last > kSmallMaxRows && cq_gemm_blockwise_streams(W, (int)last * per, epilogue, layer ? (int)last : 0))
    take(stream_bytes((int)last));
  if (units > kSmallMaxRows || !cq_gemm_blockwise_streams(W, M_total, epilogue, layer ? units : 0)) take(tile_bytes(units));
  for (int u = 1; u <= units && u * per <= 64; ++u) {
    if (u <= kSmallMaxRows && cq_gemm_blockwise_streams(W, u * per, epilogue, layer ? u : 0)) continue;
    int ksplit, ksteps;
    blockwise_tile_plan(W, u * per, epilogue, &ksplit, &ksteps);
    take(partials_bytes(W, u * per, ksplit) + tile_bytes(u));
  }
  return most;
}

extern "C" size_t cq_grouped_gemm_workspace_bytes(const cq_codebook_weights* W, int M_total) {
  if (!W || W->G <= 0 || W->N <= 0 || W->K <= 0 || M_total <= 0) return 0;
  size_t need = 0;
  for (const int epi : {CQ_EPI_NONE, CQ_EPI_SWIGLU}) {   // the kernel, and with it the need, can depend on the epilogue
    const size_t n = cq_gemm_product_bytes(W, M_total, epi, 0, true);  // worst case over the operand kinds
    if (n > need) need = n;
  }
  return need;
}

extern "C" cq_status cq_codebook_grouped_gemm(const cq_codebook_weights* W, const void* A, int a_kind,
                                              const float* row_scale, const int32_t* row_gather,
                                              const int32_t* group_offsets, int M_total, int epilogue, void* out,
                                              int out_kind, void* workspace, size_t workspace_bytes,
                                              cq_stream stream) {
  if (!W || !A || !group_offsets || (!out && M_total > 0)) return CQ_ERR_NULL;
  if ((!W->idx && !W->prepacked) || !W->cent) return CQ_ERR_NULL;
  if (W->G <= 0 || W->N <= 0 || W->K <= 0 || M_total < 0) return CQ_ERR_SHAPE;
  if (W->N % 64 != 0 || W->K % 64 != 0 || W->group_k < 0) return CQ_ERR_SHAPE;
  if (W->index_bits != 0 && W->index_bits != 4 && W->index_bits != 2) return CQ_ERR_UNSUPPORTED;
  if (cq_is_w2(W) && !cq_gemm_w2_supported(W, a_kind, epilogue)) return CQ_ERR_UNSUPPORTED;
  if (cq_tables_per_row(W) > 1 && !cq_gemm_large_supported(W)) return CQ_ERR_UNSUPPORTED;
  if (a_kind != CQ_A_INT8_CODES && a_kind != CQ_A_F16 && a_kind != CQ_A_F32 && a_kind != CQ_A_BF16)
    return CQ_ERR_UNSUPPORTED;
  if (epilogue != CQ_EPI_NONE && epilogue != CQ_EPI_SWIGLU) return CQ_ERR_UNSUPPORTED;
  if (out_kind != CQ_OUT_F32 && out_kind != CQ_OUT_F16) return CQ_ERR_UNSUPPORTED;
  if (M_total == 0) return CQ_OK;
  {
    const size_t need = cq_grouped_gemm_workspace_bytes(W, M_total);
    if (need > 0 && (!workspace || workspace_bytes < need)) return CQ_ERR_WORKSPACE;
  }
  return cq_gemm_codebook_launch(W, A, a_kind, row_scale, row_gather, group_offsets, M_total, epilogue, out,
                                 out_kind, workspace, (hipStream_t)stream, nullptr);
}
