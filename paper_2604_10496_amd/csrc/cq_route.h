// Device helpers of the routing step (a4) shared by the routing kernels and the decode front end:
// order-preserving logit keys and the wavefront top-k with softmax over the selected logits.
#pragma once
#include "cq_internal.h"

namespace cq_route {

// Order-preserving key of a logit.  -0 is folded into +0 first (they are equal logits: the lower expert id
// wins), and a NaN, whatever its sign, gets the smallest key (it is never preferred to a number).
__device__ __forceinline__ uint32_t order_key(float x) {
  if (x != x) return 0u;
  const uint32_t u = __float_as_uint(x + 0.0f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ uint64_t lanemask_lt(int lane) { return (1ull << lane) - 1ull; }

// Top-k of one token by one wavefront.  val[s] is the logit of expert s*64 + lane.  Called by all
// wavefronts of the workgroup together (it contains workgroup barriers); sk/si/sv/ss are this
// wavefront's 64-entry LDS scratch arrays.  Writes ids (descending logit, ties -> lower id) and the
// softmax over the selected logits.
template <int NSLOT>
__device__ __forceinline__ void wave_topk(const float (&val)[NSLOT], int nslot, int E, int k, bool active, int lane,
                                          uint32_t* sk, int* si, float* sv, float* ss, int32_t* ids_out,
                                          float* w_out) {
  const uint64_t lt = lanemask_lt(lane);
  uint32_t key[NSLOT];
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) key[s] = (s < nslot && (s * 64 + lane) < E) ? order_key(val[s]) : 0u;
  // k-th largest key: keep the largest prefix such that at least k keys are >= it.
  uint32_t kth = 0u;
  for (int bit = 31; bit >= 0; --bit) {
    const uint32_t cand = kth | (1u << bit);
    int cnt = 0;
#pragma unroll
    for (int s = 0; s < NSLOT; ++s)
      if (s < nslot) cnt += __popcll(__ballot((s * 64 + lane) < E && key[s] >= cand));
    if (cnt >= k) kth = cand;
  }
  int n_gt = 0;
#pragma unroll
  for (int s = 0; s < NSLOT; ++s)
    if (s < nslot) n_gt += __popcll(__ballot((s * 64 + lane) < E && key[s] > kth));
  const int need = k - n_gt;  // how many of the keys equal to kth are admitted (lowest ids first)
  int base = 0, ties_seen = 0;
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) {
    if (s < nslot) {
      const bool valid = (s * 64 + lane) < E;
      const bool eq = valid && key[s] == kth;
      const uint64_t m_eq = __ballot(eq);
      const int tie_rank = ties_seen + __popcll(m_eq & lt);
      const bool sel = valid && (key[s] > kth || (eq && tie_rank < need));
      const uint64_t m_sel = __ballot(sel);
      const int pos = base + __popcll(m_sel & lt);
      if (sel && active) {
        sk[pos] = key[s];
        si[pos] = s * 64 + lane;
        sv[pos] = val[s];
      }
      base += __popcll(m_sel);
      ties_seen += __popcll(m_eq);
    }
  }
  __syncthreads();
  if (active && lane < k) {
    const uint32_t mk = sk[lane];
    const int mi = si[lane];
    int rank = 0;
    for (int p = 0; p < k; ++p) {
      const uint32_t ok = sk[p];
      const int oi = si[p];
      rank += (ok > mk || (ok == mk && oi < mi)) ? 1 : 0;
    }
    ids_out[rank] = mi;
    ss[rank] = sv[lane];
  }
  __syncthreads();
  float ex = 0.f;
  if (active && lane < k) ex = expf(ss[lane] - ss[0]);
  float sum = ex;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
  if (active && lane < k) w_out[lane] = ex / sum;
  __syncthreads();  // the scratch arrays may be reused by the caller's next token
}

// Top-k of one token by one wavefront on its own, for at most 64 experts: lane e holds the logit of expert e.  No
// LDS and no barrier (only this wavefront's lanes take part): the k-th largest key by the same bitwise descent,
// ties admitted in ascending expert id, the selected lanes ranked by (logit descending, id ascending) against each
// other through lane reads, and one lane permutation that brings the pair of rank r to lane r.  Results as
// wave_topk writes them: ids in rank order (also to lds_ids, if given) and the softmax over the selected logits.
// Called by all 64 lanes.
__device__ __forceinline__ void wave_topk_regs(float val, int E, int k, int lane, int32_t* ids_out, float* w_out,
                                               int* lds_ids = nullptr) {
  const uint64_t lt = lanemask_lt(lane);
  const bool valid = lane < E;
  const uint32_t key = valid ? order_key(val) : 0u;
  uint32_t kth = 0u;
  for (int bit = 31; bit >= 0; --bit) {
    const uint32_t cand = kth | (1u << bit);
    if (__popcll(__ballot(valid && key >= cand)) >= k) kth = cand;
  }
  const int need = k - __popcll(__ballot(valid && key > kth));   // how many of the keys equal to kth are admitted
  const uint64_t m_eq = __ballot(valid && key == kth);
  const bool sel = valid && (key > kth || (key == kth && __popcll(m_eq & lt) < need));
  const uint64_t m_sel = __ballot(sel);
  int rank = 0;
  for (uint64_t m = m_sel; m; m &= m - 1) {
    const int j = __ffsll((long long)m) - 1;
    const uint32_t kj = (uint32_t)__builtin_amdgcn_readlane((int)key, j);
    rank += (kj > key || (kj == key && j < lane)) ? 1 : 0;
  }
  // selected lanes go to lane `rank`, the others fill the lanes from k on in order: a permutation
  const int dest = sel ? rank : k + __popcll(~m_sel & lt);
  const int id_sorted = __builtin_amdgcn_ds_permute(dest << 2, lane);
  const float v_sorted = __int_as_float(__builtin_amdgcn_ds_permute(dest << 2, __float_as_int(val)));
  const float top = __shfl(v_sorted, 0);
  const float ex = lane < k ? expf(v_sorted - top) : 0.f;
  float sum = ex;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
  if (lane < k) {
    ids_out[lane] = id_sorted;
    if (lds_ids) lds_ids[lane] = id_sorted;
    w_out[lane] = ex / sum;
  }
}

// The same for up to 128 experts, two per lane (val[s]: the logit of expert 64 s + lane): still one wavefront on its own,
// no workgroup barrier; the selected pairs are sorted through 64 entries of LDS of this wavefront's own.  Called by all 64 lanes.
__device__ __forceinline__ void wave_topk_regs2(const float (&val)[2], int E, int k, int lane, int* lds_id, float* lds_val,
                                                int32_t* ids_out, float* w_out, int* lds_ids = nullptr) {
  const uint64_t lt = lanemask_lt(lane);
  uint32_t key[2];
  bool valid[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    valid[s] = s * 64 + lane < E;
    key[s] = valid[s] ? order_key(val[s]) : 0u;
  }
  uint32_t kth = 0u;
  for (int bit = 31; bit >= 0; --bit) {
    const uint32_t cand = kth | (1u << bit);
    if (__popcll(__ballot(valid[0] && key[0] >= cand)) + __popcll(__ballot(valid[1] && key[1] >= cand)) >= k) kth = cand;
  }
  const int need = k - __popcll(__ballot(valid[0] && key[0] > kth)) - __popcll(__ballot(valid[1] && key[1] > kth));
  const uint64_t eq0 = __ballot(valid[0] && key[0] == kth), eq1 = __ballot(valid[1] && key[1] == kth);
  const bool sel[2] = {valid[0] && (key[0] > kth || (key[0] == kth && __popcll(eq0 & lt) < need)),
                       valid[1] && (key[1] > kth || (key[1] == kth && __popcll(eq0) + __popcll(eq1 & lt) < need))};
  int rank[2] = {0, 0};
#pragma unroll
  for (int s = 0; s < 2; ++s)
    for (uint64_t m = __ballot(sel[s]); m; m &= m - 1) {
      const int j = __ffsll((long long)m) - 1;
      const uint32_t kj = (uint32_t)__builtin_amdgcn_readlane((int)key[s], j);
      // (expert 64 s + j against this lane's two: of equal keys the lower id comes first)
      rank[0] += (kj > key[0] || (kj == key[0] && s == 0 && j < lane)) ? 1 : 0;
      rank[1] += (kj > key[1] || (kj == key[1] && (s == 0 || j < lane))) ? 1 : 0;
    }
#pragma unroll
  for (int s = 0; s < 2; ++s)
    if (sel[s]) {
      lds_id[rank[s]] = s * 64 + lane;
      lds_val[rank[s]] = val[s];
    }
  cq_wave_lds_fence();
  const int id_sorted = lds_id[lane < k ? lane : 0];
  const float v_sorted = lds_val[lane < k ? lane : 0];
  const float top = lds_val[0];
  const float ex = lane < k ? expf(v_sorted - top) : 0.f;
  float sum = ex;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
  if (lane < k) {
    ids_out[lane] = id_sorted;
    if (lds_ids) lds_ids[lane] = id_sorted;
    w_out[lane] = ex / sum;
  }
  cq_wave_lds_fence();   // (the entries may be reused by the caller's next token)
}

// inclusive sum over the lanes of a wavefront (data-parallel moves inside rows of 16 lanes, then across them)
__device__ __forceinline__ int wave_scan(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);    // row_shr 1, 2, 4, 8
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast 15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast 31 into rows 2 and 3
  return x;
}

// lane that holds the n-th (from 0) set bit of a ballot mask; n < popcount(mask)
__device__ __forceinline__ int nth_set_lane(uint64_t mask, int n, int lane) {
  const bool hit = ((mask >> lane) & 1ull) && __popcll(mask & lanemask_lt(lane)) == n;
  return __ffsll((long long)__ballot(hit)) - 1;
}

// Workgroups per group of a streaming launch.  n_act groups have rows, each of n_units units of work; the chip runs
// `slots` workgroups of the launch at a time and its grid holds rmax rounds of them.  With r rounds a group gets
// c = r * slots / n_act workgroups; a workgroup costs its units plus about one unit of prologue (first table, ring
// fill, activation rows), so the launch costs about r * (1 + ceil(n_units / c)): lane r - 1 prices r rounds and the
// cheapest (the fewest rounds among equals) wins.  Called by all 64 lanes; rmax is 1, 2 or 4.  (With one round there is
// nothing to price: two lane permutations less in front of the first load, 0.5 .. 1 us of the layer at 2 .. 20 tokens.)
__device__ __forceinline__ int workgroups_per_group(int n_act, int n_units, int slots, int rmax, int lane) {
  if (rmax == 1) return max(1, min(n_units, slots / n_act));
  const int r = min(lane, 3) + 1;
  const int c = min(n_units, (r * slots) / n_act);
  // (price and choice in one number: a unit of price is 2^12; prices stay below 2^19 / 4)
  uint32_t price = c >= 1 && r <= rmax ? (uint32_t)r * (1u + (uint32_t)(n_units + c - 1) / (uint32_t)c) : 0x3ffffu;
  uint32_t best = (min(price, 0x3ffffu) << 12) | ((uint32_t)r << 8);
#pragma unroll
  for (int off = 1; off < 4; off <<= 1) best = min(best, (uint32_t)__shfl_xor((int)best, off));
  best = (uint32_t)__builtin_amdgcn_readfirstlane((int)best);
  return max(1, min(n_units, (int)((best >> 8) & 15u) * slots / n_act));
}

// The group that workgroup `b` of a streaming launch works on, chosen among the groups that have between 1 and
// max_rows rows (the others cost the launch nothing: with one workgroup set per group of the layer, a batch of one
// token left three quarters of the chip without work).  A group of more than kPassRows rows counts once per kPassRows of
// them: further workgroups stream its indices again for the further rows.  Passes are counted with sums over the lanes: a
// product that has no large tiles has thousands of them (16384 rows in one group of N = 1088, K = 2048: with a ballot per
// pass in every workgroup 235 us, so 131).  Sets the group, its first row and row count (of this pass), this workgroup's
// number among the pass's workgroups and their count; false: no work for this workgroup.
// All values are uniform over the wavefront.  Called by all 64 lanes.
constexpr int kPassRows = 32;
struct group_share {
  int grp, m0, Me, chunk, chunks;
  int pass;   // (pick_group_from_ids: number of the pass within the group)
};
template <int PASS = kPassRows>
__device__ __forceinline__ bool pick_group(const int32_t* __restrict__ offsets, int G, int max_rows, int n_units,
                                           int slots, int rmax, int b, int lane, group_share& o) {
  // the offsets of the first 128 groups are requested together and stay in registers, those of further rounds of 64
  // groups are loaded again below
  int f0, r0, f1 = 0, r1 = 0;
  auto load = [&](int at, int& first, int& rows) {
    const int g = at + lane;
    first = g < G ? offsets[g] : 0;
    rows = (g < G ? offsets[g + 1] : 0) - first;
  };
  load(0, f0, r0);
  if (G > 64) load(64, f1, r1);
  auto clip = [&](int& rows) { if (rows > max_rows) rows = 0; };
  clip(r0);
  clip(r1);
  auto passes = [&](int rows) { return (rows + PASS - 1) / PASS; };
  auto sum = [&](int x) { return __builtin_amdgcn_readlane(wave_scan(x), 63); };
  auto count = [&](int rows) {   // passes over the groups of a round
    return __ballot(rows > PASS) ? sum(passes(rows)) : (int)__popcll(__ballot(rows > 0));
  };
  int n_act = count(r0);
  if (G > 64) n_act += count(r1);
  for (int at = 128; at < G; at += 64) {
    int f, r;
    load(at, f, r);
    clip(r);
    n_act += count(r);
  }
  if (n_act == 0) return false;
  o.chunks = workgroups_per_group(n_act, n_units, slots, rmax, lane);
  int n = b / o.chunks;
  if (n >= n_act) return false;
  o.chunk = b - n * o.chunks;
  int first = f0, rows = r0;
  for (int base = 0;;) {   // (n < n_act: this round or a later one has the pass)
    const int c = count(rows);
    if (n < c) {
      // the first passes of all groups come first, then the second ones, ...: pass j of all of them is preceded by as many
      // as sum(min(passes, j)); the largest j whose predecessors are no more than n, bit by bit
      int j = 0, before = 0;
      if (__ballot(rows > PASS))
        for (int step = 1 << 26; step; step >>= 1)
          if (__ballot(passes(rows) > j + step - 1)) {
            const int m = sum(min(passes(rows), j + step));
            if (m <= n) {
              j += step;
              before = m;
            }
          }
      const int src = nth_set_lane(__ballot(rows > j * PASS), n - before, lane);
      o.grp = base + src;
      o.m0 = __builtin_amdgcn_readlane(first, src) + j * PASS;
      o.Me = min(PASS, __builtin_amdgcn_readlane(rows, src) - j * PASS);
      return true;
    }
    n -= c;
    base += 64;
    if (base == 64) {
      first = f1;
      rows = r1;
    } else {
      load(base, first, rows);
      clip(rows);
    }
  }
}

// a5 folded into a product launch for decode-sized batches (cq_route_fuse): the rows of group `grp`, derived by
// one wavefront from the selected expert ids.  There are at most 64 assignments (token, choice), one per lane,
// numbered a = token * top_k + choice; the rows of expert e are the assignments that chose e, in ascending a, and
// the experts' row ranges follow each other in ascending e (the stable grouping of the routing step), so two
// ballots give the first row m0 and the row count Me, and one lane permutation hands row i's token to lane i
// (row_token).  Shared experts (grp >= E) take every token, in token order, behind the routed rows.
// writer: this wavefront also leaves offsets / perm / inv_perm / src_token behind for the launches that follow
// (exactly one wavefront of the launch must do so).  Called by all 64 lanes.
__device__ __forceinline__ void group_rows_from_ids(const cq_route_fuse& rt, int grp, int lane, bool writer, int& m0,
                                                    int& Me, int& row_token) {
  const int n_assign = rt.T * rt.top_k;
  const bool va = lane < n_assign;
  const int id = va ? rt.ids[lane] : 0x7fffffff;
  const uint64_t lt = lanemask_lt(lane);
  if (grp < rt.E) {
    const uint64_t mine = __ballot(va && id == grp);
    m0 = __popcll(__ballot(va && id < grp));
    Me = __popcll(mine);
    const int before = __popcll(mine & lt);
    // members go to lanes 0 .. Me-1 in order, the others fill the lanes behind them: a permutation
    const int dest = ((mine >> lane) & 1ull) ? before : Me + lane - before;
    row_token = __builtin_amdgcn_ds_permute(dest << 2, lane / rt.top_k);
  } else {
    m0 = n_assign + (grp - rt.E) * rt.T;
    Me = rt.T;
    row_token = lane;
  }
  if (writer) {
    int pos = 0, base = 0, my_off = 0;
    for (int e = 0; e < rt.E; ++e) {
      const uint64_t m = __ballot(va && id == e);
      if (va && id == e) pos = base + __popcll(m & lt);
      if (lane == e) my_off = base;
      base += __popcll(m);
    }
    if (lane < rt.E) rt.offsets[lane] = my_off;
    if (lane == 0) rt.offsets[rt.E] = n_assign;
    for (int sh = lane; sh < rt.S; sh += 64) rt.offsets[rt.E + sh + 1] = n_assign + (sh + 1) * rt.T;
    if (va) {
      rt.perm[pos] = lane;
      rt.inv_perm[lane] = pos;
      rt.src_token[pos] = lane / rt.top_k;
    }
    for (int i = lane; i < rt.S * rt.T; i += 64) rt.src_token[n_assign + i] = i % rt.T;
  }
}

// pick_group for a launch with the grouping folded in: the active experts are those among the selected ids (at most
// 64 experts: one bit each), and every shared expert is active; at most 2 PASS tokens, so that a group has one or two
// passes: all first ones of the experts, then all second ones, then the shared experts'.  m0 and Me come from
// group_rows_from_ids and take_pass.
template <int PASS = kPassRows>
__device__ __forceinline__ bool pick_group_from_ids(const cq_route_fuse& rt, int n_units, int slots, int rmax, int b,
                                                    int lane, group_share& o) {
  const int n_assign = rt.T * rt.top_k;
  const int id = lane < n_assign ? rt.ids[lane] : 0x7fffffff;
  uint64_t mask = 0, two = 0;   // experts with rows, and with more than a pass takes
  if (rt.E <= n_assign) {
    for (int e = 0; e < rt.E; ++e) {
      const uint64_t m = __ballot(id == e);
      if (m) mask |= 1ull << e;
      if (PASS < kPassRows && __popcll(m) > PASS) two |= 1ull << e;
    }
  } else {
    for (int a = 0; a < n_assign; ++a) mask |= 1ull << __builtin_amdgcn_readlane(id, a);
    if (PASS < kPassRows)
      for (uint64_t m = mask; m; m &= m - 1) {
        const int e = __ffsll((long long)m) - 1;
        if (__popcll(__ballot(id == e)) > PASS) two |= 1ull << e;
      }
  }
  const int n_exp = __popcll(mask), n_two = __popcll(two), per_shared = rt.T > PASS ? 2 : 1;
  const int n_all = n_exp + n_two + rt.S * per_shared;
  o.chunks = workgroups_per_group(n_all, n_units, slots, rmax, lane);
  const int n = b / o.chunks;
  if (n >= n_all) return false;
  o.chunk = b - n * o.chunks;
  o.pass = 0;
  if (n < n_exp) {
    o.grp = nth_set_lane(mask, n, lane);
  } else if (n < n_exp + n_two) {
    o.grp = nth_set_lane(two, n - n_exp, lane);
    o.pass = 1;
  } else {
    const int i = n - n_exp - n_two;
    o.grp = rt.E + (per_shared == 2 ? i >> 1 : i);
    o.pass = per_shared == 2 ? i & 1 : 0;
  }
  return true;
}

// the rows of the share's pass, from those of its group (group_rows_from_ids): row i's token moves to lane i - PASS * pass
template <int PASS>
__device__ __forceinline__ void take_pass(group_share& o, int lane, int& row_token) {
  row_token = __shfl(row_token, lane + PASS * o.pass);
  o.m0 += PASS * o.pass;
  o.Me = min(PASS, o.Me - PASS * o.pass);
}

}  // namespace cq_route
