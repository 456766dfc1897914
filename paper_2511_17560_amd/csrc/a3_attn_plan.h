// The layout of the attention's work (Eq. 4 / Eq. 5, last line): which workgroup attends which part of which tile
// of active rows.  It depends only on the list of active rows, so it is made right behind the selection (one
// workgroup) - by a kernel of its own, or at the tail of the kernel that selects (a3_topk.hip).  Shared by
// a3_attn.hip and a3_topk.hip; device code is inlined into both (no relocatable device code).
#pragma once

#include "a3_attn_stream.h"
#include "a3_internal.h"

namespace {

constexpr int kTM = 256;            // packed (row, head) pairs per work item: 32 per wave of the attention kernel
// Key steps of a share, at least (2K context: 37 us with 8, 33 with 4 or less).  Two for requests of up to 768 rows were faster (500 rows at
// 15 % 19.1 -> 15.8 us, 512 in a chunk's precompute 24.0 -> 18.7) but give other cuts, whose error against float64 is larger in places:
// 4 x 400 rows 1.963e-3 -> 1.978e-3, 1.799e-3 -> 1.823e-3 with a few large weights, precompute of 200 rows 7.026e-3 -> 7.037e-3
constexpr int kMinSteps = 4;
constexpr int kPlanThreads = 1024;
constexpr int kOneShares = 64;      // shares that one wave can lay out
constexpr size_t kFirstBytes = (size_t)kOneShares * 2 * sizeof(int4);      // room for their first items (attn_plan::wg_first)
constexpr int kPlanLdsInts = 6144;  // LDS the plan kernel sets aside for the plan's small arrays (24 KB)

// Work decomposition written by the plan kernel.
//   tile  = 256 consecutive packed (row, head) pairs of one request and one KV head group; it needs
//           ceil(visible keys of its last row / 64) key steps
//   The key steps of all tiles, laid end to end, are cut into P equal shares, one per workgroup of a
//   KV head (P = workgroups per head, at most one share per kMinSteps steps): every workgroup gets the same
//   amount of work whatever the mix of short and long tiles.
//   item  = the part of one share that lies in one tile: (tile, k_begin, k_end).  A tile that lies inside
//           one share is finished by that workgroup; the others are cut into 2 or more items whose
//           unnormalised partial results are merged afterwards, in key order.
struct attn_item { int k_begin, k_end, kv_len, m0, m_end, a0, base, whole; };   // whole: the tile's only item
struct attn_plan {
  int *a_lo;         // [n_req+1] first active row of each request
  int *tile_start;   // [n_req+1] first tile of each request
  int4 *tile_a;      // [max_tiles] (first active row of the request, first m, visible keys of the last row, rows*G of the request)
  int2 *tile_b;      // [max_tiles] (first item, number of items)
  int *tile_pre;     // [max_tiles+1] key steps of all earlier tiles
  int4 *items;       // [max_items][2] all the attention kernel needs of an item (attn_item), in work order
  int *wg_start;     // [max_wgs+1] first item of each workgroup of a head
  int4 *wg_first;    // [max_wgs][2] that item again, at a place that a workgroup knows without looking wg_start up; NULL above
                     // kOneShares workgroups
  int *counters;     // n_tiles, n_items, P, max_wgs the plan was made with (first in the workspace: its place
                     // does not depend on the sizes of the other arrays)
  float *part_o;     // [Hkv * max_items][16 rows x 16][16 dims x 8][lane][4] unnormalised partial O of cut tiles: lane (l16, lg)
                     // holds row l16, dims 4 lg .. + 3 of a block
  float2 *part_ml;   // [Hkv * max_items][256]      (exponent reference in the exp2 domain, sum)
  int max_tiles, max_items, max_wgs;
};

__device__ __forceinline__ int lower_bound_i32(const int *__restrict__ a, int n, int x) {
  int lo = 0, hi = n;            // first index with a[i] >= x
  while (lo < hi) {
    int mid = (lo + hi) >> 1;
    if (a[mid] < x) lo = mid + 1; else hi = mid;
  }
  return lo;
}
__device__ __forceinline__ int upper_bound_i32(const int *a, int n, int x) {
  int lo = 0, hi = n;            // first index with a[i] > x
  while (lo < hi) {
    int mid = (lo + hi) >> 1;
    if (a[mid] <= x) lo = mid + 1; else hi = mid;
  }
  return lo;
}

// Barrier between the steps of the plan: what they hand on lies in LDS, or in the workspace
template <bool in_lds>
__device__ __forceinline__ void plan_barrier() {
  if constexpr (in_lds) A3_LDS_BARRIER();
  else __syncthreads();
}

// exclusive prefix sum over the workgroup (threads in tid order); *total receives the sum.  wave_tot: [kPlanThreads / 64]
template <bool in_lds>
__device__ __forceinline__ int plan_scan(int v, int *wave_tot, int *total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int inc = a3_wave_prefix(v);
  plan_barrier<in_lds>();        // wave_tot may still be read by a previous scan
  if (lane == 63) wave_tot[wave] = inc;
  plan_barrier<in_lds>();
  static_assert(kPlanThreads == 16 * 64, "16 waves");
  return a3_waves_before(wave_tot, *total) + inc - v;
}

// The whole plan, by one workgroup of kPlanThreads threads.  wave_tot: [kPlanThreads / 64] ints of LDS.
// lds: lds_ints ints of LDS.  The searches below each are a chain of dependent reads; when the small arrays they
// run over (row range, first tile and first row of each request, running cost, key count and request of each tile) fit
// there, they are kept in LDS beside their copies in the workspace (which the attention kernels read) and the chains run
// at LDS latency instead of a round trip to the L2 per step.  A layout of its own for each of the two, so that the reads are known
// to be of LDS: one that might be of memory waits for the stores of the item before it (plan of eight requests of 8000 rows 18.2 ->
// 14.5 us, of 64K context 12.7 -> 10.7, of 16 x 500 rows 11.8 -> 9.3; the request of an item taken from its tile instead of a
// bisection is 2.0, 0.3 and 0.6 us of that).
// row(i): act_idx[i].
template <bool in_lds, class Row>
__device__ __forceinline__ void attn_plan_layout(const attn_plan &p, const int *act_idx, Row row, int n_act,
                                                 const int *__restrict__ seg_start, int n_req, int G, int wgs_per_head,
                                                 int item_cost, int *wave_tot, int *lds) {
  const int tid = threadIdx.x;
  int *a_lo = in_lds ? lds : p.a_lo;
  int *tile_start = in_lds ? lds + (n_req + 1) : p.tile_start;
  int *tile_pre = in_lds ? lds + 3 * (n_req + 1) : p.tile_pre;
  int *tile_kv = in_lds ? lds + 3 * (n_req + 1) + p.max_tiles + 1 : nullptr;
  int *tile_req = in_lds ? tile_kv + p.max_tiles : nullptr;
  int *req_base = lds + 2 * (n_req + 1);                     // in LDS only
  const int one_base = n_req == 1 ? seg_start[0] : 0;
  auto base_of = [&](int r) { return n_req == 1 ? one_base : in_lds ? req_base[r] : seg_start[r]; };
  // active rows are ascending, so the rows of request r are a contiguous range found by bisection (a batch of one
  // request: all of them)
  for (int r = tid; r <= n_req; r += kPlanThreads) {
    const int v = r == n_req ? n_act : (r == 0 && n_req == 1 ? 0 : lower_bound_i32(act_idx, n_act, seg_start[r]));
    a_lo[r] = v;
    if (in_lds) {
      p.a_lo[r] = v;
      if (n_req > 1 && r < n_req) req_base[r] = seg_start[r];
    }
  }
  plan_barrier<in_lds>();
  if (n_req < 64) {
    if (tid < 64) {
      const int n = tid < n_req ? ((a_lo[tid + 1] - a_lo[tid]) * G + kTM - 1) / kTM : 0, t = a3_wave_prefix(n) - n;
      if (tid <= n_req) {
        tile_start[tid] = t;
        if (in_lds) p.tile_start[tid] = t;
      }
    }
  } else if (tid == 0) {
    int t = 0;
    for (int r = 0; r < n_req; ++r) {
      tile_start[r] = t;
      if (in_lds) p.tile_start[r] = t;
      t += ((a_lo[r + 1] - a_lo[r]) * G + kTM - 1) / kTM;
    }
    tile_start[n_req] = t;
    if (in_lds) p.tile_start[n_req] = t;
  }
  plan_barrier<in_lds>();
  const int n_tiles = min(tile_start[n_req], p.max_tiles);

  // ---- tiles and their running cost -------------------------------------------------------
  // A tile is laid out as `item_cost` units of start-up (fetching its queries and first keys, storing its
  // result, and the steps in which its rows end) followed by one unit per key step.
  int carry = 0;
  for (int base = 0; base < n_tiles; base += kPlanThreads) {
    const int t = base + tid;
    int steps = 0;
    if (t < n_tiles) {
      const int r = upper_bound_i32(tile_start, n_req, t) - 1;       // last r with tile_start[r] <= t
      const int j = t - tile_start[r];
      const int nr = a_lo[r + 1] - a_lo[r];
      int last = ((j + 1) * kTM - 1) / G;
      if (last > nr - 1) last = nr - 1;
      const int kv = row(a_lo[r] + last) - base_of(r) + 1;
      steps = (kv + kTK - 1) / kTK;
      p.tile_a[t] = make_int4(a_lo[r], j * kTM, kv, nr * G);
      if (in_lds) { tile_kv[t] = kv; tile_req[t] = r; }
    }
    int total;
    const int before = plan_scan<in_lds>(t < n_tiles ? steps + item_cost : 0, wave_tot, &total);
    if (t < n_tiles) {
      tile_pre[t] = carry + before;
      if (in_lds) p.tile_pre[t] = carry + before;
    }
    carry += total;
  }
  const int W = carry;                                       // cost of one head, >= n_tiles
  if (tid == 0) {
    tile_pre[n_tiles] = W;
    if (in_lds) p.tile_pre[n_tiles] = W;
  }
  plan_barrier<in_lds>();

  // ---- equal shares ------------------------------------------------------------------------
  int P = (W - n_tiles * item_cost + kMinSteps - 1) / kMinSteps;
  if (P > wgs_per_head) P = wgs_per_head;
  if (P > p.max_wgs) P = p.max_wgs;
  if (P < 1) P = 1;
  int t0 = 0, cnt = 0;
  long long s_beg = 0, s_end = 0;
  // (a 64-bit division is some 150 instructions: only where 32 bits do not hold the products)
  const bool narrow = (long long)(W + 1) * (P + 1) < (1ll << 31);
  auto quotient = [&](long long a, int b) { return narrow ? (long long)((uint32_t)a / (uint32_t)b) : a / b; };
  if (tid < P && W > 0) {
    s_beg = quotient((long long)tid * W, P);
    s_end = quotient((long long)(tid + 1) * W, P);
    if (s_end > s_beg) {
      // tiles that hold positions s_beg and s_end - 1: the last with a start <= s_beg, and < s_end (both searches at once)
      int hi0 = n_tiles + 1, t1 = 0, hi1 = n_tiles + 1;
      while (t0 < hi0 || t1 < hi1) {
        const int m0 = (t0 + hi0) >> 1, m1 = (t1 + hi1) >> 1;
        const int p0 = tile_pre[min(m0, n_tiles)], p1 = tile_pre[min(m1, n_tiles)];
        if (t0 < hi0) { if (p0 <= (int)s_beg) t0 = m0 + 1; else hi0 = m0; }
        if (t1 < hi1) { if (p1 < (int)s_end) t1 = m1 + 1; else hi1 = m1; }
      }
      t0 -= 1;
      t1 -= 1;
      // the last tile only counts if the share reaches past its start-up units
      cnt = t1 - t0 + 1 - (s_end <= (long long)tile_pre[t1] + item_cost ? 1 : 0);
    }
  }
  // (waves that have no share begin)
  // items of a tile = share boundaries strictly inside it + 1; boundary q lies at floor(q W / P)
  for (int t = (tid + kPlanThreads / 2) % kPlanThreads; t < n_tiles; t += kPlanThreads) {
    const long long x = (long long)tile_pre[t] + item_cost, y = tile_pre[t + 1];
    const long long ub = quotient((x + 1) * P + W - 1, W);   // first q with floor(q W / P) > x
    const long long lb = quotient(y * P + W - 1, W);         // first q with floor(q W / P) >= y
    p.tile_b[t].y = (int)(lb > ub ? lb - ub : 0) + 1;
  }
  int n_items;
  const int first = plan_scan<in_lds>(cnt, wave_tot, &n_items);
  if (tid < P) p.wg_start[tid] = min(first, p.max_items);
  if (tid == 0) p.wg_start[P] = min(n_items, p.max_items);
  for (int i = 0; i < cnt; ++i) {
    const int t = t0 + i, idx = first + i;
    if (idx >= p.max_items) break;
    const int pre = tile_pre[t] + item_cost, nxt = tile_pre[t + 1];      // key step s of the tile sits at pre + s
    const int it_b = (int)(s_beg > pre ? s_beg - pre : 0), it_e = (int)((s_end < nxt ? s_end : nxt) - pre);
    const int kv = in_lds ? tile_kv[t] : p.tile_a[t].z;
    const int r = n_req == 1 ? 0 : in_lds ? tile_req[t] : upper_bound_i32(tile_start, n_req, t) - 1;
    const int4 x = make_int4(it_b * kTK, min(kv, it_e * kTK), kv, (t - tile_start[r]) * kTM);
    const int4 y = make_int4((a_lo[r + 1] - a_lo[r]) * G, a_lo[r], base_of(r), it_b == 0 && s_end >= nxt);
    p.items[2 * idx] = x;
    p.items[2 * idx + 1] = y;
    if (i == 0 && p.wg_first) { p.wg_first[2 * tid] = x; p.wg_first[2 * tid + 1] = y; }
    if (it_b == 0) p.tile_b[t].x = idx;
  }
  if (tid == 0) {
    p.counters[0] = n_tiles;
    p.counters[1] = min(n_items, p.max_items);
    p.counters[2] = P;
    p.counters[3] = p.max_wgs;
  }
}
// The same plan of one request by one wave, without barriers: a lane takes consecutive tiles, then a share.  What bounds the plan is the chain
// of its steps (LDS round trips, scans), not their number: with all 16 waves in step, a barrier on either side of every scan and bisections and
// divisions for each tile's number of items, it took 10.1 thousand cycles behind the selection of 2K rows, like this 4.7.
constexpr int kOneTiles = 512;
template <class Row>
__device__ __forceinline__ void attn_plan_one(const attn_plan &p, Row row, int n_act, int base, int G, int wgs_per_head, int item_cost, int *lds) {
  if (threadIdx.x >= 64) return;
  const int lane = threadIdx.x;
  int *pre = lds, *kvs = pre + kOneTiles + 1, *parts = kvs + kOneTiles;   // running cost, visible keys, items of a tile
  auto wave_sync = [&]() {                                   // LDS in program order over the lanes
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  const int rows = n_act * G, n_tiles = min((rows + kTM - 1) / kTM, p.max_tiles), per = (n_tiles + 63) / 64;
  int sum = 0;
  for (int u = 0; u < per; ++u) {
    const int t = lane * per + u;
    if (t >= n_tiles) break;
    const int kv = row(min(((t + 1) * kTM - 1) / G, n_act - 1)) - base + 1;
    kvs[t] = kv;
    parts[t] = 0;
    p.tile_a[t] = make_int4(0, t * kTM, kv, rows);
    pre[t] = sum;
    sum += (kv + kTK - 1) / kTK + item_cost;
  }
  const int upto = a3_wave_prefix(sum), W = __builtin_amdgcn_readlane(upto, 63);     // cost of one head
  for (int u = 0; u < per; ++u)
    if (lane * per + u < n_tiles) pre[lane * per + u] += upto - sum;
  if (lane == 0) {
    pre[n_tiles] = W;
    p.a_lo[0] = p.tile_start[0] = 0;
    p.a_lo[1] = n_act;
    p.tile_start[1] = n_tiles;
  }
  wave_sync();
  const int P = max(1, min((W - n_tiles * item_cost + kMinSteps - 1) / kMinSteps, min(wgs_per_head, p.max_wgs)));
  // share q: positions floor(q W / P) .. floor((q + 1) W / P) - 1
  const uint32_t each = (uint32_t)W / (uint32_t)P, rest = (uint32_t)W - each * (uint32_t)P;
  const int s_beg = (int)((uint32_t)lane * each + (uint32_t)lane * rest / (uint32_t)P);
  const int s_end = (int)((uint32_t)(lane + 1) * each + (uint32_t)(lane + 1) * rest / (uint32_t)P);
  int t0 = 0, cnt = 0;
  if (lane < P && s_end > s_beg) {
    // tiles that hold positions s_beg and s_end - 1: the last with a start <= s_beg, and < s_end (both searches at once)
    int hi0 = n_tiles + 1, t1 = 0, hi1 = n_tiles + 1;
    while (t0 < hi0 || t1 < hi1) {
      const int m0 = (t0 + hi0) >> 1, m1 = (t1 + hi1) >> 1;
      const int p0 = pre[min(m0, n_tiles)], p1 = pre[min(m1, n_tiles)];
      if (t0 < hi0) { if (p0 <= s_beg) t0 = m0 + 1; else hi0 = m0; }
      if (t1 < hi1) { if (p1 < s_end) t1 = m1 + 1; else hi1 = m1; }
    }
    t0 -= 1;
    t1 -= 1;
    // the last tile only counts if the share reaches past its start-up units
    cnt = t1 - t0 + 1 - (s_end <= pre[t1] + item_cost ? 1 : 0);
  }
  const int all = a3_wave_prefix(cnt), first = all - cnt, n_items = min(__builtin_amdgcn_readlane(all, 63), p.max_items);
  if (lane < P) p.wg_start[lane] = min(first, p.max_items);
  if (lane == 0) {
    p.wg_start[P] = n_items;
    p.counters[0] = n_tiles;
    p.counters[1] = n_items;
    p.counters[2] = P;
    p.counters[3] = p.max_wgs;
  }
  for (int i = 0; i < cnt; ++i) {
    const int t = t0 + i, idx = first + i;
    if (idx >= p.max_items) break;
    const int at = pre[t] + item_cost, nxt = pre[t + 1], kv = kvs[t];    // key step s of the tile sits at `at` + s
    const int it_b = max(s_beg - at, 0), it_e = min(s_end, nxt) - at;
    const int4 x = make_int4(it_b * kTK, min(kv, it_e * kTK), kv, t * kTM), y = make_int4(rows, 0, base, it_b == 0 && s_end >= nxt);
    p.items[2 * idx] = x;
    p.items[2 * idx + 1] = y;
    if (i == 0) { p.wg_first[2 * lane] = x; p.wg_first[2 * lane + 1] = y; }
    if (it_b == 0) p.tile_b[t].x = idx;
    atomicAdd(&parts[t], 1);
  }
  wave_sync();
  for (int t = lane; t < n_tiles; t += 64) p.tile_b[t].y = parts[t];
}

template <class Row>
__device__ __forceinline__ void attn_plan_body(const attn_plan &p, const int *act_idx, Row row, int n_act,
                                               const int *__restrict__ seg_start, int n_req, int G, int wgs_per_head,
                                               int item_cost, int *wave_tot, int *lds, int lds_ints) {
  if (n_req == 1 && ((long long)n_act * G + kTM - 1) / kTM <= kOneTiles && wgs_per_head <= kOneShares && p.max_wgs <= kOneShares &&
      3 * kOneTiles + 1 <= lds_ints) {
    attn_plan_one(p, row, n_act, seg_start[0], G, wgs_per_head, item_cost, lds);
    return;
  }
  const bool fits = 3 * (n_req + 1) + 3 * p.max_tiles + 1 <= lds_ints;
  if (fits) attn_plan_layout<true>(p, act_idx, row, n_act, seg_start, n_req, G, wgs_per_head, item_cost, wave_tot, lds);
  else attn_plan_layout<false>(p, act_idx, row, n_act, seg_start, n_req, G, wgs_per_head, item_cost, wave_tot, lds);
}


int attn_max_tiles(const a3_layout *L, int n_act) {
  const int G = L->n_q_heads / L->n_kv_heads;
  return (int)(((long long)n_act * G + kTM - 1) / kTM) + L->n_req;
}

// Workgroups per KV head: one per CU over all heads (256 CUs), or the tuning value "attn_wgs".
int attn_wgs_per_head(const a3_layout *L) {
  int w = (256 + L->n_kv_heads - 1) / L->n_kv_heads;
  const int v = a3_knob(A3_KNOB_ATTN_WGS);
  if (v >= 1 && v <= kPlanThreads) w = v;
  return w;
}

// Start-up cost of an item in key steps (what the share boundaries are balanced with), or the tuning value
// "attn_item_cost".  Long shares, with 4, 8 and 10: 64K context 2801, 2746 and 2722 us, seven heads per KV head at 32K 1236, 1198 and
// 1205, all rows of 16K 1712, 1654 and 1664 (the last steps of a tile, where rows end one wave after the other, and the change of
// rows take 20 - 25 thousand cycles, a step 2660); all rows of 5000 217 and 205, 3 x 5000 130 and 125.
// In shares of few steps a tile's start-up overlaps the loads of the others, and 4 is no slower.  Whole calls of 15 % of the
// rows with 4 and 8 (seven heads per KV head): 500 rows 27.3 and 28.3 us (25.7, 27.8), 3000 41.8 and 42.3 (38.5, 39.2), 5000 60.2 and
// 61.2 (54.0, 54.6), 5500 62.8 and 63.8 (59.1, 60.0), 6000 72.6 and 72.7 (63.0, 64.2), but 6500 79.9 and 77.6 (70.5, 69.5), 8000 99.1
// and 97.9 (91.0, 89.3): the line lies at 22 steps a share, rows taken to see half of the longest request each.
// Requests of up to 4608 rows keep 4 also in longer shares.  Some batches of them would be faster with 8 (8 x 1000 rows 56.5 and 48.3,
// seven heads 51.7 and 52.5; 16 x 500 63.8 and 59.5, 42.8 and 42.8; 4 x 2000 63.1 and 59.8, 57.6 and 55.5), but fewer cuts of
// these short rows mean a larger error against float64, nowhere a smaller one: 500 rows 1.732e-3 and 1.750e-3, with a few large
// weights 1.858e-3 and 1.881e-3; 8 x 1000 2.017e-3 and 2.021e-3, 1.951e-3 and 1.968e-3; 4 x 2000 1.992e-3 and 1.993e-3, 1.994e-3 and
// 2.011e-3.  Longer ones differ by less, both ways (8000 rows 2.006e-3 and 2.003e-3, 16K 2.035e-3 and 2.036e-3).
constexpr int kShortRequestRows = 4608, kShortShareSteps = 22;
int attn_item_cost(const a3_layout *L, int n_act) {
  const int v = a3_knob(A3_KNOB_ATTN_ITEM_COST), len = L->max_ctx_len + L->max_q_len;
  if (v >= 0 && v <= 64) return v;
  const double steps = (double)n_act * (L->n_q_heads / L->n_kv_heads) / kTM * len / kTK / 2 / attn_wgs_per_head(L);
  return len <= kShortRequestRows || steps < kShortShareSteps ? 4 : 8;
}

// every tile starts an item, every share boundary inside a tile starts another
int attn_max_items(const a3_layout *L, int n_act) { return attn_max_tiles(L, n_act) + attn_wgs_per_head(L); }


// carves the plan's arrays out of the workspace (the same way in every call that shares a plan)
inline void attn_plan_carve(const a3_layout *L, int n_act, void *ws, size_t ws_bytes, attn_plan *p) {
  const int max_tiles = attn_max_tiles(L, n_act), max_items = attn_max_items(L, n_act);
  const int wgs_per_head = attn_wgs_per_head(L);
  const int Hkv = L->n_kv_heads;
  a3_ws_cursor cur(ws, ws_bytes);
  p->counters = (int *)cur.take(4 * sizeof(int));
  p->a_lo = (int *)cur.take((size_t)(L->n_req + 1) * sizeof(int));
  p->tile_start = (int *)cur.take((size_t)(L->n_req + 1) * sizeof(int));
  p->tile_a = (int4 *)cur.take((size_t)max_tiles * sizeof(int4));
  p->tile_b = (int2 *)cur.take((size_t)max_tiles * sizeof(int2));
  p->tile_pre = (int *)cur.take((size_t)(max_tiles + 1) * sizeof(int));
  p->items = (int4 *)cur.take((size_t)max_items * 2 * sizeof(int4));
  p->wg_start = (int *)cur.take((size_t)(wgs_per_head + 1) * sizeof(int));
  p->part_o = (float *)cur.take((size_t)max_items * Hkv * kTM * 128 * sizeof(float));
  p->part_ml = (float2 *)cur.take((size_t)max_items * Hkv * kTM * sizeof(float2));
  p->wg_first = wgs_per_head <= kOneShares ? (int4 *)cur.take((size_t)wgs_per_head * 2 * sizeof(int4)) : nullptr;     // kFirstBytes at most
  p->max_tiles = max_tiles; p->max_items = max_items; p->max_wgs = wgs_per_head;
}

}  // namespace
