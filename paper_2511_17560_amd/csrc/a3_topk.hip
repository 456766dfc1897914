// Step 3 of the A^3 fusion path: Re = top_p(s) (Eq. 3, second line).
//
// One workgroup of 16 wavefronts per request.  The k-th largest score is found exactly by a radix
// select on an order-preserving integer image of the float (11 bits per pass; the passes start at
// the highest bit in which the request's smallest and largest key differ), then the rows are
// compacted in index order with ballots and one sum over the waves.  Compacting in index order
// gives both rules of the selection for free: among equal scores the lowest rows are taken,
// and the output is ascending.  Integer work only: the result is unique and bit-exact.
// Requests of up to 68 K rows keep every key in a register of the lane that owns it; longer ones re-read the
// scores from global memory in every pass.  One compute unit does all of it, so what bounds it is the instructions its 16
// waves issue and the chain of barriers and LDS round trips between them: sums over lanes are data-parallel moves, a wave's part of a sum
// over waves is one read, barriers wait for LDS alone, and the rows leave through LDS in whole lines.  From the first instruction to
// the last, plan included, us (with shuffles, 16 reads a sum and full barriers -> now): 2K rows 9.0 -> 6.1, 5K 10.9 -> 8.0, 16K 16.8 -> 12.3,
// 64K 39.4 -> 33.4.
#include <type_traits>

#include "a3_internal.h"
#include "a3_attn_plan.h"

namespace {

constexpr int kBlock = 1024;
constexpr int kWaves = kBlock / 64;

// Monotone map float -> uint32 (larger float <=> larger key); -0 is folded onto +0.
__device__ __forceinline__ uint32_t score_key(float s) {
  const uint32_t b = __float_as_uint(s + 0.0f);
  return b ^ ((uint32_t)((int)b >> 31) | 0x80000000u);
}

// Exclusive prefix sum of one int per thread over the workgroup (threads in tid order).
__device__ __forceinline__ int block_exclusive_scan(int v, int *wave_tot /* [kWaves] LDS */) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int inc = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    int x = __shfl_up(inc, off, 64);
    if (lane >= off) inc += x;
  }
  __syncthreads();                       // wave_tot may still be read by a previous scan
  if (lane == 63) wave_tot[wave] = inc;
  __syncthreads();
  int before = 0;
  for (int w = 0; w < wave; ++w) before += wave_tot[w];
  return before + inc - v;
}

// Adds one to hist[bin] for every active lane.  Lanes of a wave that hit the same bin are merged
// into a single LDS atomic (the top byte of the scores takes only a handful of values, and
// thousands of same-address atomics would serialise).
__device__ __forceinline__ void hist_add_merged(uint32_t *hist, uint32_t bin, bool active) {
  unsigned long long todo = __ballot(active);
  const int lane = threadIdx.x & 63;
  while (todo) {
    const int leader = __ffsll(todo) - 1;
    const uint32_t lbin = __shfl(bin, leader, 64);
    const unsigned long long same = __ballot(active && bin == lbin);
    if (lane == leader) atomicAdd(&hist[lbin], (uint32_t)__popcll(same));
    todo &= ~same;
  }
}

// Suffix sums over the 256 bins, from the highest bin downwards, by the first wave: finds the bin
// that holds the need-th largest candidate and how many candidates of that bin are still needed.
__device__ __forceinline__ void find_bin(const uint32_t *hist, uint32_t need, uint32_t *sh_bin, uint32_t *sh_need) {
  const int tid = threadIdx.x;
  if (tid < 64) {
    uint32_t c[4], t = 0;                // lane owns bins 4*lane .. 4*lane+3
#pragma unroll
    for (int j = 0; j < 4; ++j) { c[j] = hist[4 * tid + j]; t += c[j]; }
    uint32_t suf = t;                    // sum over lanes >= this one
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      uint32_t x = __shfl_down(suf, off, 64);
      if (tid + off < 64) suf += x;
    }
    uint32_t above = suf - t;            // candidates in bins of higher lanes
#pragma unroll
    for (int j = 3; j >= 0; --j) {
      if (above < need && above + c[j] >= need) { *sh_bin = 4 * tid + j; *sh_need = need - above; }
      above += c[j];
    }
  }
}

// What one workgroup ranks.  Selection of Eq. 3: the context rows of request blockIdx.x, k from sel_start.
// Eviction extension (skip != nullptr): blockIdx.y is a KV head with its own score row and output row; the
// first skip[r] context rows (system prompt) and the question rows are retained anyway and written by
// write_fixed_rows, so the candidates start behind the system prompt, the count leaves them out, and the
// output starts behind the system prompt's slots.
struct topk_problem {
  const int *seg_start, *ctx_len, *sel_start;
  const int *skip, *q_len;
  long score_stride, out_stride;
  // a batch of one request whose lengths the host knows (the layout's maxima add up to its rows): its context
  // length and count, so that the kernel starts without a chain of loads; otherwise -1
  int one_N = -1, one_k = -1;
};

struct topk_range { int s, N, k; const float *sc; int *out; };

__device__ __forceinline__ topk_range topk_range_of(const topk_problem &p, const float *scores, int *sel_idx) {
  topk_range t;
  if (p.one_N >= 0) {
    t.s = 0; t.N = p.one_N; t.k = min(p.one_k, p.one_N);
    t.sc = scores; t.out = sel_idx;
    return t;
  }
  const int r = blockIdx.x;
  const int sk = p.skip ? p.skip[r] : 0;
  t.s = p.seg_start[r] + sk;
  t.N = max(p.ctx_len[r] - sk, 0);
  t.k = p.sel_start[r + 1] - p.sel_start[r] - (p.skip ? sk + p.q_len[r] : 0);
  if (t.k > t.N) t.k = t.N;
  t.sc = scores + (size_t)blockIdx.y * p.score_stride + t.s;
  t.out = sel_idx + (size_t)blockIdx.y * p.out_stride + p.sel_start[r] + sk;
  return t;
}

// Eviction extension: keep_idx[g][keep_start[r] + i] for the system-prompt rows (i < skip[r]) and the question rows
// (the last q_len[r] slots of the request), by the workgroup that ranks the rest.
__device__ __forceinline__ void write_fixed_rows(const topk_problem &p, int *__restrict__ keep_idx) {
  const int r = blockIdx.x;
  int *out = keep_idx + (size_t)blockIdx.y * p.out_stride;
  const int s = p.seg_start[r], N = p.ctx_len[r], nq = p.q_len[r], sk = p.skip[r];
  const int o0 = p.sel_start[r], o1 = p.sel_start[r + 1];
  // (a keep_start that does not match the rule must not send a store outside the list)
  for (int i = threadIdx.x; i < sk; i += kBlock)
    if (o0 + i >= 0 && o0 + i < p.out_stride) out[o0 + i] = s + i;
  for (int j = threadIdx.x; j < nq; j += kBlock)
    if (o1 - nq + j >= 0 && o1 - nq + j < p.out_stride) out[o1 - nq + j] = s + N + j;
}

// Requests longer than the register kernel holds: 4 x 8-bit passes from the top byte, every pass
// re-reads the scores from global memory.
__global__ void __launch_bounds__(kBlock)
topk_select_kernel(const float *__restrict__ scores, topk_problem prob, int *__restrict__ sel_idx) {
  __shared__ uint32_t hist[256];
  __shared__ int wave_tot[kWaves];
  __shared__ uint32_t sh_bin, sh_need;

  const int tid = threadIdx.x;
  if (prob.skip) write_fixed_rows(prob, sel_idx);
  const topk_range rg = topk_range_of(prob, scores, sel_idx);
  const int s = rg.s, N = rg.N, k = rg.k;
  if (k <= 0) return;                    // uniform over the workgroup
  int *__restrict__ out = rg.out;
  const float *__restrict__ sc = rg.sc;
  auto key_at = [&](int i) -> uint32_t { return score_key(sc[i]); };

  // ---- radix select: key of the k-th largest score -------------------------------------
  uint32_t prefix = 0, mask = 0, need = (uint32_t)k;
  for (int shift = 24; shift >= 0; shift -= 8) {
    if (tid < 256) hist[tid] = 0;
    __syncthreads();
    const int n_round = (N + kBlock - 1) / kBlock * kBlock;  // whole waves take part in the merged add
    for (int i = tid; i < n_round; i += kBlock) {
      const uint32_t u = i < N ? key_at(i) : 0u;
      const bool active = i < N && (u & mask) == prefix;
      const uint32_t bin = (u >> shift) & 255u;
      if (shift == 24) hist_add_merged(hist, bin, active);
      else if (active) atomicAdd(&hist[bin], 1u);
    }
    __syncthreads();
    find_bin(hist, need, &sh_bin, &sh_need);
    __syncthreads();
    prefix |= sh_bin << shift;
    mask |= 255u << shift;
    need = sh_need;
    __syncthreads();
  }
  const uint32_t tau = prefix;           // key of the k-th largest; `need` rows equal to it are taken

  // ---- ordered compaction: thread tid owns rows [lo, hi) ----------------------------------
  const int per = (N + kBlock - 1) / kBlock;
  const int lo = min(N, tid * per), hi = min(N, lo + per);
  int cnt_gt = 0, cnt_eq = 0;
  for (int i = lo; i < hi; ++i) {
    uint32_t u = key_at(i);
    cnt_gt += u > tau;
    cnt_eq += u == tau;
  }
  const int eq_before = block_exclusive_scan(cnt_eq, wave_tot);
  int take_eq = (int)need - eq_before;
  take_eq = take_eq < 0 ? 0 : (take_eq > cnt_eq ? cnt_eq : take_eq);
  int pos = block_exclusive_scan(cnt_gt + take_eq, wave_tot);
  for (int i = lo; i < hi; ++i) {
    uint32_t u = key_at(i);
    if (u > tau) out[pos++] = s + i;
    else if (u == tau && take_eq > 0) { out[pos++] = s + i; --take_eq; }
  }
}

// KPT = keys per lane (compile-time bound).  Wave w owns a contiguous block of 64 * per rows, per <= KPT a multiple
// of 4; vector q of a lane are the rows 256 q + 4 lane .. + 3 of its wave's block: every load instruction of a wave is
// 1 KB in one piece, and index order is (wave, q, lane, element).  The blocks are counted from the 16-byte boundary at
// or below the request's first score, so that every load is aligned wherever the request starts; the vectors that
// reach over an end of the request are loaded element by element.
constexpr int kBins = 2048;
constexpr uint32_t kRankKeys = 256;      // candidates that are ranked directly instead of by another round
static_assert(kBlock == 4 * kRankKeys && kWaves % 4 == 0, "a quarter of the candidates to each 256 threads");

// Maximum over a wave, in every lane
__device__ __forceinline__ uint32_t wave_max(uint32_t x) {
#define A3_STEP(CTRL, ROWS) x = max(x, (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, CTRL, ROWS, 0xf, false))
  A3_STEP(0x111, 0xf); A3_STEP(0x112, 0xf); A3_STEP(0x114, 0xf); A3_STEP(0x118, 0xf);   // as in a3_wave_prefix
  A3_STEP(0x142, 0xa); A3_STEP(0x143, 0xc);
#undef A3_STEP
  return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}
// Maximum over the numbers of 16 waves
__device__ __forceinline__ uint32_t waves_max(const uint32_t *v) {
  uint32_t x = v[threadIdx.x & 15];
#define A3_STEP(CTRL) x = max(x, (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, CTRL, 0xf, 0xf, false))
  A3_STEP(0x111); A3_STEP(0x112); A3_STEP(0x114); A3_STEP(0x118);
#undef A3_STEP
  return (uint32_t)__builtin_amdgcn_readlane((int)x, 15);
}

// Rows taken and kept in LDS until all are known: they leave in whole lines
constexpr int kListRows = 6656;

// list: LDS, [kListRows]: receives the rows instead of rg.out where they fit.
template <int KPT>
__device__ __forceinline__ void topk_select_reg_body(const topk_range &rg, int *list) {
  __shared__ __align__(16) uint32_t hist[kBins];
  __shared__ __align__(16) uint32_t wave_a[kWaves], wave_b[kWaves];
  __shared__ __align__(16) uint32_t cand[kRankKeys];
  __shared__ uint32_t above_of[kWaves / 4][kRankKeys];       // candidates above and at or above one, by shares of them
  __shared__ __align__(16) uint4 sh_found;                   // the bin (or key), how many of it are wanted, how many there are
  __shared__ uint32_t sh_cand;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = rg.N, k = rg.k;
  if (k <= 0) return;                    // uniform over the workgroup
  int *__restrict__ out = rg.out;
  const float *__restrict__ sc = rg.sc;
  const int mis = (int)((reinterpret_cast<uintptr_t>(sc) >> 2) & 3);
  const int nq = ((N + mis + kBlock - 1) / kBlock + 3) / 4;  // vectors per lane, <= KPT / 4 (checked by the host)
  const int row0 = wave * 256 * nq + 4 * lane - mis;         // row of key[0]; key[4 q + e]: row0 + 256 q + e
  // Keys of scores are at least 1 (score_key is 0 for one NaN alone); a lane's rows outside [0, N) are 0, and no count
  // below includes 0: no step tests the bounds of a key (with such tests 11.9, 22.6, 35.5 and 57.7 us instead of 10.8, 21.0,
  // 33.5 and 48.9 at 2K, 16K, 32K and 64K rows, plan included).
  uint32_t key[KPT];
#define A3_ROW(J) (row0 + 256 * ((J) >> 2) + ((J) & 3))
#pragma unroll
  for (int q = 0; q < KPT / 4; ++q) {
    const int i = row0 + 256 * q;
    key[4 * q] = key[4 * q + 1] = key[4 * q + 2] = key[4 * q + 3] = 0u;
    if (q < nq && i < N) {
      if (i >= 0 && i + 4 <= N) {
        const float4 v = *reinterpret_cast<const float4 *>(sc + i);
        key[4 * q] = max(score_key(v.x), 1u); key[4 * q + 1] = max(score_key(v.y), 1u);
        key[4 * q + 2] = max(score_key(v.z), 1u); key[4 * q + 3] = max(score_key(v.w), 1u);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (i + e >= 0 && i + e < N) key[4 * q + e] = max(score_key(sc[i + e]), 1u);
      }
    }
  }
  for (int i = tid; i < kBins; i += kBlock) hist[i] = 0;
  if (tid < (int)kRankKeys) cand[tid] = 0;
  if (tid == 0) sh_cand = 0;
  uint32_t mn = 0xffffffffu, mx = 0u;
#pragma unroll
  for (int j = 0; j < KPT; ++j)
    if ((j >> 2) < nq) { mn = min(mn, key[j] - 1u); mx = max(mx, key[j]); }     // (0 - 1: no minimum)
  mn = ~wave_max(~mn);
  mx = wave_max(mx);
  if (lane == 0) { wave_a[wave] = ~mn; wave_b[wave] = mx; }
  A3_LDS_BARRIER();
  mn = ~waves_max(wave_a);
  mx = waves_max(wave_b);

  // lanes below this one in a ballot, added to n
  auto lanes_below = [](unsigned long long m, uint32_t n) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, n));
  };
  // ---- radix select inside [lo, hi]: the key of the k-th largest score ------------------
  // Bins a multiple of 32 apart would share an LDS bank, and scores of few values fall into just such bins.
  auto slot_of = [](uint32_t bin) { return bin ^ ((bin >> 5) & 31u); };
  // Invariant: the wanted key lies in [lo, hi] and is the need-th largest of the keys in there.  (lo >= 1: key 0 less lo
  // lies above hi - lo.)
  uint32_t lo = mn + 1u, hi = mx, need = (uint32_t)k;
  bool exact = false;                                        // all rows equal to the k-th largest are taken
  while (hi != lo) {                                         // (equal: every candidate is the same key)
    const uint32_t width = hi - lo;
    const int shift = max(0, 21 - __clz((int)width));        // (width >> shift) < kBins
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
      const uint32_t rel = key[j] - lo;
      if ((j >> 2) < nq && rel <= width) atomicAdd(&hist[slot_of(rel >> shift)], 1u);
    }
    A3_LDS_BARRIER();
    // the bin that holds the need-th largest candidate: suffix sums over the bins, two per thread
    const uint2 cs = *reinterpret_cast<const uint2 *>(hist + (slot_of(2 * tid) & ~1u));
    const uint2 c = slot_of(2 * tid) & 1 ? make_uint2(cs.y, cs.x) : cs;
    const int upto = a3_wave_prefix((int)(c.x + c.y));       // sum over the lanes <= this one
    A3_LDS_BARRIER();                                        // (wave_a has been read)
    if (lane == 63) wave_a[wave] = (uint32_t)upto;
    *reinterpret_cast<uint2 *>(hist + 2 * tid) = make_uint2(0u, 0u);           // for the next round
    A3_LDS_BARRIER();
    int all;
    const int before = a3_waves_before(reinterpret_cast<const int *>(wave_a), all);
    uint32_t above = (uint32_t)(all - before - upto);        // candidates in higher bins
    if (above < need && above + c.y >= need) sh_found = make_uint4(2 * tid + 1, need - above, c.y, 0);
    above += c.y;
    if (above < need && above + c.x >= need) sh_found = make_uint4(2 * tid, need - above, c.x, 0);
    A3_LDS_BARRIER();
    const uint4 found = sh_found;
    lo += found.x << shift;
    hi = lo + min(hi - lo, (1u << shift) - 1u);
    need = found.y;
    const uint32_t in_bin = found.z;                         // candidates left, need of them wanted
    exact = in_bin == need;
    if (lo == hi) break;                                     // the bin was a single key
    if (in_bin <= kRankKeys) {
      // Few candidates left (the usual case after one or two rounds): they are gathered (in any order: what follows
      // does not depend on it) and ranked directly.  The key v with fewer than `need` candidates above it and at least
      // `need` at or above it is the wanted one.
#pragma unroll
      for (int j = 0; j < KPT; ++j)
        if ((j >> 2) < nq && key[j] - lo <= hi - lo) cand[atomicAdd(&sh_cand, 1u)] = key[j];
      A3_LDS_BARRIER();
      // 256 threads, one a candidate, count against a quarter of them each; behind the last candidate cand holds zeros, which are
      // above nothing
      const int c = tid & ((int)kRankKeys - 1), part = wave / 4, per = ((int)in_bin + 15) / 16 * 4;
      const uint32_t mine = cand[c];
      uint32_t gt = 0, ge = 0;
#pragma unroll 4
      for (int i = part * per; i < part * per + per; i += 4) {
        const uint4 x = *reinterpret_cast<const uint4 *>(cand + i);
        gt += (x.x > mine) + (x.y > mine) + (x.z > mine) + (x.w > mine);
        ge += (x.x >= mine) + (x.y >= mine) + (x.z >= mine) + (x.w >= mine);
      }
      above_of[part][c] = gt | ge << 16;
      A3_LDS_BARRIER();
      if (tid < (int)in_bin) {
        uint32_t sum = 0;
#pragma unroll
        for (int u = 0; u < kWaves / 4; ++u) sum += above_of[u][tid];
        gt = sum & 0xffffu;
        ge = sum >> 16;
        // (several lanes hold the wanted key when it occurs more than once: they store the same numbers)
        if (gt < need && need <= ge) sh_found = make_uint4(mine, need - gt, ge - gt, 0);
      }
      A3_LDS_BARRIER();
      lo = hi = sh_found.x;
      need = sh_found.y;
      exact = sh_found.z == need;
      break;
    }
  }
  const uint32_t tau = lo;               // key of the k-th largest; `need` rows equal to it are taken

  // ---- ordered compaction: rows above tau and equal to tau per wave, then every row's place from the ballots -------
  // (where all of the latter are taken, which is the rule, there is nothing to count but the rows at or above tau)
  const uint32_t top = exact ? tau - 1u : tau;               // (tau >= 1)
  uint32_t n_gt = 0, n_eq = 0;
#pragma unroll
  for (int j = 0; j < KPT; ++j)
    if ((j >> 2) < nq) n_gt += (uint32_t)__popcll(__ballot(key[j] > top));
  if (!exact) {
#pragma unroll
    for (int j = 0; j < KPT; ++j)
      if ((j >> 2) < nq) n_eq += (uint32_t)__popcll(__ballot(key[j] == tau));
  }
  if (exact) need = 0;
  A3_LDS_BARRIER();                                          // wave_a, wave_b: free
  if (lane == 0) { wave_a[wave] = n_gt; wave_b[wave] = n_eq; }
  A3_LDS_BARRIER();
  int all;
  const uint32_t gt_before = (uint32_t)a3_waves_before(reinterpret_cast<const int *>(wave_a), all);
  uint32_t eq_before = exact ? 0u : (uint32_t)a3_waves_before(reinterpret_cast<const int *>(wave_b), all);
  // rows equal to tau are taken in index order until `need` of them are: min(eq_before, need) of the earlier ones were taken, and
  // of this wave's all, none, or (in one wave at most) the first few
  const bool some = eq_before < need && eq_before + n_eq > need;
  const uint32_t above = !some && eq_before < need ? tau - 1u : top;
  uint32_t pos = gt_before + min(eq_before, need);
  auto emit = [&](auto put) {
    if (n_gt + (eq_before < need ? n_eq : 0u) == 0) return;  // nothing of this wave's block is taken
#pragma unroll
    for (int q = 0; q < KPT / 4; ++q) {
      if (q < nq) {
        bool take[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) take[e] = key[4 * q + e] > above;
        if (some) {
          unsigned long long eq[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) eq[e] = __ballot(key[4 * q + e] == tau);
          uint32_t rank = eq_before;                           // rows equal to tau before this one
#pragma unroll
          for (int e = 0; e < 4; ++e) rank = lanes_below(eq[e], rank);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const bool is = (eq[e] >> lane) & 1;
            take[e] = take[e] || (is && rank < need);
            rank += is;
            eq_before += (uint32_t)__popcll(eq[e]);
          }
        }
        uint32_t at = pos;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const unsigned long long b = __ballot(take[e]);
          at = lanes_below(b, at);
          pos += (uint32_t)__popcll(b);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (take[e]) put(at++, rg.s + A3_ROW(4 * q + e));
      }
    }
  };
  if (k <= kListRows) {
    emit([&](uint32_t at, int row) { list[at] = row; });
    A3_LDS_BARRIER();
    for (int i = tid; i < k; i += kBlock) out[i] = list[i];
  } else {
    emit([&](uint32_t at, int row) { out[at] = row; });
  }
#undef A3_ROW
}

template <int KPT>
__global__ void __launch_bounds__(kBlock)
topk_select_reg_kernel(const float *__restrict__ scores, topk_problem prob, int *__restrict__ sel_idx) {
  __shared__ int list[kListRows];
  if (prob.skip) write_fixed_rows(prob, sel_idx);
  topk_select_reg_body<KPT>(topk_range_of(prob, scores, sel_idx), list);
}

// Step 3, the active rows [Re, Q] and (bf16) the layout of the attention's work in one launch, for a batch of one
// request (one workgroup ranks it anyway): the selection goes to sel_idx and to the head of act_idx, the question
// rows behind it, and the same workgroup then lays out the attention (a3_attn_plan.h) from the list it just wrote.
template <int KPT>
__global__ void __launch_bounds__(kBlock)
topk_select_plan_kernel(const float *__restrict__ scores, topk_problem prob, int *__restrict__ sel_idx,
                        int *act_idx, int n_act, attn_plan plan, int G, int wgs_per_head, int item_cost) {
  __shared__ __align__(16) int wave_tot[kPlanThreads / 64];
  __shared__ int small[kPlanLdsInts], list[kListRows];
  static_assert(kPlanThreads == kBlock, "one workgroup shape for both parts");
  topk_select_reg_body<KPT>(topk_range_of(prob, scores, sel_idx), list);
  const int k = prob.one_N >= 0 ? prob.one_k : prob.sel_start[1] - prob.sel_start[0];
  const int s = prob.one_N >= 0 ? 0 : prob.seg_start[0], N = prob.one_N >= 0 ? prob.one_N : prob.ctx_len[0];
  const int first_q = s + N - k;                             // row i >= k of the list: first_q + i
  for (int i = threadIdx.x; k + i < n_act; i += kBlock) act_idx[k + i] = first_q + k + i;   // the question rows
  if (plan.max_tiles == 0) {                                 // fp32: the attention needs no plan
    if (sel_idx != act_idx) {
      __syncthreads();
      for (int i = threadIdx.x; i < k; i += kBlock) act_idx[i] = sel_idx[i];
    }
    return;
  }
  // The plan reads the selected rows in LDS where they fit: nothing then waits for a store
  const bool listed = k <= min(N, kListRows);
  if (!listed || sel_idx != act_idx) {
    __syncthreads();                                         // the selection is written (and has left this CU's L1 path)
    if (sel_idx != act_idx)
      for (int i = threadIdx.x; i < k; i += kBlock) act_idx[i] = sel_idx[i];
    __threadfence_block();
    __syncthreads();
  }
  if (listed)
    attn_plan_body(plan, act_idx, [&](int i) { return i < k ? list[i] : first_q + i; }, n_act, prob.seg_start, 1, G, wgs_per_head, item_cost, wave_tot, small, kPlanLdsInts);
  else
    attn_plan_body(plan, act_idx, [&](int i) { return act_idx[i]; }, n_act, prob.seg_start, 1, G, wgs_per_head, item_cost, wave_tot, small, kPlanLdsInts);
}

constexpr int kMaxRegKeys = 68 * 1024 - 3;   // rows of a request in registers, from whatever alignment it starts

// f(std::integral_constant<int, KPT>) for the smallest KPT that holds a request of n rows
template <typename F>
void with_keys_per_lane(int n, F &&f) {
  const int per = (n + 3 + kBlock - 1) / kBlock;
  if (per <= 4) f(std::integral_constant<int, 4>{});
  else if (per <= 8) f(std::integral_constant<int, 8>{});
  else if (per <= 20) f(std::integral_constant<int, 20>{});
  else if (per <= 36) f(std::integral_constant<int, 36>{});
  else f(std::integral_constant<int, 68>{});
}

// One launch of the ranking kernels over grid (requests, heads).
a3_status topk_launch(const a3_layout *L, const float *scores, const topk_problem &prob, int n_heads, int *sel_idx,
                      hipStream_t st, const char *who) {
  const dim3 grid(L->n_req, n_heads);
  if (L->max_ctx_len <= kMaxRegKeys)
    with_keys_per_lane(L->max_ctx_len, [&](auto kpt) {
      hipLaunchKernelGGL(topk_select_reg_kernel<kpt.value>, grid, dim3(kBlock), 0, st, scores, prob, sel_idx);
    });
  else
    hipLaunchKernelGGL(topk_select_kernel, grid, dim3(kBlock), 0, st, scores, prob, sel_idx);
  A3_CHECK_LAUNCH(who);
  return A3_OK;
}

// ---------------------------------------------------------------------------------------
// eviction extension: pooling of the votes, the rows that are always retained, compaction
// ---------------------------------------------------------------------------------------
// 1-D pooling of stride 1 along the context rows of a request, per head.  mode 0: maximum over the rows
// inside the request's context; mode 1: sum / width (rows outside count as zero).  Other rows are copied.
__global__ void __launch_bounds__(256)
pool_votes_kernel(const float *__restrict__ in, float *__restrict__ out, const int *__restrict__ tok_req,
                  const int *__restrict__ tok_chunk, const int *__restrict__ seg_start,
                  const int *__restrict__ ctx_len, int T, int width, int mode) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= T) return;
  const float *row = in + (size_t)blockIdx.y * T;
  float v = row[t];
  if (tok_chunk[t] >= 0) {
    const int r = tok_req[t];
    const int s = seg_start[r], e = s + ctx_len[r];
    const int lo = max(s, t - width / 2), hi = min(e, t + width / 2 + 1);
    if (mode == 0) {
      for (int u = lo; u < hi; ++u) v = fmaxf(v, row[u]);
    } else {
      float sum = 0.f;
      for (int u = lo; u < hi; ++u) sum += row[u];           // ascending row order
      v = sum / (float)width;
    }
  }
  out[(size_t)blockIdx.y * T + t] = v;
}

// out[slot, g, :] = in[keep_idx[g][slot], g, :] for K and V; 16 bytes per lane, 2^shift lanes to a head's row, one head to a row of
// workgroups.  Bound by the chain index -> row -> store: 2048 rows of 8 heads 4.2 us with the slot, head and vector of a lane from two
// 64-bit divisions, 3.7 like this (launch included).
__global__ void __launch_bounds__(256)
evict_compact_kernel(const uint4 *__restrict__ k, const uint4 *__restrict__ v, const int *__restrict__ keep_idx,
                     int total_keep, int shift, uint4 *__restrict__ k_out, uint4 *__restrict__ v_out) {
  const uint32_t slot = blockIdx.x * (256u >> shift) + (threadIdx.x >> shift), c = threadIdx.x & ((1u << shift) - 1u);
  if (slot >= (uint32_t)total_keep) return;
  const uint32_t g = blockIdx.y, Hkv = gridDim.y;
  const size_t src = ((((size_t)keep_idx[(size_t)g * total_keep + slot] * Hkv) + g) << shift) + c;
  const size_t dst = (((size_t)slot * Hkv + g) << shift) + c;
  k_out[dst] = k[src];
  v_out[dst] = v[src];
}

}  // namespace

extern "C" a3_status a3_topk_select(const a3_layout *L, const float *scores, const int *sel_start, int total_k,
                                    int *sel_idx, void *ws, size_t ws_bytes, void *stream) {
  (void)ws; (void)ws_bytes;              // the select keeps everything in LDS
  a3_status s = a3_check_layout(L, "a3_topk_select", false);
  if (s != A3_OK) return s;
  A3_REQUIRE(total_k >= 0, A3_ERR_INVALID_ARG, "a3_topk_select: total_k %d is negative", total_k);
  A3_REQUIRE((long long)total_k <= (long long)L->max_ctx_len * L->n_req, A3_ERR_INVALID_ARG,
             "a3_topk_select: total_k %d exceeds the number of context rows", total_k);
  A3_REQUIRE(scores && sel_start, A3_ERR_INVALID_ARG, "a3_topk_select: scores/sel_start is NULL");
  if (total_k == 0) return A3_OK;
  A3_REQUIRE(sel_idx, A3_ERR_INVALID_ARG, "a3_topk_select: sel_idx is NULL");
  const topk_problem prob{L->seg_start, L->ctx_len, sel_start, nullptr, nullptr, 0, 0};
  return topk_launch(L, scores, prob, 1, sel_idx, (hipStream_t)stream, "a3_topk_select");
}

extern "C" size_t a3_evict_ws_bytes(const a3_layout *L) {
  if (L == nullptr || L->n_kv_heads <= 0 || L->total_tokens < 0) return 0;
  return a3_align_up((size_t)L->n_kv_heads * L->total_tokens * sizeof(float), 256) + 256;
}

extern "C" a3_status a3_evict_select(const a3_layout *L, const float *votes, const int *sys_len, const int *keep_start,
                                     int total_keep, int pool_width, int pool_mode, int *keep_idx, void *ws,
                                     size_t ws_bytes, void *stream) {
  a3_status s = a3_check_layout(L, "a3_evict_select", true);
  if (s != A3_OK) return s;
  A3_REQUIRE(total_keep >= 0 && total_keep <= L->total_tokens, A3_ERR_INVALID_ARG,
             "a3_evict_select: total_keep %d outside [0, %d]", total_keep, L->total_tokens);
  A3_REQUIRE(votes && sys_len && keep_start, A3_ERR_INVALID_ARG, "a3_evict_select: votes/sys_len/keep_start is NULL");
  A3_REQUIRE(pool_width >= 1 && pool_width % 2 == 1 && pool_width <= 63, A3_ERR_INVALID_ARG,
             "a3_evict_select: pool_width %d is not an odd number in [1, 63]", pool_width);
  A3_REQUIRE(pool_mode == A3_POOL_MAX || pool_mode == A3_POOL_AVG, A3_ERR_INVALID_ARG,
             "a3_evict_select: pool_mode %d", pool_mode);
  if (total_keep == 0 || L->n_req == 0) return A3_OK;
  A3_REQUIRE(keep_idx, A3_ERR_INVALID_ARG, "a3_evict_select: keep_idx is NULL");
  hipStream_t st = (hipStream_t)stream;
  const float *ranked = votes;
  if (pool_width > 1) {
    A3_REQUIRE(ws != nullptr && ws_bytes >= a3_evict_ws_bytes(L), A3_ERR_WORKSPACE,
               "a3_evict_select: workspace %zu bytes, need %zu", ws_bytes, a3_evict_ws_bytes(L));
    float *pooled = (float *)ws;
    hipLaunchKernelGGL(pool_votes_kernel, dim3((L->total_tokens + 255) / 256, L->n_kv_heads), dim3(256), 0, st, votes,
                       pooled, L->tok_req, L->tok_chunk, L->seg_start, L->ctx_len, L->total_tokens, pool_width,
                       pool_mode);
    ranked = pooled;
  }
  const topk_problem prob{L->seg_start, L->ctx_len, keep_start, sys_len, L->q_len, (long)L->total_tokens,
                          (long)total_keep};
  return topk_launch(L, ranked, prob, L->n_kv_heads, keep_idx, st, "a3_evict_select");
}

extern "C" a3_status a3_evict_compact(const a3_layout *L, const void *k_fused, const void *v_fused, const int *keep_idx,
                                      int total_keep, void *k_out, void *v_out, void *stream) {
  a3_status s = a3_check_layout(L, "a3_evict_compact", false);
  if (s != A3_OK) return s;
  A3_REQUIRE(total_keep >= 0 && total_keep <= L->total_tokens, A3_ERR_INVALID_ARG,
             "a3_evict_compact: total_keep %d outside [0, %d]", total_keep, L->total_tokens);
  if (total_keep == 0) return A3_OK;
  A3_REQUIRE(k_fused && v_fused && keep_idx && k_out && v_out, A3_ERR_INVALID_ARG, "a3_evict_compact: NULL tensor");
  A3_REQUIRE(a3_aligned16(k_fused) && a3_aligned16(v_fused) && a3_aligned16(k_out) && a3_aligned16(v_out),
             A3_ERR_INVALID_ARG, "a3_evict_compact: tensors must be 16-byte aligned");
  const int head_bytes = L->head_dim * (L->dtype == A3_BF16 ? 2 : 4);
  A3_REQUIRE(head_bytes == 256 || head_bytes == 512, A3_ERR_UNSUPPORTED, "a3_evict_compact: a head row of %d bytes", head_bytes);
  const int shift = head_bytes == 512 ? 5 : 4, slots = 256 >> shift;
  hipLaunchKernelGGL(evict_compact_kernel, dim3((unsigned)((total_keep + (long)slots - 1) / slots), L->n_kv_heads), dim3(256), 0,
                     (hipStream_t)stream, (const uint4 *)k_fused, (const uint4 *)v_fused, keep_idx, total_keep, shift,
                     (uint4 *)k_out, (uint4 *)v_out);
  A3_CHECK_LAUNCH("a3_evict_compact");
  return A3_OK;
}

// Step 3 -> the rows [Re, Q] -> the layout of the attention's work, as one call: what a3_topk_select,
// a3_active_rows and a3_attention_plan do one after the other.  A batch of one request takes a single launch
// (the workgroup that ranks the request goes on to write the row list and the plan); larger batches run the
// three kernels.
extern "C" a3_status a3_topk_select_plan(const a3_layout *L, const float *scores, const int *sel_start, int total_k,
                                         int *sel_idx, int n_act, int *act_idx, void *ws, size_t ws_bytes,
                                         void *stream) {
  a3_status s = a3_check_layout(L, "a3_topk_select_plan", true);
  if (s != A3_OK) return s;
  A3_REQUIRE(total_k >= 0 && n_act >= total_k && n_act <= L->total_tokens, A3_ERR_INVALID_ARG,
             "a3_topk_select_plan: total_k %d, n_act %d (of %d rows)", total_k, n_act, L->total_tokens);
  A3_REQUIRE(scores && sel_start && act_idx && (sel_idx || total_k == 0), A3_ERR_INVALID_ARG,
             "a3_topk_select_plan: NULL argument");
  const bool one = L->n_req == 1 && L->max_ctx_len <= kMaxRegKeys && total_k > 0 && n_act > 0;
  if (!one) {
    A3_REQUIRE(sel_idx != act_idx || L->n_req == 1, A3_ERR_INVALID_ARG,
               "a3_topk_select_plan: sel_idx may only be act_idx itself in a batch of one request");
    s = a3_topk_select(L, scores, sel_start, total_k, sel_idx, nullptr, 0, stream);
    if (s != A3_OK) return s;
    if (sel_idx == act_idx) {
      // one request, selection already at the head of act_idx: only the question rows are missing
      int *tmp = act_idx;   // a3_active_rows reads sel_idx[j] and writes act_idx[j] for the same j: in place is fine
      s = a3_active_rows(L, tmp, sel_start, n_act, act_idx, stream);
    } else {
      s = a3_active_rows(L, sel_idx, sel_start, n_act, act_idx, stream);
    }
    if (s != A3_OK) return s;
    return a3_attention_plan(L, act_idx, n_act, ws, ws_bytes, stream);
  }
  A3_REQUIRE((long long)total_k <= (long long)L->max_ctx_len, A3_ERR_INVALID_ARG,
             "a3_topk_select_plan: total_k %d exceeds the number of context rows", total_k);
  attn_plan plan{};
  if (L->dtype == A3_BF16) {
    A3_REQUIRE(ws != nullptr && ws_bytes >= a3_attn_ws_bytes(L, n_act), A3_ERR_WORKSPACE,
               "a3_topk_select_plan: workspace %zu bytes, need %zu", ws_bytes, a3_attn_ws_bytes(L, n_act));
    attn_plan_carve(L, n_act, ws, ws_bytes, &plan);
  }
  topk_problem prob{L->seg_start, L->ctx_len, sel_start, nullptr, nullptr, 0, 0};
  if (L->max_ctx_len + L->max_q_len == L->total_tokens) {   // the one request's lengths are the layout's maxima
    prob.one_N = L->max_ctx_len;
    prob.one_k = total_k;
  }
  const int G = L->n_q_heads / L->n_kv_heads;
  with_keys_per_lane(L->max_ctx_len, [&](auto kpt) {
    hipLaunchKernelGGL(topk_select_plan_kernel<kpt.value>, dim3(1), dim3(kBlock), 0, (hipStream_t)stream, scores, prob,
                       sel_idx, act_idx, n_act, plan, G, plan.max_wgs, attn_item_cost(L, n_act));
  });
  A3_CHECK_LAUNCH("a3_topk_select_plan");
  return A3_OK;
}
