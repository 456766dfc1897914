// Step 4 (attention part) of the A^3 fusion path: Eq. 4 and the last line of Eq. 5.
//
//   O[i, hq] = softmax( q[i, hq] . K'[u, hq/G] * scale ) V[u, hq/G]   over rows u <= act_idx[i] of the request
//
// The query rows are a sparse, ascending subset of the prompt (the selected tokens and the
// question), each with its own causal length.  bf16 path:
//   plan kernel   one workgroup: counts active rows per request and writes tile descriptors
//                 (request, first row, number of visible keys of the tile's last row)
//   main kernel   flash attention on the matrix cores.  The G query heads that share a KV head
//                 are packed with the active rows into one row space m = row*G + head, so a K/V
//                 tile is loaded once per group.  Everything is computed transposed:
//                     S^T[key][m] = K Q^T          (A = K fragment from LDS, B = Q fragment in registers)
//                     O^T[d][m]  += V^T P^T        (A = V^T fragment from LDS, B = P^T from the S^T accumulators)
//                 In this orientation four lanes share ONE query row m, and two blocks of S^T accumulators are
//                 exactly one B operand of the second product.
// What bounds the main kernel: power.  16x16x32 matrix instructions, two waves per SIMD in opposite phases: 3230 cycles
// per 64-key tile and 256 rows against 3580 with one wave's phases overlapping by chance on 32x32x16, at 1.9 GHz;
// 16K context at r = 10 %: 290 -> 255 us, 64K: 3411 -> 3030 us (1.18 PFLOP/s), seven heads per KV head at 32K: 1597 ->
// 1400 us.  Leaving out the exponentials, the loads or the fragment reads gives 9, 8 and 4 %.
// fp32 path: the fp32 matrix instruction, one workgroup per 16 packed rows.
#include <stdlib.h>
#include <string.h>

#include <type_traits>

#include "a3_internal.h"
#include "a3_attn_plan.h"

namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kD = 128;
constexpr int kAttnWaves = kTM / 32;   // waves per workgroup, two groups of four in opposite phases
constexpr int kAttnThreads = 64 * kAttnWaves;
constexpr int kTileBytes = kTK * kD * 2;             // a K or V tile [key][d] in LDS, unpadded 256-byte rows
constexpr int kStages = 4;                           // of the K ring and of the V ring
constexpr int kAhead = 4;                            // fragments read ahead of their products
constexpr int kTableItems = 16;
constexpr size_t kRingBytes = (size_t)2 * kStages * kTileBytes;
constexpr size_t kAttnLds = kRingBytes + (size_t)kAttnWaves * kTableItems * 32;   // 132 KB

__global__ void __launch_bounds__(kPlanThreads)
attn_plan_kernel(attn_plan p, const int *__restrict__ act_idx, int n_act, const int *__restrict__ seg_start,
                 int n_req, int G, int wgs_per_head, int item_cost) {
  __shared__ int wave_tot[kPlanThreads / 64];
  __shared__ int small[kPlanLdsInts];
  attn_plan_body(p, act_idx, n_act, seg_start, n_req, G, wgs_per_head, item_cost, wave_tot, small, kPlanLdsInts);
}

struct attn_args {
  const void *q, *k, *v;
  void *out;
  const int *act_idx;
  const int *seg_start;
  const int *tok_req;
  attn_plan plan;
  int n_act, Hq, Hkv, d;
  float scale2;
};

// v_exp_f32: 2^x, about 1 ulp, -inf -> 0, results below the normal range flush to 0
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
// Maximum over the four 16-lane groups of a wave (lanes l, l + 16, l + 32, l + 48), by lane-row swaps
__device__ __forceinline__ float groups_max(float x) {
  uint32_t u = __float_as_uint(x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  u = __float_as_uint(x);
  r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }

struct attn_item { int k_begin, k_end, kv_len, m0, m_end, a0, base, nseg; };

// One workgroup per share of a KV head's work: it runs the items of its share in order, their 64-key tiles as one stream.
__global__ void __launch_bounds__(kAttnThreads, 1)
attn_bf16_kernel(attn_args a) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int g = blockIdx.x % a.Hkv, wg = blockIdx.x / a.Hkv;
  // a plan made with another number of workgroups per head lies elsewhere in the workspace: touch nothing
  if (a.plan.counters[3] != a.plan.max_wgs || wg >= a.plan.counters[2]) return;
  const int item_begin = a.plan.wg_start[wg], item_end = a.plan.wg_start[wg + 1];
  if (item_begin >= item_end) return;
  const int G = a.Hq / a.Hkv;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, lg = lane >> 4, grp = wave >> 2;
  const bf16_t *__restrict__ Q = (const bf16_t *)a.q;
  const float c2 = a.scale2;

  // ---- items of this workgroup: the first kTableItems are looked up once, into a table of the wave's own -----------------
  auto fetch = [&](int i) {
    const int4 it = a.plan.items[i];
    const int4 ta = a.plan.tile_a[it.x];
    attn_item d;
    d.nseg = a.plan.tile_b[it.x].y;
    d.k_begin = it.y; d.k_end = it.z; d.kv_len = ta.z; d.m0 = ta.y; d.m_end = ta.w;
    d.a0 = a.plan.a_lo[ta.x]; d.base = a.seg_start[ta.x];
    return d;
  };
  attn_item *table = reinterpret_cast<attn_item *>(lds + kRingBytes + wave * (kTableItems * sizeof(attn_item)));
  if (lane < kTableItems && item_begin + lane < item_end) table[lane] = fetch(item_begin + lane);
  auto item_at = [&](int i) {
    attn_item d = i - item_begin < kTableItems ? table[i - item_begin] : fetch(i);
    int *f = reinterpret_cast<int *>(&d);
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = __builtin_amdgcn_readfirstlane(f[e]);
    return d;
  };

  // ---- loads: both tiles of 64 keys x 256 bytes by direct-to-LDS loads, 4 keys per wave instruction, two instructions
  // per wave and tile.  K: slot s (16 bytes) of key r holds piece s ^ (r % 16), so that the 16 keys a quarter wave reads at
  // one piece index touch all 64 banks once.  V: the 32-byte piece p of key r lies at p ^ (r % 8), so that the 8 keys x 32
  // bytes a half wave hands to the transposing read do.
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds;
  const uint32_t pitch = (uint32_t)a.Hkv * kD * sizeof(bf16_t);
  const int drow = 4 * wave + lg;                            // key of the lane in instruction 0; + 32 in instruction 1
  const uint32_t key_off = (uint32_t)drow * pitch;
  const uint32_t kpiece = 16 * (l16 ^ (drow & 15)), vpiece = 32 * ((l16 >> 1) ^ (drow & 7)) + 16 * (l16 & 1);
  const uint32_t koff0 = key_off + kpiece, koff1 = koff0 + 32 * pitch, voff0 = key_off + vpiece, voff1 = voff0 + 32 * pitch;
  // K of a tile is requested one tile before its V: l_* the tile whose K comes next, v_* the one before it
  int l_item = item_begin, l_keys, l_steps, v_keys = kTK;    // visible keys and tiles of the item from this tile on
  const char *l_kb, *l_vb, *v_vb = nullptr;
  auto load_from = [&](int i) {
    const attn_item d = item_at(i);
    l_keys = d.kv_len - d.k_begin;
    l_steps = (d.k_end - d.k_begin + kTK - 1) / kTK;
    const size_t at = ((size_t)(d.base + d.k_begin) * a.Hkv + g) * kD;
    l_kb = reinterpret_cast<const char *>((const bf16_t *)a.k + at);
    l_vb = reinterpret_cast<const char *>((const bf16_t *)a.v + at);
  };
  // Inline assembly on purpose: the compiler then neither treats these as LDS writes (it would wait for all of them before
  // every LDS read) nor moves memory accesses across them; the waits for them are the explicit s_waitcnt below.
  auto dma = [&](const char *base, uint32_t off, uint32_t to) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(lds_base + to), "v"(off), "s"(base) : "memory");
  };
  // keys past the item's last visible one are clamped onto it and masked later; past the last tile of the stream that one
  // again, unused
  auto load_half = [&](const char *base, int keys, uint32_t off0, uint32_t off1, uint32_t piece, uint32_t to) {
    if (keys < kTK) {
      const uint32_t last = (uint32_t)(keys - 1) * pitch;
      off0 = min(key_off, last) + piece;
      off1 = min(key_off + 32 * pitch, last) + piece;
    }
    dma(base, off0, to);
    dma(base, off1, to + 8192);
  };
  auto load_k = [&](int stage) { load_half(l_kb, l_keys, koff0, koff1, kpiece, stage * kTileBytes + wave * 1024); };
  auto load_v = [&](int stage) { load_half(v_vb, v_keys, voff0, voff1, vpiece, (kStages + stage) * kTileBytes + wave * 1024); };
  auto load_next = [&]() {
    v_vb = l_vb; v_keys = l_keys;
    if (--l_steps > 0) {
      l_kb += kTK * pitch; l_vb += kTK * pitch; l_keys -= kTK;
    } else if (l_item + 1 < item_end) {
      load_from(++l_item);
    } else {
      l_steps = 1;
    }
  };

  // ---- rows of an item: lane (l16, lg) holds rows m0 + 32 wave + 16 rb + l16 ---------------------------------------
  bf16x8 qf[2][4];
  int limit[2], min_limit, max_limit;                        // last visible key of the rows (request-relative)
  uint32_t out_row[2], prev_row[2];                          // row of the output, ~0: none
  attn_item cur;
  auto load_rows = [&]() {
    min_limit = 0x7fffffff; max_limit = -1;
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
      const int m = cur.m0 + 32 * wave + 16 * rb + l16, mc = min(m, cur.m_end - 1);
      const int ar = mc / G, arow = cur.a0 + ar, hq = g * G + mc - ar * G;
      out_row[rb] = (uint32_t)arow * a.Hq + hq;
      const bf16_t *qp = Q + (size_t)out_row[rb] * kD + lg * 8;
#pragma unroll
      for (int ds = 0; ds < 4; ++ds) qf[rb][ds] = *reinterpret_cast<const bf16x8 *>(qp + 32 * ds);
      limit[rb] = a.act_idx[arow] - cur.base;
      if (m >= cur.m_end) out_row[rb] = ~0u;
    }
    int lo = min(limit[0], limit[1]), hi = max(limit[0], limit[1]);
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) {
      lo = min(lo, __shfl_xor(lo, off, 64));
      hi = max(hi, __shfl_xor(hi, off, 64));
    }
    min_limit = __builtin_amdgcn_readfirstlane(lo);
    max_limit = __builtin_amdgcn_readfirstlane(hi);
  };

  f32x4 o[8][2], st[4][2];
  uint32_t pu[2][2][4];                                      // P of the tile before, pairs of bf16, [32 keys][row block]
  float ref[2], mx[2], nref[2] = {0.f, 0.f};                  // exponent reference and tile maximum in raw logit units; -ref c2
  // Row sums of P, by the matrix pipe (an all-ones V): every register.  They are fp32 sums of the weights as the product with V
  // uses them, rounded to bf16: an output is then an exact mean of the values it sees, and the weights' roundings cancel where
  // values are alike.  Relative error against float64, unrounded weights summed -> these: 8 matching rows of 100 2.04e-3
  // -> 1.99e-3 at 500 keys, 2.11e-3 -> 2.02e-3 at 2048; plain normal logits 2.20e-3 -> 2.18e-3 and 2.24e-3 -> 2.23e-3; flat logits, one
  // key with all the weight, and 16K keys and more: the same within 1 %.
  f32x4 osum[2];
  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = (bf16_t)1.0f;
  int prev_item = item_begin, prev_nseg = 0;
  auto store_rows = [&]() {
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
      const float total = osum[rb][0];
      if (prev_nseg == 1) {
        const float inv = 1.0f / total;
        if (prev_row[rb] != ~0u) {
          bf16_t *p = (bf16_t *)a.out + (size_t)prev_row[rb] * kD + 4 * lg;
#pragma unroll
          for (int db = 0; db < 8; ++db) {
            bf16x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = a3_f2bf(o[db][rb][e] * inv);
            *reinterpret_cast<bf16x4 *>(p + 16 * db) = v;
          }
        }
      } else {
        const size_t pr = ((size_t)g * a.plan.max_items + prev_item) * kTM + 32 * wave + 16 * rb + l16;
        float *p = a.plan.part_o + pr * kD + 4 * lg;
#pragma unroll
        for (int db = 0; db < 8; ++db) *reinterpret_cast<f32x4 *>(p + 16 * db) = o[db][rb];
        if (lg == 0) a.plan.part_ml[pr] = make_float2(ref[rb] * c2, total);
      }
    }
  };

  // ---- fragments: K (16 keys x 32 dims, lane = key l16, piece 4 ds + lg) by one 16-byte read, V^T (16 dims x 32 keys) by two
  // transposing 8-byte reads: lane (l16, lg) then holds dim l16, keys 4 lg .. + 3 of two 16-key blocks, which is the order in
  // which the S^T accumulators hold P (accumulator r of key block b: key 16 b + 4 lg + r, row l16)
  const uint32_t kaddr = l16 * 256 + 16 * (lg ^ l16);
  const int vkey = 4 * lg + (l16 >> 2);
  const uint32_t vaddr = vkey * 256 + 32 * (vkey & 7) + 8 * (l16 & 3);
#define A3_KFRAG(N) fr[(N) % kAhead] = *reinterpret_cast<const bf16x8 *>(kt + (kaddr ^ (64 * ((N) >> 2))) + 4096 * ((N) & 3));
#define A3_VFRAG(N)                                                                                                    \
  {                                                                                                                    \
    typedef __attribute__((address_space(3))) s16x4 *tr_ptr;                                                           \
    const unsigned char *p_ = vt + (vaddr ^ (32 * ((N) & 7))) + 8192 * ((N) >> 3);                                     \
    const s16x4 x_ = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)(p_));                                            \
    const s16x4 y_ = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)(p_ + 4096));                                     \
    fr[(16 + (N)) % kAhead] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(x_, y_, 0, 1, 2, 3, 4, 5, 6, 7));            \
  }
#define A3_FENCE __builtin_amdgcn_sched_barrier(0);
  bf16x8 fr[kAhead];                                         // fragments in the order K 0 .. 15, V 0 .. 15

  cur = item_at(item_begin);
  load_rows();
  prev_row[0] = prev_row[1] = ~0u;
  load_from(item_begin);
  __builtin_amdgcn_s_waitcnt(0);
  load_k(0); load_next();
  load_k(1); load_v(0); load_next();
  load_k(2); load_v(1); load_next();
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(4));                              // this wave's part of K of tiles 0 and 1 has landed
  __builtin_amdgcn_s_barrier();                                          // ... and everybody's
  if (grp == 1) __builtin_amdgcn_s_barrier();                            // one phase behind

  // The two waves of a SIMD belong to different groups and run in opposite phases, one barrier apart: while one has the
  // matrix pipe (S of tile u and P V of tile u - 1), the other does the softmax of its tile on the vector unit.  Group 0
  // multiplies tile u in phase 2 u, group 1 in phase 2 u + 1.  K of tile u + 3 and V of tile u + 2 are requested in the
  // vector phase of tile u; at the end of phase 2 u everything up to K of tile u + 1 and V of tile u has landed, one phase
  // before their first fragments are read.  Beside the matrix pipe a vector instruction takes about 7 cycles of its wave (10.8
  // an exponential), so the vector phase is kept to the 32 scalings, 32 exponentials and 16 conversions: the row sums are
  // matrix products, and the maxima are taken between the products of P V.
  int ring = 0, k0 = cur.k_begin, item = item_begin;         // ring: tile u % 4
  bool first = true, has_prev = false;
  bool act = k0 <= max_limit, act_prev = false;              // a wave whose rows all end before a tile leaves its products out
  {
    const unsigned char *kt = lds;
#pragma unroll
    for (int n = 0; n < kAhead; ++n) A3_KFRAG(n)
  }
#define A3_PV(N)                                                                                                       \
  {                                                                                                                    \
    if ((N) == 14) {                                                                                                   \
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(4));                                                                        \
      __builtin_amdgcn_s_barrier();                                                                                    \
      A3_FENCE                                                                                                         \
    }                                                                                                                  \
    _Pragma("unroll") for (int rb = 0; rb < 2; ++rb)                                                                   \
      o[(N) & 7][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr[(16 + (N)) % kAhead], A3_P((N) >> 3, rb), o[(N) & 7][rb], 0, 0, 0); \
    if (((N) & 7) == 4) {                                                                                              \
      _Pragma("unroll") for (int rb = 0; rb < 2; ++rb)                                                                 \
        osum[rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, A3_P((N) >> 3, rb), osum[rb], 0, 0, 0);                 \
    }                                                                                                                  \
    A3_FENCE                                                                                                           \
    if ((N) + kAhead < 16) A3_VFRAG((N) + kAhead)                                                                      \
    A3_MAX2((N) >> 1, (N) & 1)                                                                                         \
    A3_FENCE                                                                                                           \
  }
  // the N-th pair of S values of a row block, N = 0 .. 7 (key block N / 2, registers 2 (N % 2) and + 1)
  // (the empty asm statements keep the compiler from moving the arithmetic behind the products)
#define A3_EXP2(Q)                                                                                                     \
  {                                                                                                                    \
    const int b_ = (Q) >> 2, r_ = (Q) & 2, rb_ = (Q) & 1;                                                              \
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));                                                         \
    bf16x2 t_;                                                                                                         \
    t_[0] = a3_f2bf(fast_exp2(fmaf(st[b_][rb_][r_], c2, nref[rb_])));                                                  \
    t_[1] = a3_f2bf(fast_exp2(fmaf(st[b_][rb_][r_ + 1], c2, nref[rb_])));                                              \
    pu[b_ >> 1][rb_][2 * (b_ & 1) + r_ / 2] = __builtin_bit_cast(uint32_t, t_);                                        \
    asm volatile("" : "+v"(pu[b_ >> 1][rb_][2 * (b_ & 1) + r_ / 2]));                                                  \
  }
#define A3_P(KS, RB) __builtin_bit_cast(bf16x8, u32x4{pu[KS][RB][0], pu[KS][RB][1], pu[KS][RB][2], pu[KS][RB][3]})
#define A3_MAX2(N, RB) { mx[RB] = fmaxf(fmaxf(mx[RB], st[(N) >> 1][RB][2 * ((N) & 1)]), st[(N) >> 1][RB][2 * ((N) & 1) + 1]); asm volatile("" : "+v"(mx[RB])); }
  for (;;) {
    // ---- matrix phase
    const unsigned char *kt = lds + ring * kTileBytes, *vt = lds + (kStages + ((ring + 3) & 3)) * kTileBytes;
    A3_FENCE
    __builtin_amdgcn_s_setprio(1);
    if (act) {
#pragma unroll
      for (int n = 0; n < 16; ++n) {
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
          st[n & 3][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr[n % kAhead], qf[rb][n >> 2],
                                                                  n < 4 ? f32x4{0.f, 0.f, 0.f, 0.f} : st[n & 3][rb], 0, 0, 0);
        A3_FENCE
        if (n + kAhead < 16) A3_KFRAG(n + kAhead) else A3_VFRAG(n + kAhead - 16)
        A3_FENCE
      }
      if (k0 + kTK - 1 > min_limit) {                        // tile touches the causal boundary of some row
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
          for (int rb = 0; rb < 2; ++rb)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (k0 + 16 * b + 4 * lg + r > limit[rb]) st[b][rb][r] = -INFINITY;
      }
    } else {
#pragma unroll
      for (int n = 0; n < kAhead; ++n) A3_VFRAG(n)
    }
    mx[0] = mx[1] = -INFINITY;                               // (of no meaning, and not used, when the tile is left out)
    A3_FENCE
    if (act_prev) {
#pragma unroll
      for (int n = 0; n < 16; ++n) A3_PV(n)
    } else {
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(4));
      __builtin_amdgcn_s_barrier();
#pragma unroll
      for (int n = 0; n < 16; ++n) A3_MAX2(n >> 1, n & 1)
    }
    __builtin_amdgcn_s_setprio(0);
    A3_FENCE
    // ---- vector phase
    if (first) {
      if (has_prev) store_rows();
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) {
#pragma unroll
        for (int db = 0; db < 8; ++db) o[db][rb] = f32x4{0.f, 0.f, 0.f, 0.f};
        osum[rb] = f32x4{0.f, 0.f, 0.f, 0.f};
        ref[rb] = -INFINITY;
        nref[rb] = 0.f;
      }
      first = false;
    }
    load_k((ring + 3) & 3);
    load_v((ring + 2) & 3);
    load_next();
    if (act) {
      // Lazy rescaling: the exponent reference only has to stay within 2^8 of the running maximum, not equal to it, so the
      // accumulators are rescaled a handful of times per row instead of whenever the maximum moves.  P ranges up to 256.
      const bool redo = __any((mx[0] - ref[0]) * c2 > 8.0f || (mx[1] - ref[1]) * c2 > 8.0f);   // also the first visible key (-inf)
      if (redo) {
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) {
          const float new_ref = fmaxf(ref[rb], groups_max(mx[rb]));
          const float alpha = new_ref == -INFINITY ? 1.0f : fast_exp2((ref[rb] - new_ref) * c2);
          ref[rb] = new_ref;
          nref[rb] = new_ref == -INFINITY ? 0.f : -new_ref * c2;                  // no visible key yet: every P is 0
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            osum[rb][r] *= alpha;
#pragma unroll
            for (int db = 0; db < 8; ++db) o[db][rb][r] *= alpha;
          }
        }
      }
#pragma unroll
      for (int q = 0; q < 16; ++q) A3_EXP2(q)
    }
    // ---- on to the next tile
    ring = (ring + 1) & 3;
    act_prev = act;
    bool last = false;
    k0 += kTK;
    if (k0 >= cur.k_end) {
      prev_item = item; prev_nseg = cur.nseg;
      prev_row[0] = out_row[0]; prev_row[1] = out_row[1];
      has_prev = true;
      if (++item < item_end) {
        cur = item_at(item);
        load_rows();
        __builtin_amdgcn_s_waitcnt(0);
        k0 = cur.k_begin;
        first = true;
      } else {
        last = true;
      }
    }
    act = k0 <= max_limit;
    if (grp == 1) __builtin_amdgcn_s_waitcnt(vmcnt_imm(4));
    {
      const unsigned char *kt = lds + ring * kTileBytes;
      A3_FENCE
#pragma unroll
      for (int n = 0; n < kAhead; ++n) A3_KFRAG(n)
      A3_FENCE
    }
    __builtin_amdgcn_s_barrier();
    if (last) break;
  }
  // ---- P V of the last tile
  if (act_prev) {
    const unsigned char *vt = lds + (kStages + ((ring + 3) & 3)) * kTileBytes;
#pragma unroll
    for (int n = 0; n < 16; ++n) {
      A3_VFRAG(n)
#pragma unroll
      for (int rb = 0; rb < 2; ++rb)
        o[n & 7][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr[(16 + n) % kAhead], A3_P(n >> 3, rb), o[n & 7][rb], 0, 0, 0);
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) osum[rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, A3_P(ks, rb), osum[rb], 0, 0, 0);
  }
#undef A3_PV
#undef A3_P
#undef A3_EXP2
#undef A3_MAX2
#undef A3_KFRAG
#undef A3_VFRAG
#undef A3_FENCE
  if (grp == 0) __builtin_amdgcn_s_barrier();
  store_rows();
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));                  // the tail loads have landed before LDS is released
}

// Merges the partial results of tiles that were cut into key segments, in segment order.
// One workgroup per (tile, KV head, 32 of the tile's rows); 8 lanes share a row, dims 32 i + 4 lane .. + 3 each, so that
// one load of theirs covers 128 bytes in one piece (16 dims in a run per lane: 12.4 instead of 11.6 us at 16K, 17.4 instead
// of 15.8 at 64K).
__global__ void __launch_bounds__(256)
attn_combine_kernel(attn_args a) {
  const int t = blockIdx.x, g = blockIdx.y;
  if (a.plan.counters[3] != a.plan.max_wgs || t >= a.plan.counters[0]) return;
  const int2 tb = a.plan.tile_b[t];
  const int nseg = tb.y;
  if (nseg <= 1) return;
  const int4 ta = a.plan.tile_a[t];
  const int G = a.Hq / a.Hkv;
  const int ml = blockIdx.z * 32 + (threadIdx.x >> 3), d0 = (threadIdx.x & 7) * 4;
  const int m = ta.y + ml;
  if (m >= ta.w) return;
  const int arow = a.plan.a_lo[ta.x] + m / G, hq = g * G + m % G;
  const size_t p0 = (size_t)g * a.plan.max_items + tb.x;
  const float2 *ml_p = a.plan.part_ml + p0 * kTM + ml;
  const float *o_p = a.plan.part_o + (p0 * kTM + ml) * kD + d0;
  float acc[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
  float M = -INFINITY, L = 0.f;
  // two segments at a time, their loads in flight together (past the last one: that one again, with weight 0)
  for (int s0 = 0; s0 < nseg; s0 += 2) {
    float2 st[2];
    f32x4 v[2][4];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const size_t s = (size_t)min(s0 + u, nseg - 1) * kTM;
      st[u] = ml_p[s];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[u][i] = *reinterpret_cast<const f32x4 *>(o_p + s * kD + 32 * i);
    }
    float m = M;
#pragma unroll
    for (int u = 0; u < 2; ++u) m = fmaxf(m, st[u].x);
    const float old = M == -INFINITY ? 0.f : exp2f(M - m);
    L *= old;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] *= old;
    M = m;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const float wgt = s0 + u < nseg && st[u].x != -INFINITY ? exp2f(st[u].x - M) : 0.f;   // 0: the row sees nothing of it
      L += st[u].y * wgt;
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[i] = fmaf(v[u][i / 4][i % 4], wgt, acc[i]);
    }
  }
  const float inv = 1.0f / L;
  bf16_t *orow = (bf16_t *)a.out + ((size_t)arow * a.Hq + hq) * kD + d0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    bf16x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = a3_f2bf(acc[4 * i + e] * inv);
    *reinterpret_cast<bf16x4 *>(orow + 32 * i) = v;
  }
}

// ---------------------------------------------------------------------------------------
// fp32: one workgroup per 16 packed (row, head) pairs of a KV head; its eight waves take every eighth block of 16 keys
// and merge at the end
// ---------------------------------------------------------------------------------------
// fp32 matrix instruction (16x16x4), fragments straight from memory.  S^T[key][m]: register r of lane (l16, lg) is key
// 4 lg + r, pair l16 - which is the B operand of the r-th product of O^T[d][m] += V^T P^T when lane group lg supplies key
// 4 lg + r of V; its lane l16 loads coordinates 4 l16 .. + 3 at once, so block e of O holds coordinates 4 (row) + e.
// (One workgroup per row and head with a thread per key took 50 us for 108 rows x 8 heads x up to 544 keys.)
constexpr int kF32Waves = 8;
constexpr size_t kF32Lds(int d) { return (size_t)kF32Waves * 16 * (d * sizeof(float) + sizeof(float2)); }
template <int D>
__global__ void __launch_bounds__(64 * kF32Waves)
attn_f32_kernel(attn_args a) {
  extern __shared__ __align__(16) float lds_f[];               // [wave][D / 4 rows of 16 pairs] O as float4, then (ref, sum)
  f32x4 *lds_o = reinterpret_cast<f32x4 *>(lds_f);
  float2 *lds_ml = reinterpret_cast<float2 *>(lds_f + (size_t)kF32Waves * 16 * D);
  const int G = a.Hq / a.Hkv, g = blockIdx.y, rows = 16 / G;   // active rows of a workgroup
  const int a0 = blockIdx.x * rows, a_end = min(a0 + rows, a.n_act);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, lg = lane >> 4;
  const float *__restrict__ Q = (const float *)a.q;
  const float *__restrict__ K = (const float *)a.k;
  const float *__restrict__ V = (const float *)a.v;
  const int arow = min(a0 + l16 / G, a_end - 1), hq = g * G + l16 % G;
  f32x4 qf[D / 16];
  {
    const f32x4 *qp = reinterpret_cast<const f32x4 *>(Q + ((size_t)arow * a.Hq + hq) * D) + lg;
#pragma unroll
    for (int c = 0; c < D / 16; ++c) qf[c] = qp[4 * c];
  }
  const int t = a.act_idx[arow], req = a.tok_req[t];
  // the rows of one request at a time (rows are ascending: nearly always all of them)
  for (int b0 = a0; b0 < a_end;) {
    const int r = a.tok_req[a.act_idx[b0]], base = a.seg_start[r];
    int b1 = b0;
    while (b1 < a_end && a.tok_req[a.act_idx[b1]] == r) ++b1;
    const bool mine = req == r && l16 < (a_end - a0) * G;
    const int limit = mine ? t - base : -1;                    // last visible key (request-relative)
    const int n_keys = a.act_idx[b1 - 1] - base + 1;
    // The product O^T += V^T P^T gives every pair every key of a block, with weight 0 where it sees none: no harm unless V is
    // infinite or NaN there.  That shows in O, and the wave starts over with each pair adding the keys it sees one by one.
    f32x4 o[D / 16];
    float ref, sum;
    auto attend = [&](auto one_by_one) {
#pragma unroll
      for (int e = 0; e < D / 16; ++e) o[e] = f32x4{0.f, 0.f, 0.f, 0.f};
      ref = -INFINITY;
      sum = 0.f;
      f32x4 kf[D / 16];
      auto load_k = [&](int k0) {
        const f32x4 *kp = reinterpret_cast<const f32x4 *>(K + ((size_t)(base + min(k0 + l16, n_keys - 1)) * a.Hkv + g) * D) + lg;
#pragma unroll
        for (int c = 0; c < D / 16; ++c) kf[c] = kp[4 * c];
      };
      if (16 * wave < n_keys) load_k(16 * wave);
      for (int k0 = 16 * wave; k0 < n_keys; k0 += 16 * kF32Waves) {
        f32x4 vf[4][D / 64];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const f32x4 *vp = reinterpret_cast<const f32x4 *>(V + ((size_t)(base + min(k0 + 4 * lg + e, n_keys - 1)) * a.Hkv + g) * D) + l16;
#pragma unroll
          for (int h = 0; h < D / 64; ++h) vf[e][h] = vp[16 * h];
        }
        f32x4 c4[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) c4[e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < D / 16; ++c)
#pragma unroll
          for (int e = 0; e < 4; ++e) c4[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][e], qf[c][e], c4[e], 0, 0, 0);
        if (k0 + 16 * kF32Waves < n_keys) load_k(k0 + 16 * kF32Waves);
        f32x4 p;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          p[e] = k0 + 4 * lg + e <= limit ? ((c4[0][e] + c4[1][e]) + (c4[2][e] + c4[3][e])) * a.scale2 : -INFINITY;
        float mx = fmaxf(fmaxf(p[0], p[1]), fmaxf(p[2], p[3]));
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float new_ref = fmaxf(ref, mx), use = new_ref == -INFINITY ? 0.f : new_ref;
        const float alpha = exp2f(ref - use);                    // ref = -inf: 0
        ref = new_ref;
        sum *= alpha;
#pragma unroll
        for (int e = 0; e < 4; ++e) { p[e] = exp2f(p[e] - use); sum += p[e]; }
#pragma unroll
        for (int e = 0; e < D / 16; ++e)
#pragma unroll
          for (int x = 0; x < 4; ++x) o[e][x] *= alpha;
        if constexpr (one_by_one) {
#pragma unroll 1
          for (int u = 0; u < 16; ++u) {
            const float pe = (u & 2) ? ((u & 1) ? p[3] : p[2]) : ((u & 1) ? p[1] : p[0]);
            const float pu = __shfl(pe, 16 * (u >> 2) + l16, 64);
            if (k0 + u > limit) continue;
            const float *vp = V + ((size_t)(base + k0 + u) * a.Hkv + g) * D + 16 * lg;
#pragma unroll
            for (int h = 0; h < D / 64; ++h)
#pragma unroll
              for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int y = 0; y < 4; ++y) o[4 * h + x][y] = fmaf(pu, vp[64 * h + 4 * y + x], o[4 * h + x][y]);
          }
          continue;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int h = 0; h < D / 64; ++h)
#pragma unroll
            for (int x = 0; x < 4; ++x) o[4 * h + x] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[e][h][x], p[e], o[4 * h + x], 0, 0, 0);
      }
    };
    attend(std::false_type{});
    float z = 0.f;
#pragma unroll
    for (int e = 0; e < D / 16; ++e)
#pragma unroll
      for (int y = 0; y < 4; ++y) z = fmaf(o[e][y], 0.f, z);
    if (__any(z != 0.f)) attend(std::true_type{});
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
    __syncthreads();                                           // the merge of the request before has been read
    // register r of block 4 h + x: coordinate 64 h + 4 (4 lg + r) + x
#pragma unroll
    for (int h = 0; h < D / 64; ++h)
#pragma unroll
      for (int x = 0; x < 4; ++x)
        lds_o[((size_t)wave * 16 + l16) * (D / 4) + (((h * 4 + lg) * 4 + x) ^ (l16 & 7))] = o[4 * h + x];
    if (lg == 0) lds_ml[wave * 16 + l16] = make_float2(ref, sum);
    __syncthreads();
    // 16 pairs x D / 4 vectors: the waves' results in wave order
    for (int v = tid; v < 16 * (D / 4); v += 64 * kF32Waves) {
      const int m = v / (D / 4), c = v % (D / 4);              // c = (h * 4 + lg) * 4 + x
      const int row = a0 + m / G;
      if (m >= (a_end - a0) * G || row < b0 || row >= b1) continue;
      float M = -INFINITY, Z = 0.f;
#pragma unroll
      for (int w = 0; w < kF32Waves; ++w) M = fmaxf(M, lds_ml[w * 16 + m].x);
      f32x4 s4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < kF32Waves; ++w) {
        const float2 ml = lds_ml[w * 16 + m];
        const float wgt = exp2f(ml.x - M);                     // 0 for a wave that saw nothing
        Z += ml.y * wgt;
        const f32x4 ov = lds_o[((size_t)w * 16 + m) * (D / 4) + (c ^ (m & 7))];
#pragma unroll
        for (int e = 0; e < 4; ++e) s4[e] = fmaf(ov[e], wgt, s4[e]);
      }
      float *op = (float *)a.out + ((size_t)row * a.Hq + g * G + m % G) * D + 64 * (c >> 4) + 16 * ((c >> 2) & 3) + (c & 3);
#pragma unroll
      for (int e = 0; e < 4; ++e) op[4 * e] = s4[e] / Z;
    }
    b0 = b1;
  }
}

}  // namespace

size_t a3_attn_ws_bytes(const a3_layout *L, int max_active_rows) {
  if (L->dtype != A3_BF16) return 256;
  const size_t per_req = a3_align_up((size_t)(L->n_req + 1) * sizeof(int), 256);
  const size_t tiles = attn_max_tiles(L, max_active_rows), items = attn_max_items(L, max_active_rows);
  return 2 * per_req + a3_align_up(tiles * sizeof(int4), 256) + a3_align_up(tiles * sizeof(int2), 256) +
         a3_align_up((tiles + 1) * sizeof(int), 256) + a3_align_up(items * sizeof(int4), 256) +
         a3_align_up((size_t)(attn_wgs_per_head(L) + 1) * sizeof(int), 256) + 256 +
         a3_align_up(items * L->n_kv_heads * kTM * kD * sizeof(float), 256) +
         a3_align_up(items * L->n_kv_heads * kTM * sizeof(float2), 256) + 2048;
}

// parts & 1: lay out the work (plan kernel); parts & 2: attend and merge.  The plan only depends on the list of
// active rows, so a caller may have it made beside whatever else precedes the attention.
static a3_status attn_launch(const a3_layout *L, const void *q_act, const int *act_idx, int n_act,
                             const void *k_fused, const void *v_fused, void *out, void *ws, size_t ws_bytes,
                             void *stream, int parts, hipEvent_t ev_begin = nullptr, hipEvent_t ev_end = nullptr) {
  a3_status s = a3_check_layout(L, "a3_fused_attention", true);
  if (s != A3_OK) return s;
  A3_REQUIRE(n_act >= 0 && n_act <= L->total_tokens, A3_ERR_INVALID_ARG,
             "a3_fused_attention: n_act %d outside [0, %d]", n_act, L->total_tokens);
  if (n_act == 0) return A3_OK;
  A3_REQUIRE(act_idx != nullptr, A3_ERR_INVALID_ARG, "a3_fused_attention: act_idx is NULL");
  if (parts & 2) {
    A3_REQUIRE(q_act && k_fused && v_fused && out, A3_ERR_INVALID_ARG, "a3_fused_attention: NULL argument");
    A3_REQUIRE(a3_aligned16(q_act) && a3_aligned16(k_fused) && a3_aligned16(v_fused) && a3_aligned16(out),
               A3_ERR_INVALID_ARG, "a3_fused_attention: tensors must be 16-byte aligned");
  }
  hipStream_t st = (hipStream_t)stream;
  attn_args a;
  a.q = q_act; a.k = k_fused; a.v = v_fused; a.out = out;
  a.act_idx = act_idx; a.seg_start = L->seg_start; a.tok_req = L->tok_req;
  a.n_act = n_act; a.Hq = L->n_q_heads; a.Hkv = L->n_kv_heads; a.d = L->head_dim;
  a.scale2 = a3_scale_of(L) * kLog2e;
  memset(&a.plan, 0, sizeof(a.plan));
  if (L->dtype == A3_BF16) {
    // (a limit of an earlier kernel's 32-bit byte offsets; this one's bases are 64-bit per tile.  The line stays: what lies
    // beyond it was always refused and has never been run)
    A3_REQUIRE(((long long)L->max_ctx_len + L->max_q_len + 128) * L->n_kv_heads * kD * 2 < (1LL << 32), A3_ERR_UNSUPPORTED,
               "a3_fused_attention: a request of %d rows is too long (its K and V rows must stay below 4 GiB each)",
               L->max_ctx_len + L->max_q_len);
    A3_REQUIRE(ws != nullptr, A3_ERR_WORKSPACE, "a3_fused_attention: workspace is NULL");
    A3_REQUIRE(ws_bytes >= a3_attn_ws_bytes(L, n_act), A3_ERR_WORKSPACE,
               "a3_fused_attention: workspace %zu bytes, need %zu", ws_bytes, a3_attn_ws_bytes(L, n_act));
    static a3_once_per_device lds_once;
    const hipError_t e = a3_once(lds_once, []() {
      return hipFuncSetAttribute((const void *)attn_bf16_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kAttnLds);
    });
    if (e != hipSuccess) return a3_fail(A3_ERR_HIP, "a3_fused_attention: %s", hipGetErrorString(e));
    attn_plan_carve(L, n_act, ws, ws_bytes, &a.plan);
    const int wgs_per_head = a.plan.max_wgs, max_tiles = a.plan.max_tiles, Hkv = L->n_kv_heads;
    if (parts & 1)
      hipLaunchKernelGGL(attn_plan_kernel, dim3(1), dim3(kPlanThreads), 0, st, a.plan, act_idx, n_act, L->seg_start,
                         L->n_req, L->n_q_heads / L->n_kv_heads, wgs_per_head, attn_item_cost());
    if (parts & 2) {
      // blockIdx % Hkv = KV head, so with 8 KV heads each XCD's L2 serves the K/V of one head
      if (ev_begin) (void)hipEventRecord(ev_begin, st);
      hipLaunchKernelGGL(attn_bf16_kernel, dim3((unsigned)wgs_per_head * Hkv), dim3(kAttnThreads), kAttnLds, st, a);
      if (ev_end) (void)hipEventRecord(ev_end, st);
      hipLaunchKernelGGL(attn_combine_kernel, dim3((unsigned)max_tiles, Hkv, kTM / 32), dim3(256), 0, st, a);
    }
  } else if (parts & 2) {
    const int rows = 16 / (L->n_q_heads / L->n_kv_heads);
    const dim3 grid((n_act + rows - 1) / rows, L->n_kv_heads);
    static a3_once_per_device lds_once;
    const hipError_t e = a3_once(lds_once, []() {
      return hipFuncSetAttribute((const void *)attn_f32_kernel<128>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kF32Lds(128));
    });
    if (e != hipSuccess) return a3_fail(A3_ERR_HIP, "a3_fused_attention: %s", hipGetErrorString(e));
    if (L->head_dim == 64) hipLaunchKernelGGL(attn_f32_kernel<64>, grid, dim3(64 * kF32Waves), kF32Lds(64), st, a);
    else hipLaunchKernelGGL(attn_f32_kernel<128>, grid, dim3(64 * kF32Waves), kF32Lds(128), st, a);
  }
  A3_CHECK_LAUNCH("a3_fused_attention");
  return A3_OK;
}

extern "C" a3_status a3_fused_attention(const a3_layout *L, const void *q_act, const int *act_idx, int n_act,
                                        const void *k_fused, const void *v_fused, void *out, void *ws,
                                        size_t ws_bytes, void *stream) {
  return attn_launch(L, q_act, act_idx, n_act, k_fused, v_fused, out, ws, ws_bytes, stream, 3);
}

extern "C" a3_status a3_attention_plan(const a3_layout *L, const int *act_idx, int n_act, void *ws, size_t ws_bytes,
                                       void *stream) {
  return attn_launch(L, nullptr, act_idx, n_act, nullptr, nullptr, nullptr, ws, ws_bytes, stream, 1);
}

extern "C" a3_status a3_fused_attention_planned(const a3_layout *L, const void *q_act, const int *act_idx, int n_act,
                                                const void *k_fused, const void *v_fused, void *out, void *ws,
                                                size_t ws_bytes, void *stream) {
  return attn_launch(L, q_act, act_idx, n_act, k_fused, v_fused, out, ws, ws_bytes, stream, 2);
}

// a3_fused_attention_planned with two HIP events recorded on the stream right before and right after the main
// kernel (the merge of the partial results follows the second one): for measurements of that kernel alone.
extern "C" a3_status a3_fused_attention_planned_events(const a3_layout *L, const void *q_act, const int *act_idx,
                                                       int n_act, const void *k_fused, const void *v_fused, void *out,
                                                       void *ws, size_t ws_bytes, void *stream, void *ev_main_begin,
                                                       void *ev_main_end) {
  return attn_launch(L, q_act, act_idx, n_act, k_fused, v_fused, out, ws, ws_bytes, stream, 2, (hipEvent_t)ev_main_begin,
                     (hipEvent_t)ev_main_end);
}
