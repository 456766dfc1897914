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
// What bounds the main kernel: the vector issue port and power.  Two waves per SIMD in opposite phases on 16x16x32 matrix
// instructions: 2660 cycles per 64-key tile and 256 rows, 2176 of them matrix time (3220 before the phases were cut to
// what the port has room for: see the loop), at 1.75 GHz under the power limit (1.84 before).  16K context at r = 10 %: 219 -> 209
// us with the merge, 64K: 3020 -> 2730 us (1.28 PFLOP/s), seven heads per KV head at 32K: 1340 -> 1200 us.
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
constexpr int kStages = 4;                           // of the LDS ring
// A direct-to-LDS load brings four keys, 1 KB in one piece; the pieces are padded apart so that the fragment reads find 64 banks
// at addresses that differ by constants only (no address arithmetic between the products; see the loads)
constexpr int kKPiece = 1024 + 64, kVPiece = 1024 + 32;
constexpr int kVAt = kTK / 4 * kKPiece, kStageBytes = kVAt + kTK / 4 * kVPiece;   // a stage: a K tile, then a V tile
constexpr int kAhead = 4, kKAhead = 6;               // fragments of V read ahead of the phase that multiplies them, of K ahead of S
constexpr int kTableItems = 32;                      // a multiple of 2 x 8: refilled by halves
constexpr size_t kRingBytes = (size_t)kStages * kStageBytes;
constexpr size_t kAttnLds = kRingBytes + (size_t)kAttnWaves * kTableItems * 32;   // 142 KB

__global__ void __launch_bounds__(kPlanThreads)
attn_plan_kernel(attn_plan p, const int *__restrict__ act_idx, int n_act, const int *__restrict__ seg_start,
                 int n_req, int G, int wgs_per_head, int item_cost) {
  __shared__ __align__(16) int wave_tot[kPlanThreads / 64];
  __shared__ int small[kPlanLdsInts];
  attn_plan_body(p, act_idx, [&](int i) { return act_idx[i]; }, n_act, seg_start, n_req, G, wgs_per_head, item_cost, wave_tot, small, kPlanLdsInts);
}

struct attn_args {
  const void *q, *k, *v;
  void *out;
  const int *act_idx;
  const int *seg_start;
  const int *tok_req;
  attn_plan plan;
  int n_act, Hq, Hkv, d;
  uint32_t inv_G;                      // ceil(2^32 / G), G > 1: x / G = mulhi(x, inv_G) below 2^28
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

// One workgroup per share of a KV head's work: it runs the items of its share in order, their 64-key tiles as one stream.
__global__ void __launch_bounds__(kAttnThreads, 1)
attn_bf16_kernel(attn_args a) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int g = blockIdx.x % a.Hkv, wg = blockIdx.x / a.Hkv;
  // What the workgroup is to do, its first item included, is requested at once: one look-up behind the other they were three round trips
  // to what another XCD has just written, in front of the first keys (layer pass of 2K rows 110.8 -> 108.5 us with the merge, of 5K 155 -> 153.7)
  const int max_wgs = a.plan.counters[3], n_wgs = a.plan.counters[2];
  const int item_begin = a.plan.wg_start[wg], item_end = a.plan.wg_start[wg + 1];
  attn_item first_item = {};
  if (a.plan.wg_first) first_item = reinterpret_cast<const attn_item *>(a.plan.wg_first)[wg];
  asm volatile("" :: "s"(max_wgs), "s"(n_wgs), "s"(item_begin), "s"(item_end), "s"(first_item.k_begin), "s"(first_item.m_end));
  // a plan made with another number of workgroups per head lies elsewhere in the workspace: touch nothing
  if (max_wgs != a.plan.max_wgs || wg >= n_wgs || item_begin >= item_end) return;
  if (!a.plan.wg_first) first_item = reinterpret_cast<const attn_item *>(a.plan.items)[item_begin];
  const int G = a.Hq / a.Hkv;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, lg = lane >> 4, grp = wave >> 2;
  const bf16_t *__restrict__ Q = (const bf16_t *)a.q;
  const float c2 = a.scale2;

  // ---- items of this workgroup, looked up ahead into a ring of the wave's own.  The stream of loads is at most three items
  // ahead of the products: when it enters the middle of one half, the other half holds nothing that is still wanted
  typedef int i32x4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) i32x4 lds_i32x4;
  lds_i32x4 *table = (lds_i32x4 *)(lds + kRingBytes + wave * (kTableItems * sizeof(attn_item)));
  auto table_load = [&](int first) { return reinterpret_cast<const i32x4 *>(a.plan.items)[2 * min(first + lane / 2, item_end - 1) + (lane & 1)]; };
  auto table_store = [&](int first, int n, const i32x4 &x) { // items first .. first + n - 1 (2 n <= 64)
    const int i = first + lane / 2;
    if (lane < 2 * n && i < item_end) table[(i - item_begin) % kTableItems * 2 + (lane & 1)] = x;
  };
  const i32x4 first_items = table_load(item_begin);
  auto item_at = [&](int i) {
    const lds_i32x4 *d = table + (i - item_begin) % kTableItems * 2;
    const i32x4 x = d[0], y = d[1];
    attn_item it;
    it.k_begin = __builtin_amdgcn_readfirstlane(x.x); it.k_end = __builtin_amdgcn_readfirstlane(x.y);
    it.kv_len = __builtin_amdgcn_readfirstlane(x.z); it.m0 = __builtin_amdgcn_readfirstlane(x.w);
    it.m_end = __builtin_amdgcn_readfirstlane(y.x); it.a0 = __builtin_amdgcn_readfirstlane(y.y);
    it.base = __builtin_amdgcn_readfirstlane(y.z); it.whole = __builtin_amdgcn_readfirstlane(y.w);
    return it;
  };

  // ---- loads: both tiles of 64 keys x 256 bytes by direct-to-LDS loads, 4 keys per wave instruction, two instructions
  // per wave and tile; lane (l16, lg) brings 16 bytes of the lg-th of its keys to slot l16 of that key's 256 bytes.
  // K: piece t holds keys 4 t .. + 3, slot s of key r the 16 bytes number s ^ (r % 4): the 16 keys a quarter wave reads at
  // one place then lie at 64 (r / 4) + 16 (place ^ (r % 4)) modulo 256, all 64 banks once.
  // V: piece t holds keys 16 (t / 4) + t % 4 + 4 j, j = 0 .. 3, with the halves of a key's row swapped for odd j: the 8 keys x 32
  // bytes a half wave hands to the transposing read (t % 4 = 0 .. 3, two j) lie at 32 (t % 4) + 128 (j % 2), all banks once.
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds;
  const uint32_t pitch = (uint32_t)a.Hkv * kD * sizeof(bf16_t);
  const uint32_t kkey_off = (uint32_t)(4 * wave + lg) * pitch;         // key of the lane in instruction 0; + 32 keys in instruction 1
  const uint32_t vkey_off = (uint32_t)(16 * (wave >> 2) + (wave & 3) + 4 * lg) * pitch;
  const uint32_t kpiece = 16 * (l16 ^ lg), vpiece = 16 * (l16 ^ (8 * (lg & 1)));
  const uint32_t k_off[2] = {kkey_off + kpiece, kkey_off + 32 * pitch + kpiece}, v_off[2] = {vkey_off + vpiece, vkey_off + 32 * pitch + vpiece};
  // The descriptors of a request and head end behind the item's last visible key: past it the loads bring zeros.  l_k, l_v: of
  // the tile whose K comes next, v_v: of the one before it
  int l_item = item_begin;
  u32x4 l_k, l_v, v_v;
  attn_stream ld = {0, 0, 0};
  bool l_same = false;                                       // both tiles are of one item
  constexpr uint32_t kRowBytes = kD * sizeof(bf16_t);
  auto load_from = [&](const attn_item &d) {
    ld.enter(d.k_begin, d.k_end, pitch);
    const uint32_t bytes = attn_stream::bytes(d.kv_len, pitch, kRowBytes);
    const uint64_t at = ((uint64_t)(uint32_t)d.base * a.Hkv + g) * kRowBytes, pk = (uint64_t)a.k + at, pv = (uint64_t)a.v + at;
    l_k = u32x4{(uint32_t)pk, (uint32_t)(pk >> 32) & 0xffffu, bytes, 0x00020000u};
    l_v = u32x4{(uint32_t)pv, (uint32_t)(pv >> 32) & 0xffffu, bytes, 0x00020000u};
  };
  auto load_step = [&]() { ld.step(pitch, l_k[2], kRowBytes); };
  auto load_on = [&]() {                                     // what else there is to do behind load_step
    v_v = l_v;
    l_same = ld.same();
    if (!l_same) {
      if (l_item + 1 < item_end) {
        load_from(item_at(++l_item));
        if ((l_item - item_begin) % (kTableItems / 2) == kTableItems / 4)
          table_store(l_item + kTableItems / 4, kTableItems / 2, table_load(l_item + kTableItems / 4));
      } else {
        ld.end();
      }
    }
  };
  // Inline assembly on purpose: the compiler then neither treats these as LDS writes (it would wait for all of them before
  // every LDS read) nor moves memory accesses across them; the waits for them are the explicit s_waitcnt below.
  auto dma = [&](const u32x4 &base, uint32_t at, uint32_t off, uint32_t stage, uint32_t to) {
    asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %3, %4 offen lds"
                 :: "s"(stage), "s"(to), "v"(off), "s"(base), "s"(at) : "memory", "scc");
  };
  const uint32_t to_k = lds_base + wave * kKPiece, to_v = lds_base + kVAt + wave * kVPiece;
  auto load_k = [&](uint32_t stage, int i) { dma(l_k, ld.at, k_off[i], stage, to_k + i * 8 * kKPiece); };
  auto load_v = [&](uint32_t stage, int i) { dma(v_v, ld.v_at, v_off[i], stage, to_v + i * 8 * kVPiece); };

  // ---- rows of an item: lane (l16, lg) holds rows m0 + 32 wave + 16 rb + l16 ---------------------------------------
  bf16x8 qf[2][4];
  int limit[2], min_limit, max_limit;                        // last visible key of the rows (request-relative)
  uint32_t out_row[2], prev_row[2];                          // row of the output; bit 31: not stored
  attn_item cur;
  auto load_rows = [&]() {
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
      const int m = cur.m0 + 32 * wave + 16 * rb + l16, mc = min(m, cur.m_end - 1);
      const int ar = G == 1 ? mc : (int)__umulhi((uint32_t)mc, a.inv_G), arow = cur.a0 + ar, hq = g * G + mc - ar * G;
      out_row[rb] = (uint32_t)arow * a.Hq + hq;
      limit[rb] = a.act_idx[arow];
      if (m >= cur.m_end) out_row[rb] |= 1u << 31;
    }
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
      const bf16_t *qp = Q + (size_t)(out_row[rb] & ~(1u << 31)) * kD + lg * 8;
#pragma unroll
      for (int ds = 0; ds < 4; ++ds) qf[rb][ds] = *reinterpret_cast<const bf16x8 *>(qp + 32 * ds);
    }
  };
  auto row_limits = [&]() {                                  // limits ascend with the rows
    limit[0] -= cur.base; limit[1] -= cur.base;
    min_limit = __builtin_amdgcn_readlane(limit[0], 0);
    max_limit = __builtin_amdgcn_readlane(limit[1], 15);
  };

  f32x4 o[8][2], st[4][2];
  uint32_t pu[2][2][4];                                      // P of the tile before, pairs of bf16, [32 keys][row block]
  float ref[2], nref[2];                                     // exponent reference (-inf: no key seen) and what is added to an exponent
  // Row sums of P, by the matrix pipe (an all-ones V): every register.  They are fp32 sums of the weights as the product with V
  // uses them, rounded to bf16: an output is then an exact mean of the values it sees, and the weights' roundings cancel where
  // values are alike.  Relative error against float64, unrounded weights summed -> these: 8 matching rows of 100 2.04e-3
  // -> 1.99e-3 at 500 keys, 2.11e-3 -> 2.02e-3 at 2048; plain normal logits 2.20e-3 -> 2.18e-3 and 2.24e-3 -> 2.23e-3; flat logits, one
  // key with all the weight, and 16K keys and more: the same within 1 %.
  f32x4 osum[2];
  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = (bf16_t)1.0f;
  asm volatile("" : "+v"(ones));                             // kept in registers
  int prev_item = item_begin, prev_whole = 0;
  auto store_rows = [&]() {
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
      const float total = osum[rb][0];
      if (prev_whole) {
        const float inv = 1.0f / total;
        if (prev_row[rb] < 1u << 31) {
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
        f32x4 *p = reinterpret_cast<f32x4 *>(a.plan.part_o) + (((size_t)g * a.plan.max_items + prev_item) * (kTM / 16) + 2 * wave + rb) * 512 + lane;
#pragma unroll
        for (int db = 0; db < 8; ++db) p[64 * db] = o[db][rb];
        if (lg == 0) a.plan.part_ml[pr] = make_float2(ref[rb], total);
      }
    }
  };

  // ---- fragments: K (16 keys x 32 dims, lane = key l16, 16 bytes number 4 ds + lg) by one 16-byte read, V^T (16 dims x 32 keys)
  // by two transposing 8-byte reads: lane (l16, lg) then holds dim l16, keys 4 lg .. + 3 of two 16-key blocks, which is the order
  // in which the S^T accumulators hold P (accumulator r of key block b: key 16 b + 4 lg + r, row l16)
  const uint32_t kaddr = (l16 >> 2) * kKPiece + (l16 & 3) * 256 + 16 * (lg ^ (l16 & 3));
  const uint32_t vaddr = kVAt + (l16 >> 2) * kVPiece + lg * 256 + 8 * (l16 & 3);
  const uint32_t vaddr0 = vaddr + 128 * (lg & 1), vaddr1 = vaddr + 128 * (~lg & 1);      // dims 0 .. 63, 64 .. 127
  typedef __attribute__((address_space(3))) s16x4 *tr_ptr;
  s16x4 va[16][2];                                           // V^T fragment N = 8 ks + block of 16 dims, its two halves
  bf16x8 kf[16];                                             // K fragment N = 4 ds + block of 16 keys
  const unsigned char *kp = lds + kaddr, *vp0, *vp1;
#define A3_KREAD(N) kf[N] = *reinterpret_cast<const bf16x8 *>(kp + 64 * ((N) >> 2) + 4 * kKPiece * ((N) & 3));
#define A3_VREAD(N, H) va[N][H] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)(((N) & 4 ? vp1 : vp0) + 32 * ((N) & 3) + 4 * kVPiece * (2 * ((N) >> 3) + (H))));
#define A3_VF(N) __builtin_bit_cast(bf16x8, __builtin_shufflevector(va[N][0], va[N][1], 0, 1, 2, 3, 4, 5, 6, 7))
#define A3_P(KS, RB) __builtin_bit_cast(bf16x8, u32x4{pu[KS][RB][0], pu[KS][RB][1], pu[KS][RB][2], pu[KS][RB][3]})
#define A3_FENCE __builtin_amdgcn_sched_barrier(0);

  cur = first_item;
  prev_row[0] = prev_row[1] = 1u << 31;
  load_from(first_item);
  // the looked-up items are needed below only where the first has fewer than three tiles: else nothing waits for them before the keys are requested
  const bool at_once = ld.left >= 3;
  if (!at_once) table_store(item_begin, kTableItems, first_items);
  uint32_t s0 = 0, s1 = kStageBytes, s2 = 2 * kStageBytes, s3 = 3 * kStageBytes;     // stages of tiles u .. u + 3
  load_k(s0, 0); load_k(s0, 1); load_step(); load_on();
  load_k(s1, 0); load_k(s1, 1); load_v(s0, 0); load_v(s0, 1); load_step(); load_on();
  load_rows();
  load_k(s2, 0); load_k(s2, 1); load_v(s1, 0); load_v(s1, 1); load_step();
  if (at_once) table_store(item_begin, kTableItems, first_items);
  load_on();
  __builtin_amdgcn_s_waitcnt(0);                                         // this wave's part of tiles 0, 1 and K of tile 2 has landed
  __builtin_amdgcn_s_barrier();                                          // ... and everybody's
  if (grp == 1) __builtin_amdgcn_s_barrier();                            // one phase behind

  // The two waves of a SIMD belong to different groups and run in opposite phases, one barrier apart: while one has the
  // matrix pipe (P V of tile u - 1, then S of tile u), the other does the softmax of its tile on the vector unit.  Group 0
  // multiplies tile u in phase 2 u, group 1 in phase 2 u + 1.  K of tile u + 3 and V of tile u + 2 are requested at the end of the
  // matrix phase of tile u, over K of tile u - 1 and V of tile u - 2, which both groups have read; in the vector phase every wave
  // waits for all but these (attn_waits_behind), so that K of tile u + 2 and V of tile u + 1 are there when group 0 reads them.
  // What a phase may hold, measured in a loop of nothing else (cycles per tile of two phases):
  //   68 products with at most one LDS read right behind each: 2250.  A read costs nothing there, but 6 - 12 cycles of its wave behind
  //   a vector instruction or another read.
  //   with 32 scalings, 32 exponentials, 16 conversions and 8 ors in the other wave: 2280.  A product takes 8 cycles of the SIMD's
  //   vector issue, an exponential 8, any other vector instruction 4: 544 + 480 of the 1088 cycles, so nothing else is done
  //   per element: the row sums are matrix products, and instead of the maxima of a tile the bits of the weights are or-ed.
  //   barrier four products before the end of the matrix phase instead of one: 2820; fragments read ahead at the start of the vector
  //   phase instead of its end: + 350; the four requests in the vector phase: + 120 .. 200, between products without a read: + 60;
  //   s_setprio around the products: + 150; a scalar instruction at either end of a phase: + 9 each, between products: 0.
  // Hence tiles with nothing special to them run in a loop of their own without a branch or a bookkeeping instruction.
  int k0 = cur.k_begin, item = item_begin;
  bool first = true, has_prev = false;
  bool act = false, act_prev = false;                        // a wave whose rows all end before a tile leaves its products out
  // Weights of the N-th pair of S values, N = 0 .. 15 (key block N / 4, registers 2 (N / 2 % 2) and + 1, row block N % 2)
  // (the empty asm statement keeps the compiler from moving the arithmetic behind the products)
#define A3_EXP(N)                                                                                                      \
  {                                                                                                                    \
    const int b_ = (N) >> 2, r_ = (N) & 2, rb_ = (N) & 1;                                                              \
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));                                                         \
    bf16x2 t_;                                                                                                         \
    t_[0] = a3_f2bf(fast_exp2(fmaf(st[b_][rb_][r_], c2, nref[rb_])));                                                  \
    t_[1] = a3_f2bf(fast_exp2(fmaf(st[b_][rb_][r_ + 1], c2, nref[rb_])));                                              \
    pu[b_ >> 1][rb_][2 * (b_ & 1) + r_ / 2] = __builtin_bit_cast(uint32_t, t_);                                        \
    asm volatile("" : "+v"(pu[b_ >> 1][rb_][2 * (b_ & 1) + r_ / 2]));                                                  \
  }
  // ---- matrix phase: row sums and P V of keys 0 .. 31 of the tile before, then of keys 32 .. 63; fragments of V are read 9
  // products before their first, and the first of K at the end
  auto pv_products = [&]() {
#pragma unroll
    for (int m = 0; m < 36; ++m) {
      const int ks = m / 18, i = m % 18 - 2, rb = m & 1;
      if (i < 0) osum[rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, A3_P(ks, rb), osum[rb], 0, 0, 0);
      else o[i >> 1][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A3_VF(8 * ks + (i >> 1)), A3_P(ks, rb), o[i >> 1][rb], 0, 0, 0);
      A3_FENCE
      if (m < 2 * (16 - kAhead)) A3_VREAD(kAhead + (m >> 1), m & 1)
      else if (m < 2 * (16 - kAhead) + kKAhead) A3_KREAD(m - 2 * (16 - kAhead))
      A3_FENCE
    }
  };
  // the loads of K of tile u + 3 and V of tile u + 2, and the addresses of the phases to come, in six parts
  auto between = [&](int i) {
    if (i == 0) load_k(s3, 0);
    if (i == 1) load_k(s3, 1);
    if (i == 2) load_v(s2, 0);
    if (i == 3) load_v(s2, 1);
    if (i == 4) { vp0 = lds + (vaddr0 + s0); vp1 = lds + (vaddr1 + s0); load_step(); }
    if (i == 5) { const uint32_t t = s0; s0 = s1; s1 = s2; s2 = s3; s3 = t; kp = lds + (kaddr + s0); }
  };
  auto s_products = [&]() {
#pragma unroll
    for (int m = 0; m < 32; ++m) {
      const int n = m >> 1, rb = m & 1;
      if (m == 31) __builtin_amdgcn_s_barrier();
      A3_FENCE
      st[n & 3][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[n], qf[rb][n >> 2], n < 4 ? f32x4{0.f, 0.f, 0.f, 0.f} : st[n & 3][rb], 0, 0, 0);
      A3_FENCE
      if (!(m & 1) && kKAhead + n < 16) A3_KREAD(kKAhead + n)
      if ((m & 1) && m >= 19 && m < 31) between((m - 19) >> 1);
      A3_FENCE
    }
  };
  // ---- vector phase
  auto weights = [&]() -> uint32_t {                         // the or of their bits
    uint32_t bits = 0;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      A3_EXP(q)
      if (q & 1) bits |= pu[q >> 3][0][(q >> 1) & 3] | pu[q >> 3][1][(q >> 1) & 3];
      A3_FENCE
    }
    return bits;
  };
  auto maximum = [&](int rb) {
    float mx = -INFINITY;
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int r = 0; r < 4; r += 2) mx = fmaxf(fmaxf(mx, st[b][rb][r]), st[b][rb][r + 1]);
    return fmaf(groups_max(mx), c2, 7.0f);
  };
  // Lazy rescaling: the exponent reference lies 7 above the largest exponent of the row when it was set, so weights are about
  // 2^-7 and below, and moves when one reaches 2 (a bf16 that does has bit 14 set, and only such a one: one test of the or of
  // all bits), so the accumulators are rescaled a handful of times per row instead of whenever the maximum moves.
  // A row that has seen nothing but logits of -inf has no reference yet: what is added to its exponents then leaves -inf a weight of
  // 0 and makes that of its first finite logit infinite, however small the logit, so that the reference is set there.
  constexpr float kUnset = 3.402823466e38f;
  auto check = [&](uint32_t bits) {
    if (__any((bits & 0x40004000u) != 0)) {
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) {
        const float new_ref = fmaxf(ref[rb], maximum(rb));
        const float alpha = new_ref == -INFINITY ? 1.0f : fast_exp2(ref[rb] - new_ref);
        ref[rb] = new_ref;
        nref[rb] = new_ref == -INFINITY ? kUnset : -new_ref;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          osum[rb][r] *= alpha;
#pragma unroll
          for (int db = 0; db < 8; ++db) o[db][rb][r] *= alpha;
        }
      }
#pragma unroll
      for (int q = 0; q < 16; ++q) A3_EXP(q)
    }
  };
  // all but the four requests of this tile have landed; memory accesses stay on their side of it
  auto landed = [&]() {
    asm volatile("" ::: "memory");
    A3_FENCE
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(4));
    A3_FENCE
    asm volatile("" ::: "memory");
  };
  auto phase_end = [&]() {
    A3_FENCE
#pragma unroll
    for (int n = 0; n < kAhead; ++n) { A3_VREAD(n, 0) A3_VREAD(n, 1) }
    A3_FENCE
    __builtin_amdgcn_s_barrier();
    A3_FENCE
  };

  for (;;) {
    if (act_prev) {
      pv_products();
    } else {
#pragma unroll
      for (int n = 0; n < kKAhead; ++n) A3_KREAD(n)
    }
    if (first) {
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));              // the rows of the new item
      row_limits();
      act = k0 <= max_limit;
      if (has_prev) store_rows();                            // (before the loads of this tile: waits count stores too)
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) {
#pragma unroll
        for (int db = 0; db < 8; ++db) o[db][rb] = f32x4{0.f, 0.f, 0.f, 0.f};
        osum[rb] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    }
    if (act) {
      s_products();
    } else {
#pragma unroll
      for (int i = 0; i < 6; ++i) between(i);
      __builtin_amdgcn_s_barrier();
    }
    A3_FENCE
    if (k0 + kTK - 1 > min_limit) {                          // tile touches the causal boundary of some row
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) {
        const int seen = act ? limit[rb] - k0 - 4 * lg : -1;
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (16 * b + r > seen) st[b][rb][r] = -INFINITY;
      }
    }
    if (first) {
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) {
        ref[rb] = maximum(rb);
        nref[rb] = ref[rb] == -INFINITY ? kUnset : -ref[rb];
      }
    }
    check(weights());
    load_on();
    act_prev = act;
    const bool fresh = first;
    first = false;
    k0 += kTK;
    if (attn_waits_behind(fresh, k0 >= cur.k_end)) landed();
    if (k0 >= cur.k_end) {                                   // (the rows are requested behind the wait, which does not count them)
      prev_item = item; prev_whole = cur.whole;
      prev_row[0] = out_row[0]; prev_row[1] = out_row[1];
      has_prev = first = true;
      if (++item < item_end) {
        cur = item_at(item);
        load_rows();
        k0 = cur.k_begin;
      }
    }
    act = k0 <= max_limit;
    phase_end();
    if (item == item_end) break;
    if (fresh || first) continue;
    // Tiles of the same items here and in the stream of loads with nothing masked; then tiles that this wave only loads for
    const int rest = l_same ? ld.calm((cur.k_end - k0 + kTK - 1) / kTK) : 0;
    if (act && act_prev) {
      const int calm = min((min_limit + 1 - k0) / kTK, rest);
      if (calm > 0) __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));  // (or the compiler waits in the loop, for rows loaded long ago)
      for (int c = 0; c < calm; ++c) {
        pv_products();
        s_products();
        check(weights());
        landed();
        phase_end();
      }
      if (calm > 0) {
        k0 += calm * kTK;
        ld.pass(calm);
      }
    } else if (!act && !act_prev && rest > 0) {
      for (int c = 0; c < rest; ++c) {
#pragma unroll
        for (int i = 0; i < 6; ++i) between(i);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(4));
        __builtin_amdgcn_s_barrier();
      }
      k0 += rest * kTK;
      ld.pass(rest);
    }
  }
  // ---- P V of the last tile
  if (act_prev) {
#pragma unroll
    for (int n = kAhead; n < 16; ++n) { A3_VREAD(n, 0) A3_VREAD(n, 1) }
#pragma unroll
    for (int n = 0; n < 16; ++n)
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) o[n & 7][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A3_VF(n), A3_P(n >> 3, rb), o[n & 7][rb], 0, 0, 0);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) osum[rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, A3_P(ks, rb), osum[rb], 0, 0, 0);
  }
#undef A3_P
#undef A3_VF
#undef A3_EXP
#undef A3_KREAD
#undef A3_VREAD
#undef A3_FENCE
  if (grp == 0) __builtin_amdgcn_s_barrier();
  store_rows();
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));                  // the tail loads have landed before LDS is released
}

// Merges the partial results of tiles that were cut into key segments, in segment order.
// One workgroup per (tile, KV head, 32 of the tile's rows), in the order in which the lanes of the main kernel hold them: wave
// (rb, half) merges 16 rows x 64 dims, lane (l16, lg) of it row l16, dims 16 i + 4 lg .. + 3, and every load is 1 KB in one piece.
__global__ void __launch_bounds__(256)
attn_combine_kernel(attn_args a) {
  const int t = blockIdx.x, g = blockIdx.y;
  // (all of it looked up at once: the merge of 2K context 7.5 -> 7.2 us)
  const int2 tb = a.plan.tile_b[t];
  const int4 ta = a.plan.tile_a[t];
  const int n_tiles = a.plan.counters[0], max_wgs = a.plan.counters[3];
  asm volatile("" :: "s"(tb.x), "s"(tb.y), "s"(ta.x), "s"(ta.y), "s"(ta.w), "s"(n_tiles), "s"(max_wgs));
  const int nseg = tb.y;
  if (max_wgs != a.plan.max_wgs || t >= n_tiles || nseg <= 1) return;
  const int G = a.Hq / a.Hkv;
  const int lane = threadIdx.x & 63, l16 = lane & 15, lg = lane >> 4, rb = (threadIdx.x >> 6) & 1, half = threadIdx.x >> 7;
  const int ml = blockIdx.z * 32 + 16 * rb + l16;
  const int m = ta.y + ml;
  if (m >= ta.w) return;
  const int ar = G == 1 ? m : (int)__umulhi((uint32_t)m, a.inv_G), arow = ta.x + ar, hq = g * G + m - ar * G;
  const size_t p0 = (size_t)g * a.plan.max_items + tb.x;
  const float2 *ml_p = a.plan.part_ml + p0 * kTM + ml;
  const f32x4 *o_p = reinterpret_cast<const f32x4 *>(a.plan.part_o) + (p0 * (kTM / 16) + 2 * blockIdx.z + rb) * 512 + 256 * half + lane;
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
      for (int i = 0; i < 4; ++i) v[u][i] = o_p[s * (kD / 4) + 64 * i];
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
  bf16_t *orow = (bf16_t *)a.out + ((size_t)arow * a.Hq + hq) * kD + 64 * half;
  // by lane-row swaps of two blocks of 16 dims lane group lg gets dims 8 lg .. + 7 of them (a lane's own dims, stored as 8 bytes, 32 in
  // one piece: merge of eight requests of 1000 rows 10.7 us, now 9.6; of 64K context 17.9 and 16.4)
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    u32x2 w[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      bf16x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = a3_f2bf(acc[8 * h + 4 * i + e] * inv);
      w[i] = __builtin_bit_cast(u32x2, v);
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      auto r = __builtin_amdgcn_permlane32_swap(w[0][e], w[1][e], false, false);
      r = __builtin_amdgcn_permlane16_swap(r[0], r[1], false, false);
      w[0][e] = r[0]; w[1][e] = r[1];
    }
    *reinterpret_cast<u32x4 *>(orow + 32 * h + 8 * lg) = u32x4{w[0][0], w[0][1], w[1][0], w[1][1]};
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
// Sixteen waves (64 coordinates) merge twice as much for blocks half as many: 108 rows x 8 heads x 544 keys 10.9 -> 12.3 us, 32 query heads
// on 8 57 -> 65 for 339 rows of 2048 keys, 85 -> 115 for 3 x 346 of 1096; only above some 4000 keys, with as many workgroups as run at
// once, are they faster (1264 rows of 8064 keys, 2 KV heads, 206 -> 178; 8 KV heads 193 -> 198).
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
  const int first = a.seg_start[0];                            // of one request: read beside the row number, not behind it
  const int t = a.act_idx[arow], req = a.tok_req ? a.tok_req[t] : 0;
  const int first_key = a.tok_req ? a.seg_start[req] : first;
  // the rows of one request at a time (rows are ascending: nearly always all of them), found in the lanes that hold them: lane x of a
  // group belongs to row a0 + x / G, the last ones to the last row (with a loop over the rows' requests in memory 108 rows x 544 keys took 13.3 us, now 10.9)
  for (int b0 = a0; b0 < a_end;) {
    const int r = __builtin_amdgcn_readlane(req, (b0 - a0) * G), base = __builtin_amdgcn_readlane(first_key, (b0 - a0) * G);
    const uint32_t later = ((uint32_t)__ballot(req != r) & 0xffffu) >> ((b0 - a0) * G);
    const int b1 = later ? b0 + (int)__builtin_ctz(later) / G : a_end;
    const bool mine = req == r && l16 < (a_end - a0) * G;
    const int limit = mine ? t - base : -1;                    // last visible key (request-relative)
    const int n_keys = __builtin_amdgcn_readlane(t, (b1 - 1 - a0) * G) - base + 1;
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
         a3_align_up((tiles + 1) * sizeof(int), 256) + a3_align_up(items * 2 * sizeof(int4), 256) +
         a3_align_up((size_t)(attn_wgs_per_head(L) + 1) * sizeof(int), 256) + 256 +
         a3_align_up(items * L->n_kv_heads * kTM * kD * sizeof(float), 256) +
         a3_align_up(items * L->n_kv_heads * kTM * sizeof(float2), 256) + a3_align_up(kFirstBytes, 256);
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
  a.act_idx = act_idx; a.seg_start = L->seg_start; a.tok_req = L->n_req > 1 ? L->tok_req : nullptr;
  a.n_act = n_act; a.Hq = L->n_q_heads; a.Hkv = L->n_kv_heads; a.d = L->head_dim;
  a.scale2 = a3_scale_of(L) * kLog2e;
  const unsigned G = (unsigned)(L->n_q_heads / L->n_kv_heads);
  a.inv_G = G > 1 ? (uint32_t)(((1ull << 32) + G - 1) / G) : 0;
  memset(&a.plan, 0, sizeof(a.plan));
  if (L->dtype == A3_BF16) {
    // Required: offsets of a request's tiles and the sizes of its descriptors are 32-bit byte counts (attn_stream).  The furthest lane
    // of a load lies 63 rows behind the last visible key; 128 rows are kept in hand
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
                         L->n_req, L->n_q_heads / L->n_kv_heads, wgs_per_head, attn_item_cost(L, n_act));
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
