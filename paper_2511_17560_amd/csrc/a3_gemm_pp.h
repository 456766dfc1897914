// The main loop and the epilogue's lane layout of the row-tiled bf16 MFMA GEMM that the Q/K/V projection (Eq. 5, first
// lines; a3_proj.hip) and the three GEMMs of H(.) (a3_block.hip) share.  One workgroup of eight waves forms
//     acc[BM weight rows][BN activation rows] = W_tile X_tile^T,        BM = 32 IB, BN = 64 JB
// wave (grp, wn) = (wave / 4, wave % 4) owning weight rows 16 IB grp .. and activation rows 16 JB wn ..
// Both operands are reduction-contiguous in memory and go from global memory straight into LDS.  Which memory row an
// LDS row is - a head's weight row, a gate or an up row, a gathered hidden row - is the caller's business.
// Device code, inlined into each translation unit (no relocatable device code).
#pragma once

#include "a3_internal.h"
#include "a3_gemm_tiles.h"

namespace {

// s_waitcnt immediate that waits until at most n vector-memory operations are outstanding and
// nothing else (gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8)
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }

// SW / SX: LDS stages of the weight and of the activation ring (a stage = 64 elements of the reduction, 128 bytes a row)
template <int IB, int JB, int SW, int SX>
struct gemm_pp {
  static constexpr int kIB = IB, kJB = JB, kSW = SW, kSX = SX;
  static constexpr int BM = 32 * IB, BN = 64 * JB, L = 2 * IB;
  static constexpr int kWStage = BM * 128, kXStage = BN * 128, kXBase = SW * kWStage;
  static constexpr int kLW = BM / 32, kLX = BN / 32;           // direct-to-LDS loads per wave of a group and slab
  static constexpr size_t kLdsBytes = (size_t)SW * kWStage + (size_t)SX * kXStage;
  static_assert(kLdsBytes <= 160 * 1024 && SW >= 3 && SX >= 2, "LDS rings");

  // Row r of a group's 16 IB weight rows as (half q, feature f < 8 IB): chosen so that after transpose() a lane holds
  // L consecutive features of half 0 and the same L of half 1 of one activation row.
  __device__ static __forceinline__ void row_of(int r, int &q, int &f) {
    if (IB == 8) { q = r >> 6; f = r & 63; }
    else { q = (r >> 3) & 1; f = 8 * (r >> 4) + (r & 7); }
  }
  template <class WBase, class WOff, class XBase, class XOff>
  __device__ static __forceinline__ void mainloop(f32x4 (&acc)[IB][JB], unsigned char *lds, int n_slabs, WBase w_base, WOff w_off, XBase x_base,
                                                  XOff x_off);
};

// acc block (i, j), register r of a lane: weight row 16 i + 4 (lane / 16) + r, activation row 16 j + lane % 16.
// A 4 x 4 transposition of (block, lane group) by lane-row swaps leaves lane group g with all 16 rows of block g (and of
// block 4 + g): lo / hi are the L features 8 IB q + L g .. of halves q = 0 and 1.
__device__ __forceinline__ void gemm_swap16(float &a, float &b) {
  const auto t = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b), false, false);
  a = __builtin_bit_cast(float, (unsigned)t[0]);
  b = __builtin_bit_cast(float, (unsigned)t[1]);
}
__device__ __forceinline__ void gemm_swap32(float &a, float &b) {
  const auto t = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b), false, false);
  a = __builtin_bit_cast(float, (unsigned)t[0]);
  b = __builtin_bit_cast(float, (unsigned)t[1]);
}
__device__ __forceinline__ void gemm_transpose4(const f32x4 &b0, const f32x4 &b1, const f32x4 &b2, const f32x4 &b3, float (&out)[16]) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float x0 = b0[r], x1 = b1[r], x2 = b2[r], x3 = b3[r];
    gemm_swap16(x0, x1);
    gemm_swap16(x2, x3);
    gemm_swap32(x0, x2);
    gemm_swap32(x1, x3);
    out[r] = x0; out[4 + r] = x1; out[8 + r] = x2; out[12 + r] = x3;
  }
}
template <int IB, int JB>
__device__ __forceinline__ void gemm_lane_values(const f32x4 (&acc)[IB][JB], int j, float (&lo)[2 * IB], float (&hi)[2 * IB]) {
  if constexpr (IB == 8) {
    gemm_transpose4(acc[0][j], acc[1][j], acc[2][j], acc[3][j], lo);
    gemm_transpose4(acc[4][j], acc[5][j], acc[6][j], acc[7][j], hi);
  } else {
    float t[16];
    gemm_transpose4(acc[0][j], acc[1][j], acc[2][j], acc[3][j], t);
#pragma unroll
    for (int e = 0; e < 8; ++e) { lo[e] = t[e]; hi[e] = t[8 + e]; }
  }
}

// w_base(r0): start (first slab wanted) of the memory behind weight rows r0 .. r0 + 7 of the tile, wave-uniform;
// w_off(r): byte offset of row r against it (32 bits).  x_base / x_off likewise for activation rows (rows past the end of
// a list are clamped by the caller: computed, never stored).  n_slabs >= 1 slabs of 64 elements.
// On return every load has landed and every wave has left LDS.
//
// Matrix instructions are 16x16x32: with operands that are not all alike this chip's clock under matrix load is set by
// power, and a loop of nothing but 16x16x32 on N(0, 1) values runs at 2.14 PFLOP/s where 32x32x16 reaches 1.74 - 1.86.
// (One operand stays from each instruction to the next: 1 - 3 % of the same.)
template <int IB, int JB, int SW, int SX>
template <class WBase, class WOff, class XBase, class XOff>
__device__ __forceinline__ void gemm_pp<IB, JB, SW, SX>::mainloop(f32x4 (&acc)[IB][JB], unsigned char *lds, int n_slabs, WBase w_base, WOff w_off,
                                                                  XBase x_base, XOff x_off) {
  using P = gemm_pp;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, lg = lane >> 4;
  const int grp = wave >> 2, wn = wave & 3;
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds;
#pragma unroll
  for (int i = 0; i < IB; ++i)
#pragma unroll
    for (int j = 0; j < JB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Loads: one wave instruction brings 8 rows x 128 B (whole cache lines) to 1 KB of LDS; slot s of row r holds the
  // 16-byte piece s ^ ((r >> 1) & 7), so that the 16 rows a quarter wave reads at one piece index touch all 64 banks
  // once.  Group 0 brings the weights, group 1 the activation rows.  Inline assembly on purpose: the compiler then
  // neither tracks these as LDS writes (it would put a full vmcnt(0) in front of every LDS read) nor reorders accesses
  // across them; the waits for them are the explicit s_waitcnt below.  M0 is used by nothing else here.  The s_nop is
  // the wait state between a scalar write of M0 and a direct-to-LDS load that reads it.
  constexpr int kL = P::kLW > P::kLX ? P::kLW : P::kLX;
  uint32_t src[kL];
  const char *base[kL];
  {
    const int row8 = lane >> 3, slot8 = lane & 7;
#pragma unroll
    for (int j = 0; j < kL; ++j) {
      const int r0 = 8 * (4 * j + wn), r = r0 + row8;
      const uint32_t piece = 16 * (slot8 ^ ((r >> 1) & 7));
      if (grp == 0) {
        if (j < P::kLW) { base[j] = w_base(r0); src[j] = w_off(r) + piece; }
      } else {
        if (j < P::kLX) { base[j] = x_base(r0); src[j] = x_off(r) + piece; }
      }
    }
  }
#define A3_PP_LOAD(J, STAGE, SLAB)                                                                                      \
  {                                                                                                                     \
    const char *gb_ = base[J] + (size_t)min((SLAB), n_slabs - 1) * 128;      /* past the end: the last slab, unused */    \
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"                                         \
                 :: "s"(lds_base + (uint32_t)(STAGE) + (4 * (J) + wn) * 1024), "v"(src[J]), "s"(gb_) : "memory");        \
  }
#define A3_PP_FENCE __builtin_amdgcn_sched_barrier(0);
  // fragments: 16 rows x 32 elements, lane (l16, lg) = row l16, piece 4 ks + lg
  const int swz = (l16 >> 1) & 7;
  const int frag_w = (grp * 16 * IB + l16) * 128, frag_x = P::kXBase + (wn * 16 * JB + l16) * 128;
  const int slot0 = (lg ^ swz) * 16, slot1 = ((4 + lg) ^ swz) * 16;
  bf16x8 wf[2][IB], xf[2][JB];
#define A3_PP_READ(WST, XST)                                                                                            \
  _Pragma("unroll") for (int ks = 0; ks < 2; ++ks) {                                                                    \
    const unsigned char *px = lds + (XST) + frag_x + (ks ? slot1 : slot0), *pw = lds + (WST) + frag_w + (ks ? slot1 : slot0); \
    _Pragma("unroll") for (int j = 0; j < JB; ++j) xf[ks][j] = *reinterpret_cast<const bf16x8 *>(px + j * 2048);        \
    _Pragma("unroll") for (int i = 0; i < IB; ++i) wf[ks][i] = *reinterpret_cast<const bf16x8 *>(pw + i * 2048);        \
  }
  // The two waves of a SIMD belong to different groups and run in opposite phases, one barrier apart: while one reads the
  // fragments of a slab the other multiplies, so the matrix pipe changes hands instead of idling through LDS latency.
  // Group 0 reads slab s in phase 2 s and multiplies in phase 2 s + 1, group 1 one phase later.  The loads are issued
  // between matrix instructions; the barrier that ends a matrix phase comes kTail instructions before its end, so that
  // the other wave's first ones are ready when the last ones of this wave are issued.
  constexpr int kM = 2 * IB * JB, kTail = 4;
#define A3_PP_MATH(NLOADS, LOAD, WAIT)                                                                                  \
  {                                                                                                                     \
    constexpr int step = (kM - kTail) / (NLOADS);                                                                       \
    _Pragma("unroll") for (int m = 0; m < kM; ++m) {                                                                    \
      const int ks = m / (IB * JB), i = (m / JB) % IB, j = i & 1 ? JB - 1 - m % JB : m % JB;                            \
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[ks][i], xf[ks][j], acc[i][j], 0, 0, 0);                    \
      if (m % step == step - 1 && m / step < (NLOADS)) { const int n = m / step; A3_PP_FENCE LOAD A3_PP_FENCE }         \
      if (m == kM - kTail - 1) { A3_PP_FENCE WAIT __builtin_amdgcn_s_barrier(); A3_PP_FENCE }                           \
    }                                                                                                                   \
  }
  if (grp == 0) {
    int rd = 0, ld = (SW - 1) * P::kWStage, xrd = 0;
#pragma unroll
    for (int s = 0; s < SW - 1; ++s)
#pragma unroll
      for (int j = 0; j < P::kLW; ++j) A3_PP_LOAD(j, s * P::kWStage, s)
    __builtin_amdgcn_s_waitcnt(vmcnt_imm((SW - 2) * P::kLW));
    __builtin_amdgcn_s_barrier();
    for (int s = 0; s < n_slabs; ++s) {
      A3_PP_FENCE
      A3_PP_READ(rd, xrd)
      A3_PP_FENCE
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(63) & ~(15 << 8));           // fragments in registers
      __builtin_amdgcn_s_barrier();
      A3_PP_FENCE
      __builtin_amdgcn_s_setprio(1);
      // weights of slab s + SW - 1 into the stage of slab s - 1, which both groups have read by phase 2 s - 1; slab s + 1
      // must have landed: only the SW - 2 slabs behind it may be on their way
      A3_PP_MATH(P::kLW, A3_PP_LOAD(n, ld, s + SW - 1), __builtin_amdgcn_s_waitcnt(vmcnt_imm((SW - 2) * P::kLW));)
      __builtin_amdgcn_s_setprio(0);
      ld = rd;
      rd = rd == (SW - 1) * P::kWStage ? 0 : rd + P::kWStage;
      xrd = xrd == (SX - 1) * P::kXStage ? 0 : xrd + P::kXStage;
    }
    __builtin_amdgcn_s_barrier();                                      // group 1's last matrix phase
  } else {
    int rd = 0, xrd = 0;
#pragma unroll
    for (int s = 0; s < SX; ++s)
#pragma unroll
      for (int j = 0; j < P::kLX; ++j) A3_PP_LOAD(j, P::kXBase + s * P::kXStage, s)
    __builtin_amdgcn_s_waitcnt(vmcnt_imm((SX - 1) * P::kLX));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_s_barrier();                                      // one phase behind
    for (int s = 0; s < n_slabs; ++s) {
      A3_PP_FENCE
      A3_PP_READ(rd, xrd)
      A3_PP_FENCE
      // fragments in registers, and the activation rows of slab s + 1 have landed
      __builtin_amdgcn_s_waitcnt(vmcnt_imm((SX - 2) * P::kLX) & ~(15 << 8));
      __builtin_amdgcn_s_barrier();
      A3_PP_FENCE
      __builtin_amdgcn_s_setprio(1);
      // activation rows of slab s + SX into the stage of slab s, which both groups have read
      A3_PP_MATH(P::kLX, A3_PP_LOAD(n, P::kXBase + xrd, s + SX), )
      __builtin_amdgcn_s_setprio(0);
      rd = rd == (SW - 1) * P::kWStage ? 0 : rd + P::kWStage;
      xrd = xrd == (SX - 1) * P::kXStage ? 0 : xrd + P::kXStage;
    }
  }
#undef A3_PP_MATH
#undef A3_PP_READ
#undef A3_PP_FENCE
#undef A3_PP_LOAD
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));                             // the tail loads have landed before LDS is released
}

// The same product for tiles too small to keep the matrix pipe busy (few activation rows, or little left per workgroup):
// the path from the L2 and the latencies set the pace, so all eight waves stay in the same phase, every wave brings its
// share of both operands, and the fragments of slab s + 1 are read under the products of slab s: one barrier per slab.
// ST: LDS stages, each of BM + BN rows.
template <int IB, int JB, int ST>
struct gemm_pl {
  static constexpr int kIB = IB, kJB = JB;
  static constexpr int BM = 32 * IB, BN = 64 * JB, L = 2 * IB;
  static constexpr int kStage = (BM + BN) * 128, kLoads = (BM + BN) / 64;
  static constexpr size_t kLdsBytes = (size_t)ST * kStage;
  static_assert(kLdsBytes <= 160 * 1024 && ST >= 3, "LDS ring");
  __device__ static __forceinline__ void row_of(int r, int &q, int &f) { gemm_pp<IB, JB, 3, 2>::row_of(r, q, f); }

  template <class WBase, class WOff, class XBase, class XOff>
  __device__ static __forceinline__ void mainloop(f32x4 (&acc)[IB][JB], unsigned char *lds, int n_slabs, WBase w_base, WOff w_off, XBase x_base,
                                                  XOff x_off) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, lg = lane >> 4;
    const int grp = wave >> 2, wn = wave & 3;
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds;
#pragma unroll
    for (int i = 0; i < IB; ++i)
#pragma unroll
      for (int j = 0; j < JB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    constexpr int kLW = BM / 64;                                        // loads 0 .. kLW - 1 of a wave: weights
    uint32_t src[kLoads];
    const char *base[kLoads];
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      const int r0 = 8 * (8 * j + wave), r = r0 + (lane >> 3);
      const uint32_t piece = 16 * ((lane & 7) ^ ((r >> 1) & 7));
      if (j < kLW) { base[j] = w_base(r0); src[j] = w_off(r) + piece; }
      else { base[j] = x_base(r0 - BM); src[j] = x_off(r - BM) + piece; }
    }
#define A3_PL_LOAD(J, STAGE, SLAB)                                                                                      \
  {                                                                                                                     \
    const char *gb_ = base[J] + (size_t)min((SLAB), n_slabs - 1) * 128;      /* past the end: the last slab, unused */    \
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"                                         \
                 :: "s"(lds_base + (uint32_t)(STAGE) + (8 * (J) + wave) * 1024), "v"(src[J]), "s"(gb_) : "memory");      \
  }
#define A3_PL_FENCE __builtin_amdgcn_sched_barrier(0);
    const int swz = (l16 >> 1) & 7;
    const int frag_w = (grp * 16 * IB + l16) * 128, frag_x = (BM + wn * 16 * JB + l16) * 128;
    const int slot0 = (lg ^ swz) * 16, slot1 = ((4 + lg) ^ swz) * 16;
    constexpr int kM = 2 * IB * JB, kR = 2 * (IB + JB);
    // read n of a slab: per k-step the activation fragments, then the weights
#define A3_PL_READ(N, W, X, ST0)                                                                                        \
  {                                                                                                                     \
    const int ks_ = (N) / (IB + JB), i_ = (N) % (IB + JB);                                                              \
    const unsigned char *p_ = lds + (ST0) + (ks_ ? slot1 : slot0);                                                      \
    if (i_ < JB) X[ks_][i_] = *reinterpret_cast<const bf16x8 *>(p_ + frag_x + i_ * 2048);                               \
    else W[ks_][i_ - JB] = *reinterpret_cast<const bf16x8 *>(p_ + frag_w + (i_ - JB) * 2048);                           \
  }
    bf16x8 wa[2][IB], xa[2][JB], wb[2][IB], xb[2][JB];
    int rd = kStage, ld = 0;                                            // stage of slab s + 1, stage of slab s
    auto slab = [&](int s, bf16x8(&wc)[2][IB], bf16x8(&xc)[2][JB], bf16x8(&wx)[2][IB], bf16x8(&xx)[2][JB]) {
      // slab s + 1 has landed (behind it only ST - 2 slabs may be on their way), everybody's fragments of slab s are in
      // registers: its stage is free for slab s + ST
      __builtin_amdgcn_s_waitcnt(vmcnt_imm((ST - 2) * kLoads) & ~(15 << 8));
      __builtin_amdgcn_s_barrier();
      A3_PL_FENCE
#pragma unroll
      for (int m = 0; m < kM; ++m) {
        const int ks = m / (IB * JB), i = (m / JB) % IB, j = m % JB;
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wc[ks][i], xc[ks][j], acc[i][j], 0, 0, 0);
        A3_PL_FENCE
#pragma unroll
        for (int n = m * kR / kM; n < (m + 1) * kR / kM; ++n) A3_PL_READ(n, wx, xx, rd)
#pragma unroll
        for (int l = m * kLoads / kM; l < (m + 1) * kLoads / kM; ++l) A3_PL_LOAD(l, ld, s + ST)
        A3_PL_FENCE
      }
      ld = rd;
      rd = rd == (ST - 1) * kStage ? 0 : rd + kStage;
    };
#pragma unroll
    for (int s = 0; s < ST; ++s)
#pragma unroll
      for (int j = 0; j < kLoads; ++j) A3_PL_LOAD(j, s * kStage, s)
    __builtin_amdgcn_s_waitcnt(vmcnt_imm((ST - 1) * kLoads));
    __builtin_amdgcn_s_barrier();
    A3_PL_FENCE
#pragma unroll
    for (int n = 0; n < kR; ++n) A3_PL_READ(n, wa, xa, 0)
    A3_PL_FENCE
    for (int s = 0;; s += 2) {
      slab(s, wa, xa, wb, xb);
      if (s + 1 >= n_slabs) break;
      slab(s + 1, wb, xb, wa, xa);
      if (s + 2 >= n_slabs) break;
    }
#undef A3_PL_READ
#undef A3_PL_FENCE
#undef A3_PL_LOAD
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));                           // the tail loads have landed before LDS is released
  }
};

// ---- the tile as a type (which one: a3_gemm_tiles.h) -----------------------------------------------------
template <class F>
static inline a3_status gemm_with_tile(int tile, F f) {
  switch (tile) {
    case GEMM_256x256: return f(gemm_pp<8, 4, 3, 2>{});
    case GEMM_256x192: return f(gemm_pp<8, 3, 3, 2>{});
    case GEMM_256x128: return f(gemm_pl<8, 2, 3>{});
    case GEMM_128x192: return f(gemm_pl<4, 3, 4>{});
    case GEMM_128x128: return f(gemm_pl<4, 2, 5>{});
    default: return f(gemm_pl<4, 1, 6>{});
  }
}

}  // namespace
