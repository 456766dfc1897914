// Step 4 (projection part) of the A^3 fusion path: Q/K/V of the listed rows, Eq. 5 first lines.
//
//   Q = RoPE_p(x Wq^T + bq),  K = RoPE_p(x Wk^T + bk),  V = x Wv^T + bv        p = position of the row
//
// bf16: a row-gathering MFMA GEMM (main loop: a3_gemm_pp.h), the weights as the MFMA "row" operand and the gathered
// hidden rows as the "column" operand.  Both RoPE pairings (adjacent coordinates, or i with i + 64) end up lane-local
// and the rotation runs in the epilogue on the fp32 accumulators, before the single rounding to bf16.
// fp32: the fp32 matrix instruction on fragments straight from memory.
#include <stdlib.h>

#include "a3_internal.h"
#include "a3_gemm_pp.h"

namespace {

// ---------------------------------------------------------------------------------------
// bf16 MFMA kernel
// ---------------------------------------------------------------------------------------
constexpr int kHeadDim = 128;
struct proj_args {
  const bf16_t *hidden;
  const int *row_idx;
  int n_rows;
  const bf16_t *w[3];
  const bf16_t *bias[3];
  bf16_t *out[3];
  const int *tok_pos;
  const float2 *pos_cs;
  int K, Hq, Hkv, rope_layout;
  int n_heads, n_wtiles, n_tok_tiles, group;
  int scatter_kv;        // K and V go to row row_idx[i] of their output (the caches) instead of row i
};

struct head_sel { int which, head, heads_out; };

__device__ __forceinline__ head_sel select_head(int h, int Hq, int Hkv) {
  head_sel r;
  if (h < Hq) { r.which = 0; r.head = h; r.heads_out = Hq; }
  else if (h < Hq + Hkv) { r.which = 1; r.head = h - Hq; r.heads_out = Hkv; }
  else { r.which = 2; r.head = h - Hq - Hkv; r.heads_out = Hkv; }
  return r;
}

// The heads that have an output, in the order Q, K, V (a Q-only or K/V-only call has fewer tiles, not idle ones).
__device__ __forceinline__ head_sel active_head(const proj_args &a, int i) {
  head_sel r;
  r.which = 0; r.head = i; r.heads_out = a.Hq;
  const int n0 = a.out[0] ? a.Hq : 0, n1 = a.out[1] ? a.Hkv : 0;
  if (i >= n0) { r.which = 1; r.head = i - n0; r.heads_out = a.Hkv; }
  if (i >= n0 + n1) { r.which = 2; r.head = i - n0 - n1; }
  return r;
}

// IB = 8: a workgroup holds two heads, one per wave group; IB = 4: one head, group g its features 32 g .. and 64 + 32 g ..
template <class P>
__global__ void __launch_bounds__(512)
proj_bf16_kernel(proj_args a) {
  constexpr int IB = P::kIB, JB = P::kJB;
  extern __shared__ __align__(16) unsigned char lds[];
  int wt, xt;
  if (!gemm_tile_of(a.n_wtiles, a.n_tok_tiles, a.group, blockIdx.x, wt, xt)) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, lg = lane >> 4, grp = wave >> 2, wn = wave & 3;
  constexpr int kHeadsWg = IB == 8 ? 2 : 1;

  f32x4 acc[IB][JB];
  P::mainloop(
      acc, lds, a.K / 64,
      [&](int r0) -> const char * {                              // (an odd last head is computed twice, stored once)
        const head_sel hs = active_head(a, min(kHeadsWg * wt + (IB == 8 ? r0 >> 7 : 0), a.n_heads - 1));
        return reinterpret_cast<const char *>(a.w[hs.which] + (size_t)hs.head * kHeadDim * a.K);
      },
      [&](int r) -> uint32_t {
        int q, f;
        P::row_of(r % (16 * IB), q, f);
        return (uint32_t)(64 * q + f + (IB == 4 ? 32 * (r / 64) : 0)) * (uint32_t)a.K * 2u;
      },
      [&](int) -> const char * { return reinterpret_cast<const char *>(a.hidden); },
      [&](int r) -> uint32_t {
        const int m = min(xt * P::BN + r, a.n_rows - 1);         // clamp: computed but never stored
        return (uint32_t)(a.row_idx ? a.row_idx[m] : m) * (uint32_t)a.K * 2u;
      });

  // ---- epilogue: bias, RoPE, one rounding, store ---------------------------------------------------------
  // A lane holds, of one row, L consecutive features of the head's first half and the L of its second half that belong to
  // the same lanes: both RoPE pairings are inside the lane, and four lanes cover 64 or 128 consecutive bytes of a row.
  const int hi_idx = kHeadsWg * wt + (IB == 8 ? grp : 0);
  if (hi_idx >= a.n_heads) return;
  const head_sel hs = active_head(a, hi_idx);
  constexpr int L = P::L;
  const int f0 = L * lg + (IB == 4 ? 32 * grp : 0);              // lo: features f0 .. f0 + L - 1, hi: 64 + the same
  const bool inter = a.rope_layout == A3_ROPE_INTERLEAVED, rope = hs.which != 2;
  bf16_t *__restrict__ out = a.out[hs.which];
  const bf16_t *bias = a.bias[hs.which];
  int tok[JB], src[JB], pos[JB];
#pragma unroll
  for (int j = 0; j < JB; ++j) {
    tok[j] = xt * P::BN + 16 * (JB * wn + j) + l16;
    const int m = min(tok[j], a.n_rows - 1);
    src[j] = a.row_idx ? a.row_idx[m] : m;
  }
#pragma unroll
  for (int j = 0; j < JB; ++j) pos[j] = rope ? a.tok_pos[src[j]] : 0;
#pragma unroll
  for (int j = 0; j < JB; ++j) {
    float lo[L], hi[L];
    // table entries p of the row: interleaved pairs f0 / 2 .. (lo) and 32 + f0 / 2 .. (hi), halves f0 .. f0 + L - 1
    const float4 *cs = reinterpret_cast<const float4 *>(a.pos_cs + (size_t)pos[j] * (kHeadDim / 2));
    float4 t[L / 2];
    if (rope) {
#pragma unroll
      for (int e = 0; e < L / 4; ++e) {
        t[e] = cs[inter ? f0 / 4 + e : f0 / 2 + e];
        t[L / 4 + e] = cs[inter ? 16 + f0 / 4 + e : f0 / 2 + L / 4 + e];
      }
    }
    gemm_lane_values<IB, JB>(acc, j, lo, hi);
    if (bias) {
#pragma unroll
      for (int e = 0; e < L; ++e) {
        lo[e] += a3_bf2f(bias[hs.head * kHeadDim + f0 + e]);
        hi[e] += a3_bf2f(bias[hs.head * kHeadDim + 64 + f0 + e]);
      }
    }
    if (rope) {
      if (inter) {
#pragma unroll
        for (int e = 0; e < L / 4; ++e)
#pragma unroll
          for (int u = 0; u < 4; u += 2) {
            const float c0 = u ? t[e].z : t[e].x, s0 = u ? t[e].w : t[e].y;
            const float c1 = u ? t[L / 4 + e].z : t[L / 4 + e].x, s1 = u ? t[L / 4 + e].w : t[L / 4 + e].y;
            const float x0 = lo[4 * e + u], x1 = lo[4 * e + u + 1], y0 = hi[4 * e + u], y1 = hi[4 * e + u + 1];
            lo[4 * e + u] = x0 * c0 - x1 * s0; lo[4 * e + u + 1] = x0 * s0 + x1 * c0;
            hi[4 * e + u] = y0 * c1 - y1 * s1; hi[4 * e + u + 1] = y0 * s1 + y1 * c1;
          }
      } else {
#pragma unroll
        for (int e = 0; e < L; ++e) {
          const float c = (e & 1) ? t[e / 2].z : t[e / 2].x, sn = (e & 1) ? t[e / 2].w : t[e / 2].y;
          const float x = lo[e], y = hi[e];
          lo[e] = x * c - y * sn;
          hi[e] = x * sn + y * c;
        }
      }
    }
    if (tok[j] < a.n_rows) {
      const int out_row = (a.scatter_kv && hs.which != 0) ? src[j] : tok[j];
      bf16_t *p = out + ((size_t)out_row * hs.heads_out + hs.head) * kHeadDim + f0;
#pragma unroll
      for (int e = 0; e < L; e += 8) {
        bf16x8 vl, vh;
#pragma unroll
        for (int u = 0; u < 8; ++u) { vl[u] = a3_f2bf(lo[e + u]); vh[u] = a3_f2bf(hi[e + u]); }
        *reinterpret_cast<bf16x8 *>(p + e) = vl;
        *reinterpret_cast<bf16x8 *>(p + 64 + e) = vh;
      }
    }
  }
}

// ---------------------------------------------------------------------------------------
// bf16 kernels for few rows (the question tokens): weight-streaming bound
// ---------------------------------------------------------------------------------------
// Last step of both few-row kernels for one lane = one listed row: adds the NW partial tiles in wave
// order (partial w of accumulator register r is part[w * wave_stride + r * 64]), then bias, RoPE
// and the single rounding.  A workgroup holds 32 features of one head: 16 sb + (0..15) and the same
// + 64, so both RoPE pairings are inside it; accumulator register r is MFMA row
// i = 8 (r/4) + 4 lhi + r%4, and i < 16 is the first half of the head, i >= 16 the second.
template <int NW>
__device__ __forceinline__ void small_finish(const proj_args &a, const head_sel hs, int sb, int tok, int lhi,
                                             const float *part, int wave_stride) {
  if (tok >= a.n_rows) return;
  float v[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) t += part[w * wave_stride + r * 64];   // fixed order
    v[r] = t;
  }
  auto feat_of = [&](int r) {
    int i = 8 * (r >> 2) + 4 * lhi + (r & 3);
    return i < 16 ? 16 * sb + i : 64 + 16 * sb + (i - 16);
  };
  const bf16_t *bias = a.bias[hs.which];
  if (bias) {
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] += a3_bf2f(bias[hs.head * kHeadDim + feat_of(r)]);
  }
  const int src_row = a.row_idx ? a.row_idx[tok] : tok;
  if (hs.which != 2) {
    const float2 *cs = a.pos_cs + (size_t)a.tok_pos[src_row] * (kHeadDim / 2);
    if (a.rope_layout == A3_ROPE_INTERLEAVED) {
#pragma unroll
      for (int r = 0; r < 16; r += 2) {
        const float2 t = cs[feat_of(r) >> 1];
        float x0 = v[r], x1 = v[r + 1];
        v[r] = x0 * t.x - x1 * t.y;
        v[r + 1] = x0 * t.y + x1 * t.x;
      }
    } else {
#pragma unroll
      for (int r = 0; r < 8; ++r) {                            // register r + 8 holds feature + 64
        const float2 t = cs[feat_of(r)];
        float xlo = v[r], xhi = v[r + 8];
        v[r] = xlo * t.x - xhi * t.y;
        v[r + 8] = xlo * t.y + xhi * t.x;
      }
    }
  }
  const int out_row = (a.scatter_kv && hs.which != 0) ? src_row : tok;
  bf16_t *orow = a.out[hs.which] + ((size_t)out_row * hs.heads_out + hs.head) * kHeadDim;
#pragma unroll
  for (int q4 = 0; q4 < 4; ++q4) {
    bf16x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = a3_f2bf(v[4 * q4 + e]);
    *reinterpret_cast<bf16x4 *>(orow + feat_of(4 * q4)) = o;
  }
}

// Hidden size a multiple of 256.  With ~64 rows the GEMM is a stream over the 48 MB of weights.  To
// put every CU on that stream a workgroup takes only 32 features of one head x 64 rows, and its 4
// waves split the reduction dimension four ways.  Each wave runs its own pipeline with no workgroup
// barrier: stages of 64 reduction elements (32 weight rows + 64 hidden rows, 128 bytes each) go
// from global memory straight into the wave's private ring of three LDS stages with fully coalesced
// direct-to-LDS loads (8 lanes per 128-byte row), two stages ahead of the MFMAs.  (Fragments loaded
// straight into registers would touch 32 different cache lines per instruction, and the address
// path of the L1, not HBM, then sets the pace.)  LDS slot s of row r holds the 16-byte piece
// s ^ ((r/2) % 8) of the row's 128 bytes: the 16 consecutive rows a quarter wave reads at one piece
// index touch all 64 banks once.
// RB = row blocks of 32 per workgroup: 2 (64 rows), or 1 when that leaves more than half of the CUs without a
// workgroup (a call with few heads: Q of the question rows alone): twice the workgroups, each re-reading half as
// many hidden rows.
constexpr int kSmRing = 3;
constexpr int sm_stage_bytes(int rb) { return (32 + 32 * rb) * 128; }
constexpr size_t sm_lds_bytes(int rb) { return (size_t)4 * kSmRing * sm_stage_bytes(rb); }      // 144 KB / 96 KB

template <int RB>
__global__ void __launch_bounds__(256)
proj_small_dma_bf16_kernel(proj_args a) {
  constexpr int kSmStageBytes = sm_stage_bytes(RB);
  constexpr int kSmLoads = 4 + 4 * RB;                         // direct-to-LDS loads per stage
  extern __shared__ __align__(16) unsigned char lds[];

  const int head_all = blockIdx.x >> 2, sb = blockIdx.x & 3;
  const head_sel hs = select_head(head_all, a.Hq, a.Hkv);
  if (a.out[hs.which] == nullptr) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, lhi = lane >> 5;
  const int tok0 = blockIdx.y * 32 * RB;
  const int kq = a.K / 4;                                      // this wave's share: a multiple of 64

  // loading role: one instruction brings 8 rows x 128 B, lane -> (row lane/8, slot lane%8)
  const int drow = lane >> 3, dslot = lane & 7;
  const char *wsrc[4], *xsrc[4 * RB];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int row = 8 * j + drow;                              // MFMA row of the weight block
    const int feat = row < 16 ? 16 * sb + row : 64 + 16 * sb + (row - 16);
    wsrc[j] = reinterpret_cast<const char *>(a.w[hs.which] + ((size_t)hs.head * kHeadDim + feat) * a.K + wave * kq) +
              16 * (dslot ^ ((row >> 1) & 7));
  }
#pragma unroll
  for (int j = 0; j < 4 * RB; ++j) {
    const int row = 8 * j + drow;
    const int m = min(tok0 + row, a.n_rows - 1);               // clamp: computed but never stored
    const int src_row = a.row_idx ? a.row_idx[m] : m;
    xsrc[j] = reinterpret_cast<const char *>(a.hidden + (size_t)src_row * a.K + wave * kq) +
              16 * (dslot ^ ((row >> 1) & 7));
  }
  unsigned char *ring = lds + wave * (kSmRing * kSmStageBytes);
  const uint32_t lds_ring = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)ring;
  // Inline assembly as in the large kernel: lane i's 16 bytes land at M0 + 16 i, the compiler does not
  // track these loads, and the waits for them are the explicit s_waitcnt below.
#define A3_SM_ISSUE(SLOT, K0)                                                                                  \
  {                                                                                                            \
    _Pragma("unroll") for (int j = 0; j < 4; ++j)                                                              \
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"                                       \
                   :: "s"(__builtin_amdgcn_readfirstlane(lds_ring + (SLOT) * kSmStageBytes + 1024 * j)),       \
                      "v"(wsrc[j] + 2 * (K0)) : "memory");                                                     \
    _Pragma("unroll") for (int j = 0; j < 4 * RB; ++j)                                                         \
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"                                       \
                   :: "s"(__builtin_amdgcn_readfirstlane(lds_ring + (SLOT) * kSmStageBytes + 4096 + 1024 * j)), \
                      "v"(xsrc[j] + 2 * (K0)) : "memory");                                                     \
  }
  f32x16 acc[RB];
#pragma unroll
  for (int tb = 0; tb < RB; ++tb)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[tb][r] = 0.f;
  // everything the compiler loaded itself (row indices) has arrived: from here on only the
  // direct-to-LDS loads are outstanding and the counts below are exact
  __builtin_amdgcn_s_waitcnt(0);
  const int n_st = kq / 64;
  A3_SM_ISSUE(0, 0)
  if (n_st > 1) A3_SM_ISSUE(1, 64)
  const int frag = l32 * 128, fswz = (l32 >> 1) & 7;           // rows 32 tb + l32 swizzle like row l32
  int slot = 0, slot2 = 2;
  for (int s = 0; s < n_st; ++s) {
    if (s + 2 < n_st) {
      A3_SM_ISSUE(slot2, 64 * (s + 2))
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * kSmLoads));     // stage s has landed: two younger ones may be on their way
    } else if (s + 1 < n_st) {
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(kSmLoads));
    } else {
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    }
    asm volatile("" ::: "memory");
    const unsigned char *st = ring + slot * kSmStageBytes + frag;
    bf16x8 wf[4], xa[4], xb[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int po = 16 * ((2 * u + lhi) ^ fswz);
      wf[u] = *reinterpret_cast<const bf16x8 *>(st + po);
      xa[u] = *reinterpret_cast<const bf16x8 *>(st + 4096 + po);
      if (RB == 2) xb[u] = *reinterpret_cast<const bf16x8 *>(st + 8192 + po);
    }
    __builtin_amdgcn_sched_barrier(0);                         // all twelve reads in flight before the first MFMA
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[u], xa[u], acc[0], 0, 0, 0);
      if (RB == 2) acc[RB - 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[u], xb[u], acc[RB - 1], 0, 0, 0);
    }
    // the fragments are in registers before the next trip overwrites the slot read two trips ago
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    slot = slot == kSmRing - 1 ? 0 : slot + 1;
    slot2 = slot2 == kSmRing - 1 ? 0 : slot2 + 1;
  }
#undef A3_SM_ISSUE
  // the wave's own ring is free now: it holds the wave's partial tile, [row block][register][lane]
  float *red = reinterpret_cast<float *>(ring);
#pragma unroll
  for (int tb = 0; tb < RB; ++tb)
#pragma unroll
    for (int r = 0; r < 16; ++r) red[(tb * 16 + r) * 64 + lane] = acc[tb][r];
  __syncthreads();
  if (wave >= RB) return;
  const int tb = wave;                                         // one wave per row block finishes it
  small_finish<4>(a, hs, sb, tok0 + tb * 32 + l32, lhi, reinterpret_cast<const float *>(lds) + tb * 16 * 64 + lane,
                  kSmRing * kSmStageBytes / 4);
}

// Any other hidden size that is a multiple of 64: fragments straight from global memory.
// A workgroup takes 32 features of one head (16 from each half of the head, so both RoPE
// pairings stay inside it) x 64 rows, and its NW waves (2 when the hidden size is a multiple of
// 128, else 1) split the reduction dimension NW ways in shares of whole 64-wide stages; fragments
// are read straight from global memory and the partial tiles are added in LDS in wave order.
template <int NW>                                               // waves per workgroup = ways the reduction is split
__global__ void __launch_bounds__(64 * NW)
proj_small_bf16_kernel(proj_args a) {
  __shared__ float red[NW][2][16][64];                         // [wave][row block][register][lane]

  const int head_all = blockIdx.x >> 2, sb = blockIdx.x & 3;
  const head_sel hs = select_head(head_all, a.Hq, a.Hkv);
  bf16_t *__restrict__ out = a.out[hs.which];
  if (out == nullptr) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, lhi = lane >> 5;
  const int tok0 = blockIdx.y * 64;
  // MFMA row i of this workgroup's weight block <-> feature of the head
  const int feat = l32 < 16 ? 16 * sb + l32 : 64 + 16 * sb + (l32 - 16);
  const int kq = a.K / NW;                                     // this wave's share of the reduction
  const bf16_t *wp = a.w[hs.which] + ((size_t)hs.head * kHeadDim + feat) * a.K + wave * kq + lhi * 8;
  const bf16_t *xp0, *xp1;
  {
    int m = min(tok0 + l32, a.n_rows - 1);
    xp0 = a.hidden + (size_t)(a.row_idx ? a.row_idx[m] : m) * a.K + wave * kq + lhi * 8;
    m = min(tok0 + 32 + l32, a.n_rows - 1);
    xp1 = a.hidden + (size_t)(a.row_idx ? a.row_idx[m] : m) * a.K + wave * kq + lhi * 8;
  }
  f32x16 acc[2];
#pragma unroll
  for (int tb = 0; tb < 2; ++tb)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[tb][r] = 0.f;
  // Two register stages of four k-steps each: the loads of one stage are in flight while the other
  // is multiplied, so every wave always has weight bytes on their way from HBM.  The share kq is a
  // multiple of 64 (one stage).
  bf16x8 wf0[4], wf1[4], xa0[4], xa1[4], xb0[4], xb1[4];
#define A3_SMALL_LOAD(WF, XA, XB, K0)                                            \
  _Pragma("unroll") for (int u = 0; u < 4; ++u) {                                \
    WF[u] = *reinterpret_cast<const bf16x8 *>(wp + (K0) + 16 * u);               \
    XA[u] = *reinterpret_cast<const bf16x8 *>(xp0 + (K0) + 16 * u);              \
    XB[u] = *reinterpret_cast<const bf16x8 *>(xp1 + (K0) + 16 * u);              \
  }
#define A3_SMALL_MMA(WF, XA, XB)                                                 \
  _Pragma("unroll") for (int u = 0; u < 4; ++u) {                                \
    acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(WF[u], XA[u], acc[0], 0, 0, 0); \
    acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(WF[u], XB[u], acc[1], 0, 0, 0); \
  }
  A3_SMALL_LOAD(wf0, xa0, xb0, 0)
  int k = 0;
  for (; k + 128 <= kq; k += 128) {
    A3_SMALL_LOAD(wf1, xa1, xb1, k + 64)
    A3_SMALL_MMA(wf0, xa0, xb0)
    const int kn = min(k + 128, kq - 64);                      // past the end: the last stage again, unused
    A3_SMALL_LOAD(wf0, xa0, xb0, kn)
    A3_SMALL_MMA(wf1, xa1, xb1)
  }
  if (k < kq) { A3_SMALL_MMA(wf0, xa0, xb0) }                  // odd number of stages
#undef A3_SMALL_LOAD
#undef A3_SMALL_MMA
#pragma unroll
  for (int tb = 0; tb < 2; ++tb)
#pragma unroll
    for (int r = 0; r < 16; ++r) red[wave][tb][r][lane] = acc[tb][r];
  __syncthreads();
  if (wave >= 2) return;
  for (int tb = wave; tb < 2; tb += (NW > 1 ? 2 : 1))          // waves 0 and 1 finish one row block each
    small_finish<NW>(a, hs, sb, tok0 + tb * 32 + l32, lhi, &red[0][tb][0][lane], 2 * 16 * 64);
}

// ---------------------------------------------------------------------------------------
// fp32 kernel: 16 features of one head x 32 listed rows per workgroup, the four waves split the reduction
// ---------------------------------------------------------------------------------------
// fp32 matrix instruction (16x16x4), fragments straight from memory: a lane's 16-byte load holds four consecutive
// elements of one weight row or one hidden row, one for each of four instructions.  The 16 features are 8 of each half of
// the head (8 b .. and d / 2 + 8 b ..), so both RoPE pairings stay inside the workgroup.  Small calls are latency: every load
// of a wave's share is independent of the others.  (A tiled kernel with two barriers per 32 elements took 146 us for 32
// rows x 512 x 512; the new one 7.)
struct proj_args_f32 {
  const float *hidden;
  const int *row_idx;
  int n_rows;
  const float *w[3];
  const float *bias[3];
  float *out[3];
  const int *tok_pos;
  const float2 *pos_cs;
  int K, Hq, Hkv, d, rope_layout;
  int scatter_kv;
};

__global__ void __launch_bounds__(256)
proj_f32_kernel(proj_args_f32 a) {
  __shared__ float red[4][2][16][17];                          // [wave][row block][row][feature]
  const int per_head = a.d / 16, head_all = blockIdx.x / per_head, b = blockIdx.x % per_head;
  const head_sel hs = select_head(head_all, a.Hq, a.Hkv);
  float *__restrict__ out = a.out[hs.which];
  if (out == nullptr) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, lg = lane >> 4;
  const int d = a.d, half = d / 2, row0 = blockIdx.y * 32;
  const int feat = (l16 < 8 ? 0 : half - 8) + 8 * b + l16;     // MFMA row l16 of the weight block
  const f32x4 *wp = reinterpret_cast<const f32x4 *>(a.w[hs.which] + ((size_t)hs.head * d + feat) * a.K) + lg;
  const f32x4 *xp[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int m = min(row0 + 16 * j + l16, a.n_rows - 1);      // clamp: computed but never stored
    xp[j] = reinterpret_cast<const f32x4 *>(a.hidden + (size_t)(a.row_idx ? a.row_idx[m] : m) * a.K) + lg;
  }
  // 16-element chunks of the reduction: wave w takes chunks w, w + 4, ..., four at a time
  const int chunks = a.K / 16;
  f32x4 acc[2][2] = {};                                        // [row block][parity of the chunk]: two chains each
  for (int c0 = wave; c0 < chunks; c0 += 16) {
    f32x4 wf[4], xf[2][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = c0 + 4 * u;
      const bool on = c < chunks;
      wf[u] = on ? wp[4 * c] : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < 2; ++j) xf[j][u] = on ? xp[j][4 * c] : f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[j][u & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[u][e], xf[j][u][e], acc[j][u & 1], 0, 0, 0);
  }
  // register r of lane (l16, lg): feature 4 lg + r of the block, row l16
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wave][j][l16][4 * lg + r] = acc[j][0][r] + acc[j][1][r];
  __syncthreads();
  // one pair of coordinates of one row per thread: features 8 b + .. of the first half with those of the second (halves), or
  // neighbours of either half (interleaved)
  const int i = tid >> 3, q = tid & 7, tok = row0 + i;
  if (tok >= a.n_rows) return;
  const bool inter = a.rope_layout == A3_ROPE_INTERLEAVED;
  const int fa = inter ? 2 * q : q, fb = inter ? 2 * q + 1 : q + 8;              // MFMA rows of the pair
  float xa = 0.f, xb = 0.f;
#pragma unroll
  for (int w = 0; w < 4; ++w) { xa += red[w][i >> 4][i & 15][fa]; xb += red[w][i >> 4][i & 15][fb]; }
  const int ca = (fa < 8 ? 0 : half - 8) + 8 * b + fa, cb = (fb < 8 ? 0 : half - 8) + 8 * b + fb;   // coordinates in the head
  const float *bias = a.bias[hs.which];
  if (bias) { xa += bias[hs.head * d + ca]; xb += bias[hs.head * d + cb]; }
  const int src = a.row_idx ? a.row_idx[tok] : tok;
  if (hs.which != 2) {
    const float2 t = a.pos_cs[(size_t)a.tok_pos[src] * half + (inter ? ca / 2 : ca)];
    const float ya = xa * t.x - xb * t.y;
    xb = xa * t.y + xb * t.x;
    xa = ya;
  }
  float *orow = out + ((size_t)((a.scatter_kv && hs.which != 0) ? src : tok) * hs.heads_out + hs.head) * d;
  orow[ca] = xa;
  orow[cb] = xb;
}

}  // namespace

static a3_status proj_launch(const a3_layout *L, const void *hidden, const int *row_idx, int n_rows, const void *wq,
                             const void *wk, const void *wv, const void *bq, const void *bk, const void *bv,
                             void *q_out, void *k_out, void *v_out, int scatter_kv, void *stream) {
  a3_status s = a3_check_layout(L, "a3_selected_qkv_proj", true);
  if (s != A3_OK) return s;
  A3_REQUIRE(n_rows >= 0 && n_rows <= L->total_tokens, A3_ERR_INVALID_ARG,
             "a3_selected_qkv_proj: n_rows %d outside [0, %d]", n_rows, L->total_tokens);
  if (n_rows == 0 || (!q_out && !k_out && !v_out)) return A3_OK;
  A3_REQUIRE(hidden, A3_ERR_INVALID_ARG, "a3_selected_qkv_proj: hidden is NULL");
  A3_REQUIRE((!q_out || wq) && (!k_out || wk) && (!v_out || wv), A3_ERR_INVALID_ARG,
             "a3_selected_qkv_proj: an output is requested without its weight");
  const void *ptrs[] = {hidden, wq, wk, wv, bq, bk, bv, q_out, k_out, v_out};
  for (const void *p : ptrs)
    A3_REQUIRE(a3_aligned16(p), A3_ERR_INVALID_ARG, "a3_selected_qkv_proj: tensors must be 16-byte aligned");
  hipStream_t st = (hipStream_t)stream;
  const int n_heads_total = L->n_q_heads + 2 * L->n_kv_heads;
  if (L->dtype == A3_BF16) {
    A3_REQUIRE(L->hidden % 64 == 0, A3_ERR_UNSUPPORTED, "a3_selected_qkv_proj: bf16 needs hidden %% 64 == 0, got %d",
               L->hidden);
    A3_REQUIRE((long long)L->total_tokens * L->hidden * 2 < (1LL << 32), A3_ERR_UNSUPPORTED,
               "a3_selected_qkv_proj: hidden tensor larger than 4 GiB");
    proj_args a;
    a.hidden = (const bf16_t *)hidden; a.row_idx = row_idx; a.n_rows = n_rows;
    a.w[0] = (const bf16_t *)wq; a.w[1] = (const bf16_t *)wk; a.w[2] = (const bf16_t *)wv;
    a.bias[0] = (const bf16_t *)bq; a.bias[1] = (const bf16_t *)bk; a.bias[2] = (const bf16_t *)bv;
    a.out[0] = (bf16_t *)q_out; a.out[1] = (bf16_t *)k_out; a.out[2] = (bf16_t *)v_out;
    a.tok_pos = L->tok_pos; a.pos_cs = (const float2 *)L->rope_pos_cs;
    a.K = L->hidden; a.Hq = L->n_q_heads; a.Hkv = L->n_kv_heads; a.rope_layout = L->rope_layout;
    a.n_heads = n_heads_total;
    a.n_wtiles = a.n_tok_tiles = a.group = 0;
    a.scatter_kv = scatter_kv;
    const int ntw_knob = a3_knob(A3_KNOB_PROJ_NTW);            // tuning value "proj_ntw": the GEMM kernel in this width
    if (n_rows <= 192 && L->hidden % 64 == 0 && ntw_knob < 0) {
      // few rows: stream the weights with 4 x n_heads x ceil(rows/64) small workgroups.  Weights from HBM, this against the GEMM
      // in its best tile: Q, K, V of 6144 x 4096 at 64 rows 17.9 and 32.9 us, 128 rows 27.1 and 32.1, 160 rows 34.7 and 29.5, 192 rows
      // 36.9 and 31.9; of 4608 x 3584 at 192 rows 22.2 and 27.8; Q alone at 192 rows 23.2 and 29.2, 20.7 and 19.1; K and V alone 11.9
      // and 20.0, 8.8 and 18.1.  192 is the line that serves all but the widest call.
      const dim3 grid(4 * n_heads_total, (n_rows + 63) / 64);
      if (L->hidden % 256 == 0) {
        static a3_once_per_device small_once;
        const hipError_t once_err = a3_once(small_once, []() {
          hipError_t e = hipFuncSetAttribute((const void *)proj_small_dma_bf16_kernel<2>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm_lds_bytes(2));
          hipError_t e1 = hipFuncSetAttribute((const void *)proj_small_dma_bf16_kernel<1>,
                                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm_lds_bytes(1));
          return e != hipSuccess ? e : e1;
        });
        if (once_err != hipSuccess) return a3_fail(A3_ERR_HIP, "a3_selected_qkv_proj: cannot raise the dynamic LDS limit");
        // workgroups that have an output: 4 per head of the tensors asked for, per 64 rows
        const int heads_out = (q_out ? L->n_q_heads : 0) + (k_out ? L->n_kv_heads : 0) + (v_out ? L->n_kv_heads : 0);
        if (4 * heads_out * (int)grid.y <= 128 && n_rows > 32)
          hipLaunchKernelGGL(proj_small_dma_bf16_kernel<1>, dim3(grid.x, (n_rows + 31) / 32), dim3(256), sm_lds_bytes(1), st, a);
        else
          hipLaunchKernelGGL(proj_small_dma_bf16_kernel<2>, grid, dim3(256), sm_lds_bytes(2), st, a);
      } else if (L->hidden % 128 == 0) {
        hipLaunchKernelGGL(proj_small_bf16_kernel<2>, grid, dim3(128), 0, st, a);
      } else {
        hipLaunchKernelGGL(proj_small_bf16_kernel<1>, grid, dim3(64), 0, st, a);
      }
      A3_CHECK_LAUNCH("a3_selected_qkv_proj");
      return A3_OK;
    }
    const int heads_out = (q_out ? L->n_q_heads : 0) + (k_out ? L->n_kv_heads : 0) + (v_out ? L->n_kv_heads : 0);
    a.n_heads = heads_out;
    gemm_tile_choice c = gemm_choose_tile(heads_out * kHeadDim, n_rows, L->hidden / 64, 1);
    if (gemm_tile_of_knob(ntw_knob) >= 0) c.tile = gemm_tile_of_knob(ntw_knob);
    return gemm_with_tile(c.tile, [&](auto t) -> a3_status {
      using P = decltype(t);
      auto kern = proj_bf16_kernel<P>;
      static a3_once_per_device lds_once;
      if (a3_once(lds_once, [&]() { return hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)P::kLdsBytes); }) != hipSuccess)
        return a3_fail(A3_ERR_HIP, "a3_selected_qkv_proj: cannot raise the dynamic LDS limit");
      proj_args b = a;
      b.n_wtiles = P::kIB == 8 ? (heads_out + 1) / 2 : heads_out;
      b.n_tok_tiles = (n_rows + P::BN - 1) / P::BN;
      b.group = gemm_tile_group(b.n_wtiles, b.n_tok_tiles);
      hipLaunchKernelGGL(kern, dim3(gemm_tile_grid(b.n_wtiles, b.n_tok_tiles)), dim3(512), P::kLdsBytes, st, b);
      A3_CHECK_LAUNCH("a3_selected_qkv_proj");
      return A3_OK;
    });
  } else {
    proj_args_f32 a;
    a.hidden = (const float *)hidden; a.row_idx = row_idx; a.n_rows = n_rows;
    a.w[0] = (const float *)wq; a.w[1] = (const float *)wk; a.w[2] = (const float *)wv;
    a.bias[0] = (const float *)bq; a.bias[1] = (const float *)bk; a.bias[2] = (const float *)bv;
    a.out[0] = (float *)q_out; a.out[1] = (float *)k_out; a.out[2] = (float *)v_out;
    a.tok_pos = L->tok_pos; a.pos_cs = (const float2 *)L->rope_pos_cs;
    a.K = L->hidden; a.Hq = L->n_q_heads; a.Hkv = L->n_kv_heads; a.d = L->head_dim; a.rope_layout = L->rope_layout;
    a.scatter_kv = scatter_kv;
    const dim3 grid(n_heads_total * (L->head_dim / 16), (n_rows + 31) / 32);
    hipLaunchKernelGGL(proj_f32_kernel, grid, dim3(256), 0, st, a);
  }
  A3_CHECK_LAUNCH("a3_selected_qkv_proj");
  return A3_OK;
}

extern "C" a3_status a3_selected_qkv_proj(const a3_layout *L, const void *hidden, const int *row_idx, int n_rows,
                                          const void *wq, const void *wk, const void *wv, const void *bq,
                                          const void *bk, const void *bv, void *q_out, void *k_out, void *v_out,
                                          void *stream) {
  return proj_launch(L, hidden, row_idx, n_rows, wq, wk, wv, bq, bk, bv, q_out, k_out, v_out, 0, stream);
}

extern "C" a3_status a3_selected_qkv_proj_scatter(const a3_layout *L, const void *hidden, const int *row_idx,
                                                  int n_rows, const void *wq, const void *wk, const void *wv,
                                                  const void *bq, const void *bk, const void *bv, void *q_out,
                                                  void *k_fused, void *v_fused, void *stream) {
  return proj_launch(L, hidden, row_idx, n_rows, wq, wk, wv, bq, bk, bv, q_out, k_fused, v_fused, 1, stream);
}
