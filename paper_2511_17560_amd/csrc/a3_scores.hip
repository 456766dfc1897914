// Step 2 of the A^3 fusion path: question-relevance score, Eq. 3 first line.
//
//   s_i = sum_{hq} sum_j softmax_i( q_{j,hq} . k'_{i, hq/G} * scale )      softmax over the context keys
//
// A column sum of row softmaxes needs every row's (max, sum exp) before any column can be
// summed, so the logits are formed twice:
//   pass A   per (tile of keys, row): partial (max, sum exp)      -> workspace
//   pass B   per tile of keys: the partials of a row are merged (by the pass itself, or by a small kernel before it where there are
//            many), then sum over all rows of exp(l - max)/sum -> per KV head column sums
//   head sum per token: the KV heads in order                      -> scores
// Rows, then heads, are reduced in a fixed order, so the result is deterministic (no atomics).
//
// bf16: logits on the matrix cores (16x16x32 bf16 MFMA), a wave's keys in registers, the rows' Q through LDS.  exp2 with log2(e) folded
// into the scale.
// fp32: the same two passes on the fp32 matrix instruction.
#include <mutex>
#include <type_traits>

#include "a3_internal.h"

namespace {

constexpr float kLog2e = 1.4426950408889634f;
// Where a row's maximum starts.  The first keys that a lane, wave or tile sees may all have logits of -inf for a row, by their values or
// as masked question keys: the maximum is finite all the same, and their weights come out as exp2(-inf) = 0
constexpr float kLeast = -3.402823466e38f;

// log2(z 2^m), z > 0: the logarithm of a number in [1/2, 1), so that its error is small against the sum's rounding whatever z is
__device__ __forceinline__ float log2_sum(float m, float z) {
  const int e = __builtin_amdgcn_frexp_expf(z);
  return m + ((float)e + log2f(__builtin_amdgcn_frexp_mantf(z)));
}

// largest i in [0, n) with a[i] <= x (a ascending, a[0] <= x)
__device__ __forceinline__ int find_segment(const int *__restrict__ a, int n, int x) {
  int lo = 0, hi = n;
  while (lo < hi) {
    int mid = (lo + hi) >> 1;
    if (a[mid] <= x) lo = mid + 1; else hi = mid;
  }
  return lo - 1;
}

struct scores_args {
  const void *q;            // [sum q_len, Hq, d]
  const void *k;            // [T, Hkv, d]
  const int *seg_start, *ctx_len, *q_len, *q_start;
  float2 *part;             // fp32: [n_tiles + 1, total_rows] partial (max, sum) in the exp2 domain
  float *part_z, *part_m;   // bf16, in its place: [n_tiles + 1, total_rows] each, the sum z = sum exp2(l), or -z and the maximum that z
                            // is taken against
  float2 *stats;            // [total_rows] (max + log2(sum), unused): written by the combine kernel
  int merged;               // the combine kernel has run; otherwise the second pass merges the partials itself
  float *scores;            // [T]
  float *part_scores;       // [Hkv, T] bf16 path: per KV head partial scores
  int n_req, Hq, Hkv, d, T, total_rows, n_tiles, tile_keys;
  uint32_t inv_G;           // ceil(2^32 / G) for G > 1: m / G = umulhi(m, inv_G) for every m < 2^32 / G
  uint32_t inv_heads, inv_runs[2];   // the same for Hkv and the tiles of a request in either pass; 0: no such number, divide
  float scale2;             // sm_scale * log2(e)
  int one_ctx_len, one_q_len;   // a single request whose segment starts at row 0: its lengths; otherwise -1
  // fused position recovery (first pass): stale keys in, realigned keys out
  const void *k_cat;        // [T, Hkv, d] keys at chunk-local positions
  void *k_out;              // [T, Hkv, d] realigned keys (may be k_cat itself)
  const int *tok_chunk;     // [T] chunk of a context row, -1 for question rows
  const float2 *chunk_cs;   // [n_chunks, d/2] (cos, sin) of chunk offset x theta_i
  int rope_layout;
  // the softmax of a question token also runs over the question keys up to itself (their (max, sum) sits
  // in the extra partial slot n_tiles): the literal denominator of Eq. 3 and the window votes of the
  // eviction extension.  own_tile: bf16, that slot is written by a tile of the first pass
  int causal_q, own_tile;
};

// bf16: a partial (max, sum) as the sum alone, or minus the sum and the maximum
__device__ __forceinline__ void store_partial(float *pz, float *pm, size_t i, float m, float z) {
  pz[i] = m == 0.f || z == 0.f ? z : -z;
  if (m != 0.f && z != 0.f) pm[i] = m;
}

// ---------------------------------------------------------------------------------------
// (max, sum exp) of a question row over the question keys it sees (itself and the earlier ones of its
// request): one wave per (question token, query head), lanes over keys.  A few hundred short dot products.
// ---------------------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(256)
scores_question_stats_kernel(scores_args a) {
  const int lane = threadIdx.x & 63, row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= a.total_rows) return;
  const int jq = row / a.Hq, hq = row % a.Hq;
  const int r = find_segment(a.q_start, a.n_req, jq);
  const int j = jq - a.q_start[r];
  if (j >= a.q_len[r]) return;                                 // rows past the last request's question
  const int g = hq / (a.Hq / a.Hkv);
  const T *__restrict__ Q = (const T *)a.q + (size_t)row * a.d;
  const T *__restrict__ K = (const T *)a.k;
  const int key0 = a.seg_start[r] + a.ctx_len[r];
  float m = kLeast, z = 0.f;
  for (int u = lane; u <= j; u += 64) {
    // 16-byte loads of both rows (element by element this kernel took 28 us for 64 question tokens x 32 heads)
    constexpr int V = a3_elem<T>::kVec;
    typedef T vec_t __attribute__((ext_vector_type(V)));
    const vec_t *kp = reinterpret_cast<const vec_t *>(K + ((size_t)(key0 + u) * a.Hkv + g) * a.d);
    const vec_t *qp = reinterpret_cast<const vec_t *>(Q);
    float dot = 0.f;
#pragma unroll 8
    for (int c = 0; c < a.d / V; ++c) {
      const vec_t kv = kp[c], qv = qp[c];
#pragma unroll
      for (int e = 0; e < V; ++e) dot = fmaf((float)qv[e], (float)kv[e], dot);
    }
    const float l = dot * a.scale2;
    const float mn = fmaxf(m, l);
    z = z * exp2f(m - mn) + exp2f(l - mn);                     // first key: 0 * 0
    m = mn;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const float pm = __shfl_xor(m, off), pz = __shfl_xor(z, off);
    const float mn = fmaxf(m, pm);
    const float za = z > 0.f ? z * exp2f(m - mn) : 0.f, zb = pz > 0.f ? pz * exp2f(pm - mn) : 0.f;
    z = (lane & off) ? zb + za : za + zb;
    m = mn;
  }
  // (bf16: the rows of a KV head one after the other)
  const int G = a.Hq / a.Hkv, at = sizeof(T) == 2 ? (a.q_start[r]) * a.Hq + g * a.q_len[r] * G + j * G + hq - g * G : row;
  if (lane != 0) return;
  if constexpr (sizeof(T) == 2) store_partial(a.part_z, a.part_m, (size_t)a.n_tiles * a.total_rows + at, m, z);
  else a.part[(size_t)a.n_tiles * a.total_rows + at] = make_float2(m, z);
}

// ---------------------------------------------------------------------------------------
// combine partial row statistics (shared by both element types)
// ---------------------------------------------------------------------------------------
constexpr int kTileKeys = 64;      // fp32 kernels

template <bool BF16>
__global__ void __launch_bounds__(256)
scores_combine_kernel(scores_args a) {
  auto part = [&](int t, int row) {
    const size_t i = (size_t)t * a.total_rows + row;
    if constexpr (BF16) return make_float2(0.f, a.part_z[i]);
    else return a.part[i];
  };
  auto maximum = [&](int t, int row, float2 &p) {              // bf16: the maximum of a partial, looked up where there is one
    if constexpr (BF16) {
      p.x = p.y < 0.f ? a.part_m[(size_t)t * a.total_rows + row] : p.y > 0.f ? 0.f : kLeast;
      p.y = fabsf(p.y);
    }
  };
  // one row per 16 lanes: the lanes split the row's tiles, then merge pairwise (fixed tree)
  const int row = blockIdx.x * 16 + (threadIdx.x >> 4);
  const int slice = threadIdx.x & 15;
  float m = kLeast, z = 0.f;
  if (row < a.total_rows) {
    const int jq = row / a.Hq;
    const int r = find_segment(a.q_start, a.n_req, jq);
    const int tiles = (a.ctx_len[r] + a.tile_keys - 1) / a.tile_keys;
    for (int t = slice; t < tiles; t += 64) {                  // the loads of four tiles together
      float2 p[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) p[u] = part(min(t + 16 * u, tiles - 1), row);
#pragma unroll
      for (int u = 0; u < 4; ++u) maximum(min(t + 16 * u, tiles - 1), row, p[u]);
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (t + 16 * u < tiles) {
          const float mn = fmaxf(m, p[u].x);
          z = z * exp2f(m - mn) + p[u].y * exp2f(p[u].x - mn);
          m = mn;
        }
    }
    if (a.causal_q && slice == 15) {                           // the question keys' share (slice 15 has the fewest tiles)
      float2 p = part(a.n_tiles, row);
      maximum(a.n_tiles, row, p);
      const float mn = fmaxf(m, p.x);
      z = (z > 0.f ? z * exp2f(m - mn) : 0.f) + p.y * exp2f(p.x - mn);
      m = mn;
    }
  }
#pragma unroll
  for (int off = 8; off > 0; off >>= 1) {
    const float pm = __shfl_xor(m, off, 16), pz = __shfl_xor(z, off, 16);
    const float mn = fmaxf(m, pm);
    // a side that saw no tile has (m, z) = (-inf, 0): its factor must not become exp2(nan)
    const float za = z > 0.f ? z * exp2f(m - mn) : 0.f, zb = pz > 0.f ? pz * exp2f(pm - mn) : 0.f;
    z = (slice & off) ? zb + za : za + zb;                     // same operand order in both lanes of a pair
    m = mn;
  }
  // exp2(l - m) / z = exp2(l - (m + log2 z)): pass B subtracts one number per row
  if (slice == 0 && row < a.total_rows) a.stats[row] = make_float2(z > 0.f ? log2_sum(m, z) : INFINITY, 0.f);
}

// ---------------------------------------------------------------------------------------
// bf16 MFMA kernel, head_dim 128.  PASS 0 = partial row statistics, PASS 1 = column sums.
//
// Workgroup (8 waves, two per CU) = one KV head of one request against a tile of 256 context keys (or 288, scores_tile_keys).  A wave keeps its 32 keys
// in registers, as matrix operands, and walks all rows m = (question token, head) of the KV head; the rows' Q comes through two LDS buffers of 128
// rows, which all waves share.  So no key goes through LDS; a wave forms whole column sums by itself and meets the others only where
// row statistics are merged or Q is exchanged; and Eq. 2 turns the keys where they lie (a lane holds whole pairs of either layout).
//   PASS 0  C[key][row]: a lane owns a row; sums of exp2(l) over the wave's keys, merged over the waves -> one partial (max, sum) per
//           (tile, row).  The sums are taken as they come, without the row's maximum: fp32 holds them over 2^-64 .. 2^100 with the
//           precision it has anywhere.  Where one lies outside, the wave takes those of the 32 rows at hand against their maximum, and
//           from there on all of them: the check costs calls of many rows 1 - 2 % (28 query heads on 4, eight requests of 8000 keys, 32 .. 128 question
//           tokens 112 -> 114 us), one check per 128 rows, with another pass over these rows, costs calls outside the range 10 - 20 % more.
//   PASS 1  C[row][key]: a lane owns a key; the partials of all tiles are merged per row (fixed order, the same in every workgroup),
//           then sum over rows of exp2(l - stat) -> per KV head column sums; a last small kernel adds them in fixed order.
// What bounds it: the issue port.  32 rows x 32 keys are 16 products, 16 x (fma, exp2, add) and 10 LDS reads of a wave, 390 cycles of a
// SIMD with four waves in a loop of nothing else; 450 - 650 are reached, the rest goes into a tile's start.  All LDS addresses are four
// registers and constants, Q's offsets six instructions a row, and a partial is one number as long as nothing left fp32's range.
// Whole calls with position recovery, us, and without (before: keys through LDS, rows in registers, a kernel each for up to 256 rows and for
// more): 65.6K keys of eight requests, 32 .. 128 question tokens, 209 -> 178 and 172 -> 150; 30K keys, 96 tokens, 106 -> 85 and 92 -> 71; 64K, 64 tokens,
// 147 -> 136 and 109 -> 107; 16K, 64 tokens, 48 -> 45 and 37.5 -> 35.4; 2K, 32 tokens, 24 -> 21 and 19.5 -> 17; 5K, 64 tokens, 27 -> 26.5 and 21.4 -> 21.7.
// Slower are calls of 129 .. 256 rows per KV head that leave most CUs idle, whose second chunk is one more chain of latencies: 500 keys, 32 tokens, 28 query
// heads on 4, 20.3 -> 22.4 and 19.0 -> 19.9; four requests of 500 keys, 32 .. 64 tokens, 22.7 -> 24.2 and 20.8 -> 21.7 (no gain: Q's second
// chunk requested behind the first, no barrier between the two); and of such rows a little behind 256 or 512 workgroups where
// scores_tile_keys keeps 256 keys: 10K keys, 64 tokens, 32 heads on 8, 23.9 -> 26.8 and (realign + scores) 32.0 -> 36.4.
// Scores against float64: 1.6 .. 6e-7 -> 0.8 .. 2.8e-7 (log2_sum; 2-norm, keys of which a tenth stand out by 6 in the logit, the rest alike). With
// all logits at +-40 or more the products themselves are that large and their rounding counts: 2-norm 0.2 .. 8e-6, 0.6 .. 1.3 of before, largest error
// of one key up to 2.2 times what it was up to 256 rows per KV head, where the second pass used to start its products from the statistics.
// ---------------------------------------------------------------------------------------
constexpr int kD = 128;
constexpr int kKRowBytes = kD * 2;
constexpr int kKeysWave = 32;                      // keys of a wave
constexpr int kWaves = 8;
constexpr int kTile = kKeysWave * kWaves;          // keys of a workgroup
constexpr int kThreads = 64 * kWaves;
constexpr int kChunk = 128;                        // rows of Q in an LDS buffer
constexpr int kChunkBytes = kChunk * kKRowBytes;
constexpr int kStatRows = 512;                     // row statistics in LDS (PASS 1)
constexpr float kSumLow = 0x1p-64f, kSumHigh = 0x1p100f;
// Q's buffers, then PASS 0: (max, sum) of a chunk's rows of every wave, twice; PASS 1: statistics of kStatRows rows, half of a merge
constexpr size_t scores_lds_bytes(int bufs, int pass) {
  return (size_t)bufs * kChunkBytes + (pass == 0 ? 2 * kWaves * kChunk * sizeof(float2) : kStatRows * sizeof(float) + kThreads / 2 * sizeof(float2));
}
static_assert(kWaves * kKeysWave * sizeof(float) <= kThreads / 2 * sizeof(float2), "the other keys' column sums take the place of half of a merge");
static_assert(2 * scores_lds_bytes(2, 0) <= 160 * 1024 && scores_lds_bytes(2, 1) <= scores_lds_bytes(2, 0), "two workgroups per CU");


__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float halves_max(float x) {
  const uint32_t u = __float_as_uint(x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);   // low-half values / high-half values in all lanes
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float halves_sum(float x) {
  const uint32_t u = __float_as_uint(x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap16_add(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// MORE: tiles of 288 keys, two chunks of rows at most.  Once through the rows with 256 keys, then with the other 32, which every wave holds, for an eighth of
// the rows each.
template <int PASS, bool REALIGN, bool MORE>
__global__ void __launch_bounds__(kThreads, 4)
scores_bf16_kernel(scores_args a) {
  constexpr int kKeys = MORE ? kTile + kKeysWave : kTile;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  // blockIdx % Hkv = KV head: with 8 heads an XCD has one, and its L2 that head's Q rows and partial statistics.  PASS 0 of the causal
  // denominator has one more tile per request, its question keys, each row up to its own token
  auto quotient = [](uint32_t x, uint32_t d, uint32_t inv) { return d == 1 ? x : inv ? __umulhi(x, inv) : x / d; };
  const uint32_t n_runs = (uint32_t)(a.n_tiles + (PASS == 0 && !REALIGN ? a.own_tile : 0));
  const uint32_t rest = quotient(blockIdx.x, a.Hkv, a.inv_heads);
  const int g = (int)(blockIdx.x - rest * a.Hkv), r = a.n_req == 1 ? 0 : (int)quotient(rest, n_runs, a.inv_runs[PASS]), t = (int)(rest - r * n_runs);
  const bool own = PASS == 0 && !REALIGN && t == a.n_tiles;
  const int n_ctx = a.one_ctx_len >= 0 ? a.one_ctx_len : a.ctx_len[r];
  const int i0 = own ? 0 : t * kKeys;
  if (!own && i0 >= n_ctx) return;
  const int G = a.Hq / a.Hkv, n_q = a.one_ctx_len >= 0 ? a.one_q_len : a.q_len[r];
  const int Mg = n_q * G;                                      // rows of this KV head: m = j * G + hh
  const int N = own ? n_q : n_ctx;
  const int s = (a.one_ctx_len >= 0 ? 0 : a.seg_start[r]) + (own ? n_ctx : 0), qrow0 = a.one_ctx_len >= 0 ? 0 : a.q_start[r];
  const int row0 = qrow0 * a.Hq + g * Mg;                      // first of the head's rows in part and stats
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lg = lane >> 4;
  // waves with question keys, of which there may be few: the others take some of their rows
  const int key_waves = !own || n_q > 128 ? kWaves : n_q > 64 ? 4 : n_q > 32 ? 2 : 1;
  int share = kWaves / key_waves, sub = wave / key_waves;
  int iw = i0 + kKeysWave * (wave & (key_waves - 1));          // the wave's first key
  const int n_chunks = (Mg + kChunk - 1) / kChunk;
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds_raw;
  unsigned char *extra = lds_raw + min(n_chunks, 2) * kChunkBytes;
  float *St = reinterpret_cast<float *>(extra);                // PASS 1: [kStatRows]
  float *pz = reinterpret_cast<float *>(extra), *pm = pz + 2 * kWaves * kChunk;        // PASS 0: partials of the waves, [2][kWaves][kChunk]

  // ---- keys from i on: fragment (kb, ks) of a lane: 16 bytes of key i + 16 kb + l16, dims 32 ks + 8 lg ..
  bf16x8 kf[2][4];
  int krow[2], chunk[2];
  const bf16_t *Kin = (const bf16_t *)(REALIGN ? a.k_cat : a.k);
  auto load_keys = [&](int i) {
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      krow[kb] = min(s + i + 16 * kb + l16, a.T - 1);          // past the run: loaded, masked or never stored
      if (REALIGN) chunk[kb] = i + 16 * kb + l16 < N ? a.tok_chunk[krow[kb]] : -1;
    }
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
        kf[kb][ks] = *reinterpret_cast<const bf16x8 *>(Kin + ((size_t)krow[kb] * a.Hkv + g) * kD + 32 * ks + 8 * lg);
  };
  load_keys(iw);
  // ---- Q: chunk C of rows to its buffer, as 32-bit offsets from the first token that it reaches into (of the request they would end at 4 GiB)
  const int drow = 4 * wave + (lane >> 4), dpiece = (lane & 15) ^ (drow & 15);
  const bf16_t *Qr = (const bf16_t *)a.q + ((size_t)qrow0 * a.Hq + g * G) * kD;      // row 0 of the head
#define A3_QDMA(C)                                                                                             \
  {                                                                                                            \
    const uint32_t j0_ = G > 1 ? __umulhi((uint32_t)((C) * kChunk), a.inv_G) : (uint32_t)((C) * kChunk);       \
    const bf16_t *qc_ = Qr + (size_t)j0_ * a.Hq * kD;                                                          \
    _Pragma("unroll") for (int j = 0; j < kChunk / (4 * kWaves); ++j) {                                        \
      const uint32_t m_ = (uint32_t)min((C) * kChunk + drow + 4 * kWaves * j, Mg - 1);                         \
      const uint32_t off_ = (m_ + (G > 1 ? __umulhi(m_, a.inv_G) : m_) * (uint32_t)(a.Hq - G) - j0_ * a.Hq) * (kD * 2) + 16 * dpiece; \
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"                             \
                   :: "s"(lds_base + ((C) & 1) * kChunkBytes + (4 * wave + 4 * kWaves * j) * kKRowBytes), "v"(off_), "s"(qc_) : "memory"); \
    }                                                                                                          \
  }
  static_assert((4 * kWaves) % 16 == 0, "the swizzle of a lane's rows is one number");
  if (n_chunks > 0) { A3_QDMA(0) }
  if (n_chunks > 1) { A3_QDMA(1) }

  if (PASS == 1 && Mg > 0) {
    if (a.merged) {
      for (int m = tid; m < min(n_chunks * kChunk, kStatRows); m += kThreads) St[m] = m < Mg ? a.stats[row0 + m].x : INFINITY;
    } else {
      // two threads a row where there are enough (up to 64 runs), else one (up to 32)
      const bool two = Mg <= kThreads / 2;
      const int m = two ? tid % (kThreads / 2) : tid, first = two ? tid / (kThreads / 2) * 32 : 0;
      const int runs = (N + kKeys - 1) / kKeys;
      const size_t at = (size_t)row0 + min(m, Mg - 1);
      float mx = 0.f, z = 0.f, p[32];
#pragma unroll
      for (int u = 0; u < 32; ++u) p[u] = first + u < runs ? a.part_z[(size_t)(first + u) * a.total_rows + at] : 0.f;
      const float pq = a.causal_q && first == 0 ? a.part_z[(size_t)a.n_tiles * a.total_rows + at] : 0.f;
      float least = pq;
#pragma unroll
      for (int u = 0; u < 32; ++u) { z += p[u]; least = fminf(least, p[u]); }
      z += pq;
      if (least < 0.f) {                                       // sums against a maximum among them: those of 16 tiles requested together
        mx = pq < 0.f ? a.part_m[(size_t)a.n_tiles * a.total_rows + at] : pq > 0.f ? 0.f : kLeast;
        z = fabsf(pq);
#pragma unroll
        for (int u0 = 0; u0 < 32; u0 += 16) {
          float m[16], mn = mx;
#pragma unroll
          for (int u = 0; u < 16; ++u) m[u] = p[u0 + u] < 0.f ? a.part_m[(size_t)(first + u0 + u) * a.total_rows + at] : p[u0 + u] > 0.f ? 0.f : kLeast;
#pragma unroll
          for (int u = 0; u < 16; ++u) mn = fmaxf(mn, m[u]);
          z *= fast_exp2(mx - mn);
#pragma unroll
          for (int u = 0; u < 16; ++u) z += fabsf(p[u0 + u]) * fast_exp2(m[u] - mn);
          mx = mn;
        }
      }
      if (!(z > 0.f)) mx = kLeast;                             // (a half without tiles)
      if (two) {
        float2 *half = reinterpret_cast<float2 *>(St + kStatRows);          // [kThreads / 2]
        if (first) half[m] = make_float2(mx, z);
        __syncthreads();
        if (!first) {
          const float2 o = half[m];
          const float mn = fmaxf(mx, o.x);
          z = (z > 0.f ? z * fast_exp2(mx - mn) : 0.f) + (o.y > 0.f ? o.y * fast_exp2(o.x - mn) : 0.f);
          mx = mn;
        }
      }
      if (!first) St[m] = m < Mg && z > 0.f ? log2_sum(mx, z) : INFINITY;
    }
  }

  auto turn_keys = [&]() {
    const bool inter = a.rope_layout == A3_ROPE_INTERLEAVED;
#pragma unroll
    for (int p = 0; p < 2; ++p) {                              // dims of fragments 2 p and 2 p + 1 (interleaved), or p and p + 2
      float2 cs[8];
      int cur = -1;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        if (chunk[kb] >= 0) {
          if (chunk[kb] != cur) {
            const float2 *tab = a.chunk_cs + (size_t)chunk[kb] * (kD / 2) + (inter ? 32 * p + 4 * lg : 32 * p + 8 * lg);
#pragma unroll
            for (int e = 0; e < 8; ++e) cs[e] = tab[inter && e >= 4 ? e + 12 : e];
            cur = chunk[kb];
          }
          if (inter) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              bf16x8 &f = kf[kb][2 * p + (e >> 2)];
              float y0, y1;
              a3_rotate_pair(a3_bf2f(f[2 * (e & 3)]), a3_bf2f(f[2 * (e & 3) + 1]), cs[e], y0, y1);
              f[2 * (e & 3)] = a3_f2bf(y0);
              f[2 * (e & 3) + 1] = a3_f2bf(y1);
            }
          } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              float y0, y1;
              a3_rotate_pair(a3_bf2f(kf[kb][p][e]), a3_bf2f(kf[kb][p + 2][e]), cs[e], y0, y1);
              kf[kb][p][e] = a3_f2bf(y0);
              kf[kb][p + 2][e] = a3_f2bf(y1);
            }
          }
        }
      }
    }
    __builtin_amdgcn_s_waitcnt(0);                             // Q has landed: nothing below waits for the stores
    asm volatile("" ::: "memory");
  };
  auto store_keys = [&](int i) {
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
      if (i + 16 * kb + l16 < N) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
          *reinterpret_cast<bf16x8 *>((bf16_t *)a.k_out + ((size_t)krow[kb] * a.Hkv + g) * kD + 32 * ks + 8 * lg) = kf[kb][ks];
      }
  };
  if (REALIGN) {
    turn_keys();
    store_keys(iw);
  }

  bool have = iw < N, tail = own || iw + kKeysWave > N;
  bool careful = false;                                        // PASS 0: the wave takes its sums against their maximum
  float colsum[2] = {0.f, 0.f};
  // LDS addresses of a lane's fragments of the rows l16 of a chunk, dims 32 ks + 8 lg ..: everything else is a constant offset
  typedef __attribute__((address_space(3))) const unsigned char *lds_ptr;
  const uint32_t stat_at = lds_base + min(n_chunks, 2) * kChunkBytes + 16 * lg;
  uint32_t qat[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) qat[ks] = lds_base + l16 * kKRowBytes + ((64 * ks) ^ (16 * (lg ^ l16)));
  // Q and the keys are there
  if (!REALIGN) __builtin_amdgcn_s_waitcnt(0);
  A3_LDS_BARRIER();
  const int i1 = i0 + kTile, n_more = own ? 0 : min(kKeysWave, N - i1);       // MORE: the other keys
  for (int part = 0; part < (MORE ? 2 : 1); ++part) {
    if (MORE && part == 1) {
      if (n_more > 0) {
        load_keys(i1);
        if (REALIGN) {
          turn_keys();
          A3_LDS_BARRIER();                                      // (in place: every wave has read the keys)
          if (wave == 0) store_keys(i1);
        }
      }
      iw = i1;
      share = kWaves;
      sub = wave;
      have = n_more > 0;
      tail = iw + kKeysWave > N;
      colsum[0] = colsum[1] = 0.f;
    }
    for (int c = 0; c < n_chunks; ++c) {
      if (c > 0 && c + 1 < n_chunks) { A3_QDMA(c + 1) }
      if (PASS == 1 && a.merged && (c + 1) * kChunk >= kStatRows && c + 1 < n_chunks && tid < kChunk) {
        const int m = (c + 1) * kChunk + tid;
        St[m % kStatRows] = m < Mg ? a.stats[row0 + m].x : INFINITY;
      }
      const uint32_t cb = (c & 1) * kChunkBytes;
      const int rows = min(kChunk, Mg - c * kChunk);
      if (have) {
        // logits of the 16 rows from row q of the chunk on
        auto logits = [&](int q, f32x4 (&acc)[2]) {
          bf16x8 qf[4];
#pragma unroll
          for (int ks = 0; ks < 4; ++ks) qf[ks] = *(__attribute__((address_space(3))) const bf16x8 *)((lds_ptr)(uintptr_t)(qat[ks] + cb) + q * kKRowBytes);
#pragma unroll
          for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
              const f32x4 c0 = ks == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[kb];
              acc[kb] = PASS == 0 ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kb][ks], qf[ks], c0, 0, 0, 0)
                                  : __builtin_amdgcn_mfma_f32_16x16x32_bf16(qf[ks], kf[kb][ks], c0, 0, 0, 0);
            }
        };
        if (PASS == 0) {
          // of the wave's keys, those that the lane's row sees
          auto seen_by = [&](int q) {
            if (!own) return N - iw;
            const int m = c * kChunk + q + l16;
            return min(N, (G > 1 ? (int)__umulhi((uint32_t)m, a.inv_G) : m) + 1) - iw;
          };
          auto mask = [&](int seen, f32x4 (&acc)[2]) {
            seen -= 4 * lg;
            asm volatile("" : "+v"(seen));
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
              for (int e = 0; e < 4; ++e)
                if (16 * kb + e >= seen) acc[kb][e] = -INFINITY;
          };
          float *pzw = pz + ((c & 1) * kWaves + wave) * kChunk, *pmw = pm + ((c & 1) * kWaves + wave) * kChunk;
          auto add = [&](int m, float mx, float z) {             // onto what the wave has of row m
            const float z0 = pzw[m];
            if (z0 >= 0.f && mx == 0.f) {
              pzw[m] = z0 + z;
            } else {
              const float m0 = z0 < 0.f ? pmw[m] : z0 > 0.f ? 0.f : kLeast, mn = fmaxf(m0, mx);
              store_partial(pzw, pmw, m, mn, fabsf(z0) * fast_exp2(m0 - mn) + z * fast_exp2(mx - mn));
            }
          };
#pragma unroll
          for (int rg = 0; rg < kChunk; rg += 32) {
            if (rg >= rows) break;
            if (share > 1 && ((c * (kChunk / 32) + rg / 32) & (share - 1)) != sub) {             // (another wave's rows)
              if (!(MORE && part == 1) && lane < 32) pzw[rg + lane] = 0.f;
              continue;
            }
            f32x4 acc[2][2];
            logits(rg, acc[0]);
            logits(rg + 16, acc[1]);
            if (tail) {
              mask(seen_by(rg), acc[0]);
              mask(seen_by(rg + 16), acc[1]);
            }
            // both sums over the wave's keys: lane groups 0 and 2 get the first 16 rows', lane groups 1 and 3 the others'
            auto sums = [&](auto power) {
              float z[2];
#pragma unroll
              for (int b = 0; b < 2; ++b) {
                float z0 = power(b, acc[b][0][0]), z1 = power(b, acc[b][1][0]);
#pragma unroll
                for (int e = 1; e < 4; ++e) {
                  z0 += power(b, acc[b][0][e]);
                  z1 += power(b, acc[b][1][e]);
                }
                z[b] = z0 + z1;
              }
              return halves_sum(swap16_add(z[0], z[1]));
            };
            if (!careful) {
              const float zz = sums([&](int, float x) { return fast_exp2(x * a.scale2); });
              careful = __any(!(zz >= kSumLow && zz <= kSumHigh) && !(own && seen_by(rg + (lane & 16)) <= 0));   // (0: the row sees none of the keys)
              if (MORE && part == 1) {
                if (!careful && lane < 32) add(rg + lane, 0.f, zz);
              } else if (!careful && lane < 32) {
                pzw[rg + lane] = zz;
              }
            }
            if (careful) {
              float mx[2];
#pragma unroll
              for (int b = 0; b < 2; ++b) {
                mx[b] = fmaxf(acc[b][0][0], acc[b][1][0]);
#pragma unroll
                for (int e = 1; e < 4; ++e) mx[b] = fmaxf(fmaxf(mx[b], acc[b][0][e]), acc[b][1][e]);
              }
              const auto w = __builtin_amdgcn_permlane16_swap(__float_as_uint(mx[0]), __float_as_uint(mx[1]), false, false);
              const float own_mx = fmaxf(halves_max(fmaxf(__uint_as_float(w[0]), __uint_as_float(w[1]))) * a.scale2, kLeast);
              const auto u = __builtin_amdgcn_permlane16_swap(__float_as_uint(own_mx), __float_as_uint(own_mx), false, false);
              const float of[2] = {__uint_as_float(u[0]), __uint_as_float(u[1])};
              const float zz = sums([&](int b, float x) { return fast_exp2(fmaf(x, a.scale2, -of[b])); });
              if (MORE && part == 1) {
                if (lane < 32) add(rg + lane, own_mx, zz);
              } else if (lane < 32) {
                store_partial(pzw, pmw, rg + lane, own_mx, zz);
              }
            }
          }
        } else {
          const uint32_t sat = stat_at + (c * kChunk) % kStatRows * 4;
#pragma unroll
          for (int rg = 0; rg < kChunk; rg += 32) {
            if (rg >= rows) break;
            if (MORE && part == 1 && c * (kChunk / 32) + rg / 32 != wave) continue;
            f32x4 acc[2][2], st[2];
#pragma unroll
            for (int b = 0; b < 2; ++b) st[b] = *(__attribute__((address_space(3))) const f32x4 *)((lds_ptr)(uintptr_t)sat + (rg + 16 * b) * 4);
            logits(rg, acc[0]);
            logits(rg + 16, acc[1]);
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
              float p0 = fast_exp2(fmaf(acc[0][kb][0], a.scale2, -st[0][0])), p1 = fast_exp2(fmaf(acc[1][kb][0], a.scale2, -st[1][0]));
#pragma unroll
              for (int e = 1; e < 4; ++e) {
                p0 += fast_exp2(fmaf(acc[0][kb][e], a.scale2, -st[0][e]));
                p1 += fast_exp2(fmaf(acc[1][kb][e], a.scale2, -st[1][e]));
              }
              colsum[kb] += p0 + p1;
            }
          }
        }
      } else if (PASS == 0 && !(MORE && part == 1)) {
        for (int m = lane; m < rows; m += 64) pz[((c & 1) * kWaves + wave) * kChunk + m] = 0.f;
      }
      if (MORE && part == 0) continue;                           // (all of Q is in LDS, the rows are merged behind the other keys)
      if (c + 1 < n_chunks) __builtin_amdgcn_s_waitcnt(0);       // the next chunk of Q has landed
      if (PASS == 0 || c + 1 < n_chunks) { A3_LDS_BARRIER(); }
      if (PASS == 0 && tid < rows) {
        const float *zc = pz + (c & 1) * kWaves * kChunk + tid, *mc = pm + (c & 1) * kWaves * kChunk + tid;
        float mx = 0.f, z = 0.f, least = 0.f, x[kWaves];
#pragma unroll
        for (int w = 0; w < kWaves; ++w) { x[w] = zc[w * kChunk]; z += x[w]; least = fminf(least, x[w]); }
        if (least < 0.f) {
          float xm[kWaves];
          mx = kLeast;
          z = 0.f;
#pragma unroll
          for (int w = 0; w < kWaves; ++w) xm[w] = mc[w * kChunk];
#pragma unroll
          for (int w = 0; w < kWaves; ++w) { xm[w] = x[w] < 0.f ? xm[w] : x[w] > 0.f ? 0.f : kLeast; mx = fmaxf(mx, xm[w]); }
#pragma unroll
          for (int w = 0; w < kWaves; ++w) z += fabsf(x[w]) * fast_exp2(xm[w] - mx);
        }
        store_partial(a.part_z, a.part_m, (size_t)t * a.total_rows + row0 + c * kChunk + tid, mx, z);
      }
    }
    if (PASS == 1 && part == 0) {
      // lane groups 0 and 2: key block 0, groups 1 and 3: key block 1
      const float v = halves_sum(swap16_add(colsum[0], colsum[1]));
      if (lane < kKeysWave && iw + lane < N) a.part_scores[(size_t)g * a.T + s + iw + lane] = v;
    }
  }
#undef A3_QDMA
  if (MORE && PASS == 1) {
    float *red = St + kStatRows;                               // [kWaves][kKeysWave] column sums of the other keys (the merge's place)
    const float v = halves_sum(swap16_add(colsum[0], colsum[1]));
    if (lane < kKeysWave) red[wave * kKeysWave + lane] = v;
    A3_LDS_BARRIER();
    if (tid < n_more) {
      float sum = 0.f;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) sum += red[w * kKeysWave + tid];
      a.part_scores[(size_t)g * a.T + s + i1 + tid] = sum;
    }
  }
}

// scores[t] = sum over KV heads of their column sums, in head order; question rows get -inf.  Nothing but the latency of its loads, so
// those of eight heads and of the row's chunk are requested together (one after the other 3.3 us for 544 rows and 8 heads, now 1.9; a layer
// pass of 2K rows 117.5 -> 115.9).
__global__ void __launch_bounds__(256)
scores_head_sum_kernel(scores_args a, const int *__restrict__ tok_chunk) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= a.T) return;
  const int chunk = tok_chunk[t];
  float v = 0.f;
  for (int g0 = 0; g0 < a.Hkv; g0 += 8) {
    float p[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) p[u] = a.part_scores[(size_t)min(g0 + u, a.Hkv - 1) * a.T + t];
#pragma unroll
    for (int u = 0; u < 8; ++u) v = g0 + u < a.Hkv ? v + p[u] : v;
  }
  a.scores[t] = chunk >= 0 ? v : -INFINITY;
}

// ---------------------------------------------------------------------------------------
// fp32 kernels (head_dim 64 or 128): logits on the fp32 matrix instruction, fragments straight from memory
// ---------------------------------------------------------------------------------------
// One workgroup per (64-key tile, KV head, request); a wave owns 16 of the keys and walks the head's rows 16 at a time.
// 16x16x4 products: a lane's 16-byte load holds four consecutive coordinates of one key or row, one for each of four
// instructions (which coordinate goes to which does not matter as long as both operands agree).  C[key][row]: register
// r of lane (l16, lg) is key 4 lg + r, row l16.  (One thread per key and row slice, 64 coordinates deep, took 280 +
// 188 us for 512 keys x 256 rows.)  Small calls are launches and latency: with REALIGN the first pass turns the stale keys itself (a lane holds
// whole pairs of either layout) and stores them, and the second (MERGE) merges the row statistics itself (512 keys, 32 rows per head: four launches of 3 - 5 us
// -> two of 5 - 6).
constexpr int kF32MergeRows = 1024;              // row statistics in LDS
// Every workgroup merges tiles x rows partials where the combine kernel would merge them once, for a launch of 3 to 5 us.  Calls with the merge in
// the pass and with the kernel, us: 8 tiles 154 and 165 (1024 rows, 384 workgroups), 759 and 772 (1536); 16 tiles, 256 workgroups 112 and 119
// (1024 rows), 768 workgroups 39 and 41 (128 rows), 66 and 67 (256), 232 and 221 (1024), 512 workgroups of 128 coordinates 48.3 and 48.2 (128),
// 84 and 80 (256); 32 tiles, 256 workgroups 36 and 37 (256), 62 and 60 (512), 121 and 107 (1024), 512 workgroups 33 and 32 (128), 52 and
// 49 (256).  Many workgroups of few rows lose as well: 16 tiles, 1536 workgroups, 8 rows 24.6 and 23.7.
constexpr bool f32_merges(long long tiles, long long workgroups, long long rows) {
  if (rows > kF32MergeRows) return false;
  return tiles <= 8 || (tiles <= 16 && (workgroups <= 256 || (workgroups <= 768 && rows <= 128))) || (tiles <= 32 && workgroups <= 256 && rows <= 256);
}
template <int PASS, int D, bool REALIGN, bool MERGE>
__global__ void __launch_bounds__(256)
scores_f32_kernel(scores_args a) {
  __shared__ float2 red[4][16];                                // PASS 0: (max, sum) of the rows over a wave's keys
  __shared__ float stats[MERGE ? kF32MergeRows : 1];
  const int r = blockIdx.z, g = blockIdx.y;
  const int N = a.ctx_len[r], i0 = blockIdx.x * kTileKeys;
  if (i0 >= N) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, lg = lane >> 4;
  const int s = a.seg_start[r], G = a.Hq / a.Hkv, Mg = a.q_len[r] * G, qrow0 = a.q_start[r];
  const float *__restrict__ Q = (const float *)a.q;
  const int key0 = i0 + 16 * wave;                             // first key of the wave
  f32x4 kf[D / 16];
  {
    const size_t at = ((size_t)min(s + key0 + l16, a.T - 1) * a.Hkv + g) * (D / 4) + lg;
    const f32x4 *kp = reinterpret_cast<const f32x4 *>(REALIGN ? a.k_cat : a.k) + at;
#pragma unroll
    for (int c = 0; c < D / 16; ++c) kf[c] = kp[4 * c];
    if (REALIGN && key0 + l16 < N) {
      // coordinates 16 c + 4 lg .. + 3: two pairs of the interleaved layout, or the first members of pairs with fragment c + D / 32
      const int chunk = a.tok_chunk[s + key0 + l16];
      if (chunk < 0) {                                         // (a row of no chunk: it stays what it is)
        const f32x4 *kp0 = reinterpret_cast<const f32x4 *>(a.k) + at;
#pragma unroll
        for (int c = 0; c < D / 16; ++c) kf[c] = kp0[4 * c];
      } else {
        const float2 *tab = a.chunk_cs + (size_t)chunk * (D / 2);
        if (a.rope_layout == A3_ROPE_INTERLEAVED) {
#pragma unroll
          for (int c = 0; c < D / 16; ++c) {
            float y[4];
            a3_rotate_pair(kf[c][0], kf[c][1], tab[8 * c + 2 * lg], y[0], y[1]);
            a3_rotate_pair(kf[c][2], kf[c][3], tab[8 * c + 2 * lg + 1], y[2], y[3]);
            kf[c] = f32x4{y[0], y[1], y[2], y[3]};
          }
        } else {
#pragma unroll
          for (int c = 0; c < D / 32; ++c) {
            float lo[4], hi[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) a3_rotate_pair(kf[c][e], kf[c + D / 32][e], tab[16 * c + 4 * lg + e], lo[e], hi[e]);
            kf[c] = f32x4{lo[0], lo[1], lo[2], lo[3]};
            kf[c + D / 32] = f32x4{hi[0], hi[1], hi[2], hi[3]};
          }
        }
        f32x4 *ko = reinterpret_cast<f32x4 *>(a.k_out) + at;
#pragma unroll
        for (int c = 0; c < D / 16; ++c) ko[4 * c] = kf[c];
      }
    }
  }
  auto row_of = [&](int m) { return (qrow0 + m / G) * a.Hq + g * G + m % G; };
  f32x4 qf[D / 16];
  auto load_q = [&](int m0) {
    const f32x4 *qp = reinterpret_cast<const f32x4 *>(Q + (size_t)row_of(min(m0 + l16, Mg - 1)) * D) + lg;
#pragma unroll
    for (int c = 0; c < D / 16; ++c) qf[c] = qp[4 * c];
  };
  f32x4 colsum = {0.f, 0.f, 0.f, 0.f};
  if (Mg > 0) load_q(0);
  if constexpr (MERGE) {                                       // at most kF32MergeRows rows
    for (int m = threadIdx.x; m < Mg; m += 256) {
      const float2 *pp = a.part + row_of(m);
      const int tiles = (N + kTileKeys - 1) / kTileKeys;
      const float2 own = a.causal_q ? pp[(size_t)a.n_tiles * a.total_rows] : make_float2(kLeast, 0.f);
      float mx = own.x, z = own.y;
      for (int t0 = 0; t0 < tiles; t0 += 8) {
        float2 p[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) p[u] = pp[(size_t)min(t0 + u, tiles - 1) * a.total_rows];
        float mn = mx;
#pragma unroll
        for (int u = 0; u < 8; ++u) mn = fmaxf(mn, p[u].x);
        z *= exp2f(mx - mn);
#pragma unroll
        for (int u = 0; u < 8; ++u) z += t0 + u < tiles ? p[u].y * exp2f(p[u].x - mn) : 0.f;
        mx = mn;
      }
      stats[m] = z > 0.f ? mx + log2f(z) : INFINITY;
    }
    __syncthreads();
  }
  for (int m0 = 0; m0 < Mg; m0 += 16) {
    const int m = m0 + l16, row = row_of(min(m, Mg - 1));
    const float stat = PASS == 0 ? 0.f : MERGE ? stats[min(m, Mg - 1)] : a.stats[row].x;
    f32x4 c4[4];                                               // four chains, so that no product waits for the one before
#pragma unroll
    for (int e = 0; e < 4; ++e) c4[e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < D / 16; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) c4[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][e], qf[c][e], c4[e], 0, 0, 0);
    if (m0 + 16 < Mg) load_q(m0 + 16);
    f32x4 l;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      l[e] = key0 + 4 * lg + e < N ? ((c4[0][e] + c4[1][e]) + (c4[2][e] + c4[3][e])) * a.scale2 : -INFINITY;
    if (PASS == 0) {
      float mx = fmaxf(fmaxf(l[0], l[1]), fmaxf(l[2], l[3]));
      mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      float z = 0.f;
      if (mx > -INFINITY) z = (exp2f(l[0] - mx) + exp2f(l[1] - mx)) + (exp2f(l[2] - mx) + exp2f(l[3] - mx));
      z += __shfl_xor(z, 16, 64);
      z += __shfl_xor(z, 32, 64);
      __syncthreads();                                         // the block before has been read
      if (lg == 0) red[wave][l16] = make_float2(mx, z);
      __syncthreads();
      if (threadIdx.x < 16 && m < Mg) {
        float mm = kLeast, zz = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) mm = fmaxf(mm, red[w][l16].x);
#pragma unroll
        for (int w = 0; w < 4; ++w) zz += red[w][l16].y * exp2f(red[w][l16].x - mm);
        a.part[(size_t)blockIdx.x * a.total_rows + row] = make_float2(mm, zz);
      }
    } else if (m < Mg) {
#pragma unroll
      for (int e = 0; e < 4; ++e) colsum[e] += exp2f(l[e] - stat);
    }
  }
  if (PASS == 1) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
#pragma unroll
      for (int off = 1; off < 16; off <<= 1) colsum[e] += __shfl_xor(colsum[e], off, 64);
      if (l16 == 0 && key0 + 4 * lg + e < N) a.part_scores[(size_t)g * a.T + s + key0 + 4 * lg + e] = colsum[e];
    }
  }
}

}  // namespace

size_t a3_scores_ws_bytes(const a3_layout *L) {
  // rows of the score matrix over the whole batch are bounded by n_req * max_q_len * Hq
  const size_t total_rows = (size_t)L->n_req * L->max_q_len * L->n_q_heads;
  const int tk = L->dtype == A3_BF16 ? kTile : kTileKeys;
  const size_t n_tiles = (size_t)(L->max_ctx_len + tk - 1) / tk;
  return a3_align_up((n_tiles + 1) * total_rows * sizeof(float2), 256) + a3_align_up(total_rows * sizeof(float2), 256) +
         a3_align_up((size_t)L->n_kv_heads * L->total_tokens * sizeof(float), 256) + 256;
}

// Keys of a tile of the bf16 passes.  A pass lasts as long as the CUs with the most workgroups: where a few more than 256, or than 512, would be left
// over, each takes 32 more keys, up to 256 rows per KV head (all of Q in LDS).  Votes and realign + scores with 256 and 288 keys, us, 8 KV heads:
// 256 rows, 280 workgroups 28.0 and 22.7, 36.3 and 32.2; 528 40.1 and 33.5, 52.0 and 48.0; 552 40.6 and 34.6, 52.0 and 48.6.
// 64 rows, 272 workgroups 16.6 and 15.7, 27.1 and 25.8.
// Lines: behind 256, context for 264 workgroups up to one and a half chunks (for 258 64 rows 14.4 and 15.5, 22.5 and 25.2; 256 rows 24.5 and 22.5,
// 32.3 and 32.1).  Behind 512, room for one workgroup more per KV head (256 rows, 576 and 504: votes 39.6 and 42.6); votes from the second chunk on (64
// rows, 528: 23.8 and 24.9); scores, which may realign, from 520 (256 rows, 514: 45.0 and 47.4 in one run, 48.9 and 47.9 in another) and 192 rows (160
// rows, 528 of two requests: votes 33.5 and 29.8, realign + scores 43.5 and 44.8).  Inside them the worst that was seen is realign + scores of 36000 keys
// on 4 KV heads, 252 rows: 50.7 and 52.0.
// heads: KV heads of all requests, one workgroup each per tile.  own: votes, whose question keys have workgroups of their own.  The same
// for scores with and without position recovery: they give the same bits.
constexpr int scores_tile_keys(int max_ctx_len, long long heads, long long rows, bool own) {
  const long long now = heads * ((max_ctx_len + kTile - 1) / kTile), less = heads * ((max_ctx_len + kTile + kKeysWave - 1) / (kTile + kKeysWave));
  const bool many = rows > kChunk + kChunk / 2;
  const bool first = now > 256 && less + (own ? heads : 0) <= 256 && (many || heads * max_ctx_len >= 264LL * kTile);
  const bool second = less + heads <= 512 && (own ? now > 512 && rows > kChunk : many && heads * max_ctx_len >= 520LL * kTile);
  return rows <= 2 * kChunk && (first || second) ? kTile + kKeysWave : kTile;
}

// k_cat != nullptr: the first pass also realigns (k_cat -> k_fused).
// causal_q: the question keys a question token sees join its softmax denominator.  votes != nullptr: the per
// KV head column sums [Hkv, T] go there; scores may then be NULL (no sum over heads).
static a3_status scores_launch(const a3_layout *L, const void *q_question, const void *k_cat, void *k_fused,
                               float *scores, void *ws, size_t ws_bytes, void *stream, int causal_q = 0,
                               float *votes = nullptr) {
  a3_status s = a3_check_layout(L, "a3_question_scores", true);
  if (s != A3_OK) return s;
  A3_REQUIRE(q_question && k_fused && (scores || votes), A3_ERR_INVALID_ARG, "a3_question_scores: NULL tensor");
  A3_REQUIRE(a3_aligned16(q_question) && a3_aligned16(k_fused), A3_ERR_INVALID_ARG,
             "a3_question_scores: tensors must be 16-byte aligned");
  A3_REQUIRE(ws != nullptr, A3_ERR_WORKSPACE, "a3_question_scores: workspace is NULL");
  A3_REQUIRE(ws_bytes >= a3_scores_ws_bytes(L), A3_ERR_WORKSPACE,
             "a3_question_scores: workspace %zu bytes, need %zu", ws_bytes, a3_scores_ws_bytes(L));
  A3_REQUIRE(L->max_ctx_len > 0 && L->max_q_len > 0, A3_ERR_UNSUPPORTED,
             "a3_question_scores: needs max_ctx_len > 0 and max_q_len > 0");
  hipStream_t st = (hipStream_t)stream;
  const bool bf16 = L->dtype == A3_BF16;
  const size_t total_rows = (size_t)L->n_req * L->max_q_len * L->n_q_heads;   // upper bound, used as row pitch
  const int G = L->n_q_heads / L->n_kv_heads;
  // the question keys' share of the denominators: a tile of the first pass itself in bf16, up to its 256 keys; a kernel before the
  // passes otherwise
  const bool own_runs = causal_q && bf16 && L->max_q_len <= kTile;
  const int tk = bf16 ? scores_tile_keys(L->max_ctx_len, (long long)L->n_req * L->n_kv_heads, (long long)L->max_q_len * G, own_runs) : kTileKeys;
  const int n_tiles = (L->max_ctx_len + tk - 1) / tk;
  a3_ws_cursor cur(ws, ws_bytes);
  scores_args a;
  a.q = q_question; a.k = k_fused;
  a.seg_start = L->seg_start; a.ctx_len = L->ctx_len; a.q_len = L->q_len; a.q_start = L->q_start;
  a.part = (float2 *)cur.take((size_t)(n_tiles + 1) * total_rows * sizeof(float2));
  a.part_z = (float *)a.part;
  a.part_m = a.part_z + (size_t)(n_tiles + 1) * total_rows;
  a.stats = (float2 *)cur.take(total_rows * sizeof(float2));
  a.part_scores = (float *)cur.take((size_t)L->n_kv_heads * L->total_tokens * sizeof(float));
  if (votes) a.part_scores = votes;                            // a KV head's column sums are its votes
  a.inv_G = G > 1 ? (uint32_t)(((1ull << 32) + G - 1) / G) : 0u;
  a.causal_q = causal_q;
  a.merged = 0;
  a.scores = scores;
  a.n_req = L->n_req; a.Hq = L->n_q_heads; a.Hkv = L->n_kv_heads; a.d = L->head_dim; a.T = L->total_tokens;
  a.total_rows = (int)total_rows; a.n_tiles = n_tiles; a.tile_keys = tk;
  a.scale2 = a3_scale_of(L) * kLog2e;
  const bool one = L->n_req == 1 && L->max_ctx_len + L->max_q_len == L->total_tokens;
  a.one_ctx_len = one ? L->max_ctx_len : -1;
  a.one_q_len = one ? L->max_q_len : -1;
  a.k_cat = k_cat; a.k_out = k_fused; a.tok_chunk = L->tok_chunk; a.chunk_cs = (const float2 *)L->rope_chunk_cs;
  a.rope_layout = L->rope_layout;
  const bool fuse = k_cat != nullptr && L->n_chunks > 0;
  if (k_cat != nullptr && !fuse) {
    s = a3_rope_realign(L, k_cat, k_fused, stream);
    if (s != A3_OK) return s;
  }
  a.own_tile = own_runs;
  if (causal_q && !own_runs) {
    const dim3 qgrid((unsigned)((total_rows + 3) / 4));
    if (bf16) hipLaunchKernelGGL(scores_question_stats_kernel<bf16_t>, qgrid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL(scores_question_stats_kernel<float>, qgrid, dim3(256), 0, st, a);
  }
  if (bf16) {
    static a3_once_per_device lds_once;
    const hipError_t e = a3_once(lds_once, []() {
      for (const void *fn : {(const void *)scores_bf16_kernel<0, false, false>, (const void *)scores_bf16_kernel<0, true, false>, (const void *)scores_bf16_kernel<1, false, false>,
                             (const void *)scores_bf16_kernel<0, false, true>, (const void *)scores_bf16_kernel<0, true, true>, (const void *)scores_bf16_kernel<1, false, true>}) {
        const hipError_t e_ = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)scores_lds_bytes(2, 0));
        if (e_ != hipSuccess) return e_;
      }
      return hipSuccess;
    });
    if (e != hipSuccess) return a3_fail(A3_ERR_HIP, "a3_question_scores: cannot raise the dynamic LDS limit: %s", hipGetErrorString(e));
    const long long wgs = (long long)L->n_req * n_tiles * L->n_kv_heads, wgs0 = wgs + (own_runs ? (long long)L->n_req * L->n_kv_heads : 0);
    A3_REQUIRE(wgs0 < (1LL << 31), A3_ERR_UNSUPPORTED, "a3_question_scores: batch too large");
    const long long rows = (long long)L->max_q_len * G;          // of a KV head, at most
    // The second pass merges the partials of a row in its threads, 32 each: two threads a row up to 256 rows.  (A launch of the combine
    // kernel is 5 us.)
    a.merged = n_tiles > (rows <= kThreads / 2 ? 64 : rows <= kThreads ? 32 : 0);
    auto inverse = [](long long d, long long n) { return d > 1 && n * d < (1LL << 32) ? (uint32_t)(((1ull << 32) + d - 1) / d) : 0u; };
    a.inv_heads = inverse(L->n_kv_heads, wgs0);
    a.inv_runs[0] = inverse(n_tiles + (fuse ? 0 : own_runs), wgs0);
    a.inv_runs[1] = inverse(n_tiles, wgs);
    const int bufs = rows > kChunk ? 2 : 1;
    auto passes = [&](auto more) {
      constexpr bool kMore = decltype(more)::value;
      if (fuse) hipLaunchKernelGGL((scores_bf16_kernel<0, true, kMore>), dim3((unsigned)wgs), dim3(kThreads), scores_lds_bytes(bufs, 0), st, a);
      else hipLaunchKernelGGL((scores_bf16_kernel<0, false, kMore>), dim3((unsigned)wgs0), dim3(kThreads), scores_lds_bytes(bufs, 0), st, a);
      if (a.merged) hipLaunchKernelGGL(scores_combine_kernel<true>, dim3((unsigned)((total_rows + 15) / 16)), dim3(256), 0, st, a);
      hipLaunchKernelGGL((scores_bf16_kernel<1, false, kMore>), dim3((unsigned)wgs), dim3(kThreads), scores_lds_bytes(bufs, 1), st, a);
    };
    if (tk > kTile) passes(std::true_type{});
    else passes(std::false_type{});
  } else {
    const dim3 grid(n_tiles, L->n_kv_heads, L->n_req), cgrid((unsigned)((total_rows + 15) / 16));
    a.merged = !f32_merges(n_tiles, (long long)n_tiles * L->n_kv_heads * L->n_req, (long long)L->max_q_len * G);
    auto launch = [&](auto dim) {
      constexpr int D = decltype(dim)::value;
      if (fuse) hipLaunchKernelGGL((scores_f32_kernel<0, D, true, false>), grid, dim3(256), 0, st, a);
      else hipLaunchKernelGGL((scores_f32_kernel<0, D, false, false>), grid, dim3(256), 0, st, a);
      if (a.merged) {
        hipLaunchKernelGGL(scores_combine_kernel<false>, cgrid, dim3(256), 0, st, a);
        hipLaunchKernelGGL((scores_f32_kernel<1, D, false, false>), grid, dim3(256), 0, st, a);
      } else {
        hipLaunchKernelGGL((scores_f32_kernel<1, D, false, true>), grid, dim3(256), 0, st, a);
      }
    };
    if (L->head_dim == 64) launch(std::integral_constant<int, 64>{});
    else launch(std::integral_constant<int, 128>{});
  }
  if (scores)
    hipLaunchKernelGGL(scores_head_sum_kernel, dim3((L->total_tokens + 255) / 256), dim3(256), 0, st, a, L->tok_chunk);
  A3_CHECK_LAUNCH("a3_question_scores");
  return A3_OK;
}


extern "C" a3_status a3_question_scores(const a3_layout *L, const void *q_question, const void *k_fused, float *scores,
                                        void *ws, size_t ws_bytes, void *stream) {
  return scores_launch(L, q_question, nullptr, const_cast<void *>(k_fused), scores, ws, ws_bytes, stream);
}

extern "C" a3_status a3_realign_scores(const a3_layout *L, const void *q_question, const void *k_cat, void *k_fused,
                                       float *scores, void *ws, size_t ws_bytes, void *stream) {
  if (k_cat == nullptr) return a3_fail(A3_ERR_INVALID_ARG, "a3_realign_scores: k_cat is NULL");
  if (!a3_aligned16(k_cat)) return a3_fail(A3_ERR_INVALID_ARG, "a3_realign_scores: tensors must be 16-byte aligned");
  return scores_launch(L, q_question, k_cat, k_fused, scores, ws, ws_bytes, stream);
}

// ---------------------------------------------------------------------------------------
// a3_question_scores for callers that cannot allocate (code under graph capture, serving loops that forbid
// it): the partial row statistics and per-head partial scores that a3_question_scores keeps in the caller's
// workspace live in a fixed array of the library's own device image instead.  One array per GPU, shared by
// every call on that GPU and holding the last call's contents; every word a call reads it has written itself
// before, so nothing has to be cleared between calls.
// ---------------------------------------------------------------------------------------
constexpr size_t kScratchBytes = (size_t)A3_SCORES_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::once_flag scratch_once[kMaxDevices];
void *scratch_ptr[kMaxDevices];          // device address of `scratch` on each GPU (the symbol itself is a host stand-in)
hipError_t scratch_err[kMaxDevices];
}  // namespace

extern "C" a3_status a3_question_scores_noalloc(const a3_layout *L, const void *q_question, const void *k_fused,
                                                float *scores, void *stream) {
  a3_status s = a3_check_layout(L, "a3_question_scores_noalloc", true);
  if (s != A3_OK) return s;
  A3_REQUIRE(q_question && k_fused && scores, A3_ERR_INVALID_ARG, "a3_question_scores_noalloc: NULL tensor");
  const size_t need = a3_scores_ws_bytes(L);
  A3_REQUIRE(need <= kScratchBytes, A3_ERR_WORKSPACE,
             "a3_question_scores_noalloc: this batch needs %zu bytes of scratch, the built-in array holds %zu "
             "(use a3_question_scores with a workspace)", need, kScratchBytes);
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return a3_fail(A3_ERR_HIP, "a3_question_scores_noalloc: hipGetDevice: %s", hipGetErrorString(e));
  A3_REQUIRE(dev >= 0 && dev < kMaxDevices, A3_ERR_UNSUPPORTED, "a3_question_scores_noalloc: device %d", dev);
  // once per device, with that device current: each GPU holds its own copy of the array at its own address
  std::call_once(scratch_once[dev], [dev]() {
    void *p = nullptr;
    scratch_err[dev] = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    scratch_ptr[dev] = scratch_err[dev] == hipSuccess ? p : nullptr;
  });
  if (scratch_err[dev] != hipSuccess || scratch_ptr[dev] == nullptr)
    return a3_fail(A3_ERR_HIP, "a3_question_scores_noalloc: hipGetSymbolAddress: %s", hipGetErrorString(scratch_err[dev]));
  return scores_launch(L, q_question, nullptr, const_cast<void *>(k_fused), scores, scratch_ptr[dev], kScratchBytes, stream);
}

// Eq. 3, first line, with the softmax of a question token taken over every key it sees: the context keys
// and the question keys up to itself (the literal reading of the equation's denominator).
extern "C" a3_status a3_question_scores_causal(const a3_layout *L, const void *q_question, const void *k_fused,
                                               float *scores, void *ws, size_t ws_bytes, void *stream) {
  A3_REQUIRE(scores != nullptr, A3_ERR_INVALID_ARG, "a3_question_scores_causal: scores is NULL");
  return scores_launch(L, q_question, nullptr, const_cast<void *>(k_fused), scores, ws, ws_bytes, stream, 1);
}

// Eviction extension: votes of the question window per KV head (same normalisation, no sum over KV heads).
extern "C" a3_status a3_window_votes(const a3_layout *L, const void *q_question, const void *k_fused, float *votes,
                                     void *ws, size_t ws_bytes, void *stream) {
  A3_REQUIRE(votes != nullptr, A3_ERR_INVALID_ARG, "a3_window_votes: votes is NULL");
  return scores_launch(L, q_question, nullptr, const_cast<void *>(k_fused), nullptr, ws, ws_bytes, stream, 1, votes);
}
