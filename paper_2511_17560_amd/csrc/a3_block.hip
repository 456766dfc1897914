// H(.) of Eq. 5: from the attention output of one layer to the input of the next, for the active rows.
//
//   r1 = r0 + O Wo^T                                   output projection, residual
//   r2 = r1 + (silu(n1 Wg^T) * (n1 Wu^T)) Wd^T         n1 = RMSNorm(r1; g_post): gated MLP, residual
//   x' = RMSNorm(r2; g_next)                           input norm of the next block (or the final norm)
//
// The paper names H in one clause (layer normalisation and feed-forward network applied to the attention
// output); this is the pre-norm block of the model families it evaluates.
//
// bf16: three launches of the row-tiled MFMA GEMM of a3_gemm_pp.h (weights [out, in], both operands
// reduction-contiguous) with the epilogues "add to the residual row", "silu(gate) * up" on the fp32 accumulators
// (gate and up of one output meet in one lane) and "store the partial product", and RMSNorm kernels.
// fp32: plain LDS-tiled FMA kernels (correctness configuration, not tuned).
#include "a3_internal.h"
#include "a3_gemm_pp.h"

namespace {

// EPI_RESID_SUM: EPI_RESID of a product whose reduction is split, the shares one after the other in one workgroup
enum { EPI_RESID = 0, EPI_SWIGLU = 1, EPI_PART = 2, EPI_RESID_SUM = 3 };

// ---------------------------------------------------------------------------------------
// RMSNorm: one wave per row.  A row of up to 16 vectors a lane (8192 bf16, 4096 fp32) is requested whole, with its gains,
// and stays in registers; a longer one is read twice, the second time from cache.  Bound by memory at many rows: 16448 rows x
// 4096 58.5 -> 41.3 us (6.5 TB/s), 5240 rows 19.7 -> 14.0, against a loop that waited for every vector in turn and read the row twice.
// ---------------------------------------------------------------------------------------
template <typename T, int N>                                    // N vectors a lane; 0: any number, in two passes
__global__ void __launch_bounds__(256)
rms_norm_kernel(const T *x, const int *__restrict__ in_idx, const T *__restrict__ g, float eps, T *out,
                const int *__restrict__ out_idx, int n_rows, int h) {   // x and out may be the same buffer
  constexpr int V = a3_elem<T>::kVec;
  const int lane = threadIdx.x & 63, row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n_rows) return;
  const int src = in_idx ? in_idx[row] : row, dst = out_idx ? out_idx[row] : row;
  const T *xr = x + (size_t)src * h;
  T *orow = out + (size_t)dst * h;
  typedef T vec_t __attribute__((ext_vector_type(V)));
  vec_t keep[N > 0 ? N : 1], w[N > 0 ? N : 1];
  float ss = 0.f;
  if constexpr (N > 0) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int v = min(lane + 64 * i, h / V - 1);              // past the end: the last vector, unused
      keep[i] = *reinterpret_cast<const vec_t *>(xr + v * V);
      w[i] = *reinterpret_cast<const vec_t *>(g + v * V);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
      if (lane + 64 * i >= h / V) break;
#pragma unroll
      for (int e = 0; e < V; ++e) { const float f = (float)keep[i][e]; ss = fmaf(f, f, ss); }
    }
  } else {
    for (int v = lane; v < h / V; v += 64) {
      const vec_t t = *reinterpret_cast<const vec_t *>(xr + v * V);
#pragma unroll
      for (int e = 0; e < V; ++e) { const float f = (float)t[e]; ss = fmaf(f, f, ss); }
    }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) ss += __shfl_xor(ss, o);
  const float inv = 1.0f / sqrtf(ss / (float)h + eps);
  auto write = [&](int v, const vec_t &t, const vec_t &gv) {
    vec_t y;
#pragma unroll
    for (int e = 0; e < V; ++e) y[e] = (T)((float)t[e] * inv * (float)gv[e]);
    *reinterpret_cast<vec_t *>(orow + v * V) = y;
  };
  if constexpr (N > 0) {
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (lane + 64 * i < h / V) write(lane + 64 * i, keep[i], w[i]);
  } else {
    for (int v = lane; v < h / V; v += 64)
      write(v, *reinterpret_cast<const vec_t *>(xr + v * V), *reinterpret_cast<const vec_t *>(g + v * V));
  }
}

// ---------------------------------------------------------------------------------------
// bf16 MFMA GEMM with the two epilogues
// ---------------------------------------------------------------------------------------
struct gemm_args {
  const bf16_t *a;       // activation rows [n_rows, K]
  int n_rows;
  const bf16_t *w0;      // [N, K]; EPI_SWIGLU: the gate weights
  const bf16_t *w1;      // EPI_SWIGLU: the up weights [N, K]
  bf16_t *out;           // EPI_RESID: [*, N], row out_idx[i] += product row i; EPI_SWIGLU: [n_rows, N]
  const int *out_idx;
  int K, N;
  float *part;           // EPI_PART: [splits, n_rows, N] partial products
  int splits;
  int n_wtiles, n_tok_tiles, group;
};

template <class P, int EPI>
__global__ void __launch_bounds__(512)
gemm_bf16_kernel(gemm_args a) {
  constexpr int IB = P::kIB, JB = P::kJB;
  // output features per workgroup and per wave group (EPI_SWIGLU: half 0 of a group's rows are gate rows, half 1 the up
  // rows of the same features)
  constexpr int kFeat = EPI == EPI_SWIGLU ? P::BM / 2 : P::BM, kFeatGrp = kFeat / 2;
  extern __shared__ __align__(16) unsigned char lds[];
  int wt, xt;
  if (!gemm_tile_of(a.n_wtiles, a.n_tok_tiles, a.group, blockIdx.x, wt, xt)) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, lg = lane >> 4, grp = wave >> 2, wn = wave & 3;

  // share y of the reduction, of a.splits nearly equal ones: its first slab and its slabs
  int s0 = 0, ns = a.K / 64;
  auto share = [&](int y) {
    const int all = a.K / 64, b = all / a.splits, rem = all - b * a.splits;
    s0 = y * b + min(y, rem);
    ns = b + (y < rem ? 1 : 0);
  };
  f32x4 acc[IB][JB];
  auto product = [&]() {
    P::mainloop(
        acc, lds, ns,
        [&](int r0) -> const char * {
          int q = 0, f;
          if (EPI == EPI_SWIGLU) P::row_of(r0 % (16 * IB), q, f);
          return reinterpret_cast<const char *>((q ? a.w1 : a.w0) + (size_t)wt * kFeat * a.K + 64 * s0);
        },
        [&](int r) -> uint32_t {
          int q, f;
          P::row_of(r % (16 * IB), q, f);
          f += (r / (16 * IB)) * kFeatGrp + (EPI == EPI_SWIGLU ? 0 : 8 * IB * q);
          return (uint32_t)min(f, a.N - 1 - wt * kFeat) * (uint32_t)a.K * 2u;
        },
        [&](int) -> const char * { return reinterpret_cast<const char *>(a.a + (size_t)xt * P::BN * a.K + 64 * s0); },
        [&](int r) -> uint32_t {
          return (uint32_t)min(r, a.n_rows - 1 - xt * P::BN) * (uint32_t)a.K * 2u;   // clamp: computed but never stored
        });
  };
  if constexpr (EPI == EPI_RESID_SUM) {
    f32x4 sum[IB][JB] = {};
    for (int y = 0; y < a.splits; ++y) {                         // the sums sum_norm_kernel forms, in its order
      share(y);
      product();
#pragma unroll
      for (int i = 0; i < IB; ++i)
#pragma unroll
        for (int j = 0; j < JB; ++j) sum[i][j] += acc[i][j];
      __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < IB; ++i)
#pragma unroll
      for (int j = 0; j < JB; ++j) acc[i][j] = sum[i][j];
  } else {
    if constexpr (EPI == EPI_PART) share(blockIdx.y);
    product();
  }

  // ---- epilogue: a lane holds L consecutive features of half 0 and of half 1 of one row; four lanes cover 64 or 128
  // consecutive bytes of a bf16 row
  constexpr int L = P::L;
  const int feat = wt * kFeat + grp * kFeatGrp;                  // first feature of the group
  if (feat >= a.N) return;
#pragma unroll
  for (int j = 0; j < JB; ++j) {
    const int tok = xt * P::BN + 16 * (JB * wn + j) + l16;
    float lo[L], hi[L];
    if constexpr (EPI == EPI_RESID || EPI == EPI_RESID_SUM) {
      const int row = tok < a.n_rows ? (a.out_idx ? a.out_idx[tok] : tok) : -1;
      bf16_t *p = a.out + (size_t)max(row, 0) * a.N + feat + L * lg;
      bf16x8 rl[L / 8], rh[L / 8];
      if (row >= 0) {
#pragma unroll
        for (int e = 0; e < L / 8; ++e) {
          rl[e] = *reinterpret_cast<const bf16x8 *>(p + 8 * e);
          rh[e] = *reinterpret_cast<const bf16x8 *>(p + 8 * IB + 8 * e);
        }
      }
      gemm_lane_values<IB, JB>(acc, j, lo, hi);
      if (row >= 0) {
#pragma unroll
        for (int e = 0; e < L / 8; ++e) {
          bf16x8 vl, vh;
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            vl[u] = a3_f2bf(a3_bf2f(rl[e][u]) + lo[8 * e + u]);
            vh[u] = a3_f2bf(a3_bf2f(rh[e][u]) + hi[8 * e + u]);
          }
          *reinterpret_cast<bf16x8 *>(p + 8 * e) = vl;
          *reinterpret_cast<bf16x8 *>(p + 8 * IB + 8 * e) = vh;
        }
      }
    } else if constexpr (EPI == EPI_SWIGLU) {
      gemm_lane_values<IB, JB>(acc, j, lo, hi);                  // gate, up
      if (tok < a.n_rows) {
        bf16_t *p = a.out + (size_t)tok * a.N + feat + L * lg;
#pragma unroll
        for (int e = 0; e < L; e += 8) {
          bf16x8 v;
#pragma unroll
          for (int u = 0; u < 8; ++u) v[u] = a3_f2bf(lo[e + u] / (1.0f + __expf(-lo[e + u])) * hi[e + u]);
          *reinterpret_cast<bf16x8 *>(p + e) = v;
        }
      }
    } else {
      gemm_lane_values<IB, JB>(acc, j, lo, hi);
      if (tok < a.n_rows) {
        float *p = a.part + ((size_t)blockIdx.y * a.n_rows + tok) * a.N + feat + L * lg;
#pragma unroll
        for (int e = 0; e < L; e += 4) {
          *reinterpret_cast<f32x4 *>(p + e) = f32x4{lo[e], lo[e + 1], lo[e + 2], lo[e + 3]};
          *reinterpret_cast<f32x4 *>(p + 8 * IB + e) = f32x4{hi[e], hi[e + 1], hi[e + 2], hi[e + 3]};
        }
      }
    }
  }
}

// Rows of a product whose reduction was split: residual row += the partial rows in share order (one rounding), then the
// RMSNorm of the new row.  One workgroup per row; the row stays in registers between the two (up to 8 vectors a thread).
// SP = 0 shares: the residual row has its product already.
// SP (2, 4 or 8) is a constant so that the loads of all shares of a vector are on their way together: the tail of a block of
// 3584 x 18944, 512 rows, 259 -> 252 us, 64 rows 121 -> 117 (4096 x 14336: 212 -> 209, 103 -> 99).
constexpr int kSumNormThreads = 256, kSumNormVecs = 8;
template <int SP>
__global__ void __launch_bounds__(kSumNormThreads)
sum_norm_kernel(const float *__restrict__ part, int n_rows, bf16_t *resid, const int *__restrict__ idx,
                const bf16_t *__restrict__ g, float eps, bf16_t *out, const int *__restrict__ out_idx, int h) {
  __shared__ float red[kSumNormThreads / 64];
  const int i = blockIdx.x, row = idx ? idx[i] : i, dst = out_idx ? out_idx[i] : i;
  bf16_t *rr = resid + (size_t)row * h;
  float x[kSumNormVecs][8], ss = 0.f;
#pragma unroll
  for (int v = 0; v < kSumNormVecs; ++v) {
    const int c = (v * kSumNormThreads + threadIdx.x) * 8;
    if (c >= h) break;
    const bf16x8 r = *reinterpret_cast<const bf16x8 *>(rr + c);
    float t[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) t[e] = 0.f;
    f32x4 a[SP > 0 ? SP : 1], b[SP > 0 ? SP : 1];
#pragma unroll
    for (int s = 0; s < SP; ++s) {
      const float *p = part + ((size_t)s * n_rows + i) * h + c;
      a[s] = *reinterpret_cast<const f32x4 *>(p);
      b[s] = *reinterpret_cast<const f32x4 *>(p + 4);
    }
#pragma unroll
    for (int s = 0; s < SP; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e) { t[e] += a[s][e]; t[4 + e] += b[s][e]; }
    bf16x8 y;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      y[e] = SP > 0 ? a3_f2bf(a3_bf2f(r[e]) + t[e]) : r[e];
      x[v][e] = a3_bf2f(y[e]);
      ss = fmaf(x[v][e], x[v][e], ss);
    }
    if (SP > 0) *reinterpret_cast<bf16x8 *>(rr + c) = y;
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) ss += __shfl_xor(ss, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  ss = (red[0] + red[1]) + (red[2] + red[3]);
  const float inv = 1.0f / sqrtf(ss / (float)h + eps);
#pragma unroll
  for (int v = 0; v < kSumNormVecs; ++v) {
    const int c = (v * kSumNormThreads + threadIdx.x) * 8;
    if (c >= h) break;
    const bf16x8 w = *reinterpret_cast<const bf16x8 *>(g + c);
    bf16x8 y;
#pragma unroll
    for (int e = 0; e < 8; ++e) y[e] = a3_f2bf(x[v][e] * inv * a3_bf2f(w[e]));
    *reinterpret_cast<bf16x8 *>(out + (size_t)dst * h + c) = y;
  }
}

// ---------------------------------------------------------------------------------------
// fp32 GEMM with the same two epilogues (correctness configuration)
// ---------------------------------------------------------------------------------------
struct gemm_args_f32 {
  const float *a;
  const int *a_idx;
  int n_rows;
  const float *w0, *w1;
  float *out;
  const int *out_idx;
  int K, N;
};

template <int EPI>
__global__ void __launch_bounds__(256)
gemm_f32_kernel(gemm_args_f32 a) {
  constexpr int R = 16, F = 64, BK = 32;
  __shared__ float As[R][BK + 1];
  __shared__ float W0s[F][BK + 1];
  __shared__ float W1s[EPI == EPI_SWIGLU ? F : 1][BK + 1];
  const int f0 = blockIdx.x * F, m0 = blockIdx.y * R;
  const int tid = threadIdx.x, ty = tid >> 4, tx = tid & 15;
  float acc0[4] = {0.f, 0.f, 0.f, 0.f}, acc1[4] = {0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < a.K; k0 += BK) {
    for (int i = tid; i < R * BK; i += 256) {
      const int r = i / BK, c = i % BK, m = m0 + r;
      float v = 0.f;
      if (m < a.n_rows && k0 + c < a.K) v = a.a[(size_t)(a.a_idx ? a.a_idx[m] : m) * a.K + k0 + c];
      As[r][c] = v;
    }
    for (int i = tid; i < F * BK; i += 256) {
      const int r = i / BK, c = i % BK;
      const bool ok = f0 + r < a.N && k0 + c < a.K;
      W0s[r][c] = ok ? a.w0[(size_t)(f0 + r) * a.K + k0 + c] : 0.f;
      if (EPI == EPI_SWIGLU) W1s[r][c] = ok ? a.w1[(size_t)(f0 + r) * a.K + k0 + c] : 0.f;
    }
    __syncthreads();
    for (int c = 0; c < BK; ++c) {
      const float x = As[ty][c];
#pragma unroll
      for (int f = 0; f < 4; ++f) {
        acc0[f] = fmaf(x, W0s[tx + 16 * f][c], acc0[f]);
        if (EPI == EPI_SWIGLU) acc1[f] = fmaf(x, W1s[tx + 16 * f][c], acc1[f]);
      }
    }
    __syncthreads();
  }
  const int m = m0 + ty;
  if (m >= a.n_rows) return;
  const int orow = a.out_idx ? a.out_idx[m] : m;
#pragma unroll
  for (int f = 0; f < 4; ++f) {
    const int feat = f0 + tx + 16 * f;
    if (feat >= a.N) continue;
    float *p = a.out + (size_t)orow * a.N + feat;
    if (EPI == EPI_RESID) *p += acc0[f];
    else *p = acc0[f] / (1.0f + expf(-acc0[f])) * acc1[f];
  }
}

template <class P, int EPI>
a3_status gemm_bf16_launch_in(gemm_args a, hipStream_t st, const char *who) {
  auto kern = gemm_bf16_kernel<P, EPI>;
  static a3_once_per_device lds_once;
  if (a3_once(lds_once, [&]() { return hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)P::kLdsBytes); }) != hipSuccess)
    return a3_fail(A3_ERR_HIP, "%s: cannot raise the dynamic LDS limit", who);
  const int feat = EPI == EPI_SWIGLU ? P::BM / 2 : P::BM;
  a.n_wtiles = (a.N + feat - 1) / feat;
  a.n_tok_tiles = (a.n_rows + P::BN - 1) / P::BN;
  a.group = gemm_tile_group(a.n_wtiles, a.n_tok_tiles);
  hipLaunchKernelGGL(kern, dim3(gemm_tile_grid(a.n_wtiles, a.n_tok_tiles), EPI == EPI_PART ? a.splits : 1), dim3(512),
                     P::kLdsBytes, st, a);
  A3_CHECK_LAUNCH(who);
  return A3_OK;
}

template <int EPI>
a3_status gemm_bf16_launch(const gemm_args &a, int tile, hipStream_t st, const char *who) {
  return gemm_with_tile(tile, [&](auto t) -> a3_status { return gemm_bf16_launch_in<decltype(t), EPI>(a, st, who); });
}

int tile_of_knob(int tile) {
  const int t = gemm_tile_of_knob(a3_knob(A3_KNOB_GEMM_TB));
  return t >= 0 ? t : tile;
}

// Tile and split of a residual GEMM of H(.): by its shape alone, so that a row's sums do not depend on the workspace.
constexpr int kMaxSplits = 8, kSumNormMaxHidden = 8 * kSumNormThreads * kSumNormVecs;
gemm_tile_choice residual_tile(int h, int n_rows, int K) { return gemm_choose_tile(h, n_rows, K / 64, h <= kSumNormMaxHidden ? kMaxSplits : 1); }
// fp32 partial results of a residual GEMM whose reduction is split (0: it is not)
size_t split_bytes(const gemm_tile_choice &c, int n_rows, int h) {
  return c.splits > 1 ? (size_t)c.splits * n_rows * h * sizeof(float) : 0;
}

template <int EPI>
a3_status gemm_f32_launch(const gemm_args_f32 &a, hipStream_t st, const char *who) {
  dim3 grid((a.N + 63) / 64, (a.n_rows + 15) / 16);
  hipLaunchKernelGGL(gemm_f32_kernel<EPI>, grid, dim3(256), 0, st, a);
  A3_CHECK_LAUNCH(who);
  return A3_OK;
}

a3_status rms_norm_launch(const a3_layout *L, const void *x, const int *in_idx, const void *g, float eps, void *out,
                          const int *out_idx, int n_rows, hipStream_t st, const char *who) {
  const dim3 grid((n_rows + 3) / 4);
  auto launch = [&](auto elem) {
    typedef decltype(elem) T;
    const int n = (L->hidden / a3_elem<T>::kVec + 63) / 64;     // vectors a lane
    auto kern = n <= 2 ? rms_norm_kernel<T, 2> : n <= 4 ? rms_norm_kernel<T, 4> : n <= 8 ? rms_norm_kernel<T, 8>
              : n <= 16 ? rms_norm_kernel<T, 16> : rms_norm_kernel<T, 0>;
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, (const T *)x, in_idx, (const T *)g, eps, (T *)out, out_idx, n_rows, L->hidden);
  };
  if (L->dtype == A3_BF16) launch(bf16_t{});
  else launch(0.f);
  A3_CHECK_LAUNCH(who);
  return A3_OK;
}

size_t elem_bytes(const a3_layout *L) { return L->dtype == A3_BF16 ? 2 : 4; }

// without partial results
size_t tail_base_bytes(const a3_layout *L, int ffn, int n_rows) {
  const size_t e = elem_bytes(L);
  return a3_align_up((size_t)n_rows * L->hidden * e, 256) + a3_align_up((size_t)n_rows * ffn * e, 256) + 256;
}

}  // namespace

extern "C" size_t a3_block_tail_ws_bytes(const a3_layout *L, int ffn, int n_rows) {
  if (L == nullptr || ffn <= 0 || n_rows < 0 || L->hidden <= 0) return 0;
  if (L->dtype != A3_BF16 && L->dtype != A3_F32) return 0;
  size_t part = 0;
  if (L->dtype == A3_BF16 && n_rows > 0) {
    const size_t p0 = split_bytes(residual_tile(L->hidden, n_rows, L->n_q_heads * L->head_dim), n_rows, L->hidden);
    const size_t p1 = split_bytes(residual_tile(L->hidden, n_rows, ffn), n_rows, L->hidden);
    part = p0 > p1 ? p0 : p1;
  }
  return tail_base_bytes(L, ffn, n_rows) + a3_align_up(part, 256);
}

extern "C" a3_status a3_rms_norm(const a3_layout *L, const void *x, const int *row_idx, int n_rows, const void *g,
                                 float eps, void *out, void *stream) {
  a3_status s = a3_check_layout(L, "a3_rms_norm", false);
  if (s != A3_OK) return s;
  A3_REQUIRE(n_rows >= 0 && n_rows <= L->total_tokens, A3_ERR_INVALID_ARG, "a3_rms_norm: n_rows %d outside [0, %d]",
             n_rows, L->total_tokens);
  if (n_rows == 0) return A3_OK;
  A3_REQUIRE(x && g && out, A3_ERR_INVALID_ARG, "a3_rms_norm: NULL tensor");
  A3_REQUIRE(a3_aligned16(x) && a3_aligned16(g) && a3_aligned16(out), A3_ERR_INVALID_ARG,
             "a3_rms_norm: tensors must be 16-byte aligned");
  A3_REQUIRE(eps >= 0.f, A3_ERR_INVALID_ARG, "a3_rms_norm: eps %g is negative", (double)eps);
  A3_REQUIRE(L->hidden % 8 == 0, A3_ERR_UNSUPPORTED, "a3_rms_norm: needs hidden %% 8 == 0, got %d", L->hidden);
  return rms_norm_launch(L, x, row_idx, g, eps, out, row_idx, n_rows, (hipStream_t)stream, "a3_rms_norm");
}

extern "C" a3_status a3_block_tail(const a3_layout *L, const void *attn_out, const int *act_idx, int n_act,
                                   const a3_block_weights *w, void *resid, void *hidden_next, void *ws,
                                   size_t ws_bytes, void *stream) {
  a3_status s = a3_check_layout(L, "a3_block_tail", false);
  if (s != A3_OK) return s;
  A3_REQUIRE(n_act >= 0 && n_act <= L->total_tokens, A3_ERR_INVALID_ARG, "a3_block_tail: n_act %d outside [0, %d]",
             n_act, L->total_tokens);
  if (n_act == 0) return A3_OK;
  A3_REQUIRE(w != nullptr, A3_ERR_INVALID_ARG, "a3_block_tail: weights are NULL");
  A3_REQUIRE(attn_out && resid && hidden_next, A3_ERR_INVALID_ARG, "a3_block_tail: NULL tensor");
  A3_REQUIRE(w->wo && w->g_post && w->w_gate && w->w_up && w->w_down && w->g_next, A3_ERR_INVALID_ARG,
             "a3_block_tail: a weight is NULL");
  const void *ptrs[] = {attn_out, resid, hidden_next, w->wo, w->g_post, w->w_gate, w->w_up, w->w_down, w->g_next};
  for (const void *p : ptrs)
    A3_REQUIRE(a3_aligned16(p), A3_ERR_INVALID_ARG, "a3_block_tail: tensors must be 16-byte aligned");
  A3_REQUIRE(w->ffn > 0, A3_ERR_INVALID_ARG, "a3_block_tail: ffn %d", w->ffn);
  A3_REQUIRE(w->eps >= 0.f, A3_ERR_INVALID_ARG, "a3_block_tail: eps %g is negative", (double)w->eps);
  A3_REQUIRE(L->hidden % 8 == 0, A3_ERR_UNSUPPORTED, "a3_block_tail: needs hidden %% 8 == 0, got %d", L->hidden);
  const int h = L->hidden, f = w->ffn, qd = L->n_q_heads * L->head_dim;
  if (L->dtype == A3_BF16)
    A3_REQUIRE(h % 128 == 0 && f % 64 == 0 && qd % 32 == 0, A3_ERR_UNSUPPORTED,
               "a3_block_tail: bf16 needs hidden %% 128 == 0, ffn %% 64 == 0, heads x head_dim %% 32 == 0 (got %d, %d, %d)",
               h, f, qd);
  A3_REQUIRE(ws != nullptr, A3_ERR_WORKSPACE, "a3_block_tail: workspace is NULL");
  const size_t need = tail_base_bytes(L, f, n_act);
  A3_REQUIRE(ws_bytes >= need, A3_ERR_WORKSPACE, "a3_block_tail: workspace %zu bytes, need %zu", ws_bytes, need);
  hipStream_t st = (hipStream_t)stream;
  a3_ws_cursor cur(ws, ws_bytes);
  void *normed = cur.take((size_t)n_act * h * elem_bytes(L));
  void *act = cur.take((size_t)n_act * f * elem_bytes(L));

  if (L->dtype == A3_BF16) {
    // A residual GEMM and the norm behind it: in one pass over the reduction and a norm kernel, or - where too few tiles
    // would be left to fill the chip - with the reduction split over workgroups and a kernel that sums, adds and norms.
    // A workspace without room for the partial results gets the same sums from workgroups that form all shares, about as fast as
    // an unsplit product would be (4096 x 14336: 64 rows 219 us, 206 unsplit and 105 with room; 1344 rows 490, 490 and 470).
    auto resid_norm = [&](const bf16_t *x, const void *weight, int K, const void *g, bf16_t *out, const int *out_idx) -> a3_status {
      gemm_args a{x, n_act, (const bf16_t *)weight, nullptr, (bf16_t *)resid, act_idx, K, h, nullptr, 1, 0, 0, 0};
      gemm_tile_choice c = residual_tile(h, n_act, K);
      if (a3_knob(A3_KNOB_GEMM_TB) >= 0) c = {tile_of_knob(c.tile), 1};
      a3_status e;
      if (c.splits == 1) {
        if ((e = gemm_bf16_launch<EPI_RESID>(a, c.tile, st, "a3_block_tail")) != A3_OK) return e;
        return rms_norm_launch(L, resid, act_idx, g, w->eps, out, out_idx, n_act, st, "a3_block_tail");
      }
      a.splits = c.splits;
      const bool room = ws_bytes - need >= split_bytes(c, n_act, h);
      if (room) {
        a.part = (float *)((char *)ws + a3_align_up(cur.off, 256));
        e = gemm_bf16_launch<EPI_PART>(a, c.tile, st, "a3_block_tail");
      } else {
        // (tiles that leave room in the registers for a second set of accumulators)
        switch (gemm_choose_tile(h, n_act, K / 64, 1, GEMM_256x128).tile) {
          case GEMM_256x128: e = gemm_bf16_launch_in<gemm_pl<8, 2, 3>, EPI_RESID_SUM>(a, st, "a3_block_tail"); break;
          case GEMM_128x192: e = gemm_bf16_launch_in<gemm_pl<4, 3, 4>, EPI_RESID_SUM>(a, st, "a3_block_tail"); break;
          case GEMM_128x128: e = gemm_bf16_launch_in<gemm_pl<4, 2, 5>, EPI_RESID_SUM>(a, st, "a3_block_tail"); break;
          default: e = gemm_bf16_launch_in<gemm_pl<4, 1, 6>, EPI_RESID_SUM>(a, st, "a3_block_tail");
        }
      }
      if (e != A3_OK) return e;
      const int sp = room ? c.splits : 0;
      auto sum_norm = sp == 0 ? sum_norm_kernel<0> : sp == 2 ? sum_norm_kernel<2> : sp == 4 ? sum_norm_kernel<4> : sum_norm_kernel<8>;
      static_assert(kMaxSplits == 8, "splits are 2, 4 or 8");
      hipLaunchKernelGGL(sum_norm, dim3(n_act), dim3(kSumNormThreads), 0, st, a.part, n_act, (bf16_t *)resid,
                         act_idx, (const bf16_t *)g, w->eps, out, out_idx, h);
      A3_CHECK_LAUNCH("a3_block_tail");
      return A3_OK;
    };
    // r1 = r0 + O Wo^T, n1 = RMSNorm(r1; g_post) (compact)
    if ((s = resid_norm((const bf16_t *)attn_out, w->wo, qd, w->g_post, (bf16_t *)normed, nullptr)) != A3_OK) return s;
    // act = silu(n1 Wg^T) * (n1 Wu^T)
    gemm_args a{(const bf16_t *)normed, n_act, (const bf16_t *)w->w_gate, (const bf16_t *)w->w_up, (bf16_t *)act, nullptr, h, f, nullptr, 1, 0, 0, 0};
    if ((s = gemm_bf16_launch<EPI_SWIGLU>(a, tile_of_knob(gemm_choose_tile(2 * f, n_act, h / 64, 1).tile), st, "a3_block_tail")) != A3_OK) return s;
    // r2 = r1 + act Wd^T, x' = RMSNorm(r2; g_next) at the rows' own places
    return resid_norm((const bf16_t *)act, w->w_down, f, w->g_next, (bf16_t *)hidden_next, act_idx);
  }
  gemm_args_f32 a{(const float *)attn_out, nullptr, n_act, (const float *)w->wo, nullptr, (float *)resid, act_idx, qd, h};
  if ((s = gemm_f32_launch<EPI_RESID>(a, st, "a3_block_tail")) != A3_OK) return s;
  if ((s = rms_norm_launch(L, resid, act_idx, w->g_post, w->eps, normed, nullptr, n_act, st, "a3_block_tail")) != A3_OK)
    return s;
  gemm_args_f32 u{(const float *)normed, nullptr, n_act, (const float *)w->w_gate, (const float *)w->w_up, (float *)act, nullptr, h, f};
  if ((s = gemm_f32_launch<EPI_SWIGLU>(u, st, "a3_block_tail")) != A3_OK) return s;
  gemm_args_f32 b{(const float *)act, nullptr, n_act, (const float *)w->w_down, nullptr, (float *)resid, act_idx, f, h};
  if ((s = gemm_f32_launch<EPI_RESID>(b, st, "a3_block_tail")) != A3_OK) return s;
  return rms_norm_launch(L, resid, act_idx, w->g_next, w->eps, hidden_next, act_idx, n_act, st, "a3_block_tail");
}
