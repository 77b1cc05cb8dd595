// Weight re-packing, normalisation and the skinny bf16 GEMM with fused epilogues
// (QKV + rotary + KV append, residual add, GELU, SwiGLU, vocabulary argmax).
#include "gelu_poly.h"
#include "mfma_common.h"

#include <algorithm>
#include <type_traits>

#ifndef PD_GEMM_EPI   // ---- common part: weight packing, norm kernel -------------------------------

// ---------------------------------------------------------------------------
// weight re-packing (runs once, in pd_create)
//   mode 0: row(n) = n
//   mode 1: rotary QKV.  Inside the Q and K sections every 16-row tile holds 8 low
//           dims and their rotation partners: tile th of head h, packed row m:
//           dim = th*8 + (m & 7) + (m >= 8 ? hd/2 : 0).  V section: identity.
//   mode 2: SwiGLU.  Tile t holds gate rows t*8..t*8+7 (from src) then up rows
//           t*8..t*8+7 (from src2).
// ---------------------------------------------------------------------------
__global__ void k_pack_weight(bf16_t *dst, const bf16_t *src, const bf16_t *src2, int N_src,
                              int N_pad, int K, int mode, int d, int hd) {
  size_t gran = (size_t)blockIdx.x * blockDim.x + threadIdx.x;   // 16-byte granule index
  int KT = K >> 5;
  size_t total = (size_t)(N_pad >> 4) * KT * 64;
  if (gran >= total) return;
  int lane = gran & 63;
  size_t frag = gran >> 6;
  int kt = frag % KT, nt = frag / KT;
  int m = lane & 15, g = lane >> 4;
  int n = nt * 16 + m;
  const bf16_t *row = nullptr;
  if (mode == 0) {
    if (n < N_src) row = src + (size_t)n * K;
  } else if (mode == 1) {
    if (n < 2 * d) {
      int sec = n / d, nl = n % d, h = nl / hd, th = (nl % hd) >> 4;
      int dim = th * 8 + (m & 7) + (m >= 8 ? hd / 2 : 0);
      row = src + ((size_t)sec * d + h * hd + dim) * K;
    } else {
      row = src + (size_t)n * K;
    }
  } else {
    int f = nt * 8 + (m & 7);
    row = (m < 8 ? src : src2) + (size_t)f * K;
  }
  uint4 v = make_uint4(0, 0, 0, 0);
  if (row) v = *(const uint4 *)(row + kt * 32 + g * 8);
  ((uint4 *)dst)[gran] = v;
}

static int pack(bf16_t *dst, const void *src, const void *src2, int N_src, int N_pad, int K,
                int mode, int d, int hd, hipStream_t s) {
  size_t total = (size_t)(N_pad / 16) * (K / 32) * 64;
  hipLaunchKernelGGL(k_pack_weight, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, dst,
                     (const bf16_t *)src, (const bf16_t *)src2, N_src, N_pad, K, mode, d, hd);
  PD_CHECK_HIP(hipGetLastError());
  return PD_OK;
}

int mfma_pack_matrix(bf16_t *dst, const void *src, int N, int K, hipStream_t s) {
  return pack(dst, src, nullptr, N, (N + 15) / 16 * 16, K, 0, 0, 0, s);
}

int mfma_pack_weights(pd_ctx *c, hipStream_t s) {
  const pd_config &g = c->cfg;
  int d = g.d_model, ff = g.d_ff, hd = g.head_dim, rc;
  for (int l = 0; l < g.n_layer; ++l) {
    LayerPtrs &lp = c->layers[l];
    if ((rc = pack(lp.p_wqkv, lp.wqkv, nullptr, 3 * d, 3 * d, d, g.pos_kind == 1 ? 1 : 0, d, hd, s))) return rc;
    if ((rc = pack(lp.p_wo, lp.wo, nullptr, d, d, d, 0, d, hd, s))) return rc;
    if (g.ffn_kind == 1) {
      if ((rc = pack(lp.p_w1, lp.w1, lp.w_up, ff, 2 * ff, d, 2, d, hd, s))) return rc;
    } else {
      if ((rc = pack(lp.p_w1, lp.w1, nullptr, ff, ff, d, 0, d, hd, s))) return rc;
    }
    if ((rc = pack(lp.p_w2, lp.w2, nullptr, d, d, ff, 0, d, hd, s))) return rc;
  }
  return pack(c->p_lm_head, c->lm_head, nullptr, g.vocab, c->vocab_pad, d, 0, d, hd, s);
}

// ---------------------------------------------------------------------------
// c1[n] = sum_k W[n][k] gain[k], c2[n] = sum_k W[n][k] bias[k] over a packed weight matrix (columns n
// in packed order): what a projection needs to finish a norm in its epilogue when it is fed
// gain * x instead of the normalised row.  One wave per 16-column tile; runs once, in pd_create.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_norm_fold(float *c1, float *c2, const bf16_t *Wp, const float *gain,
                                                  const float *bias, int KT) {
  const int nt = blockIdx.x, lane = threadIdx.x, m = lane & 15, g = lane >> 4;
  const uint4 *wp = (const uint4 *)Wp + (size_t)nt * KT * 64 + lane;
  float s1 = 0.f, s2 = 0.f;
  for (int kt = 0; kt < KT; ++kt) {
    Frag w;
    w.u = wp[(size_t)kt * 64];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int k = kt * 32 + g * 8 + e;
      const float wv = bf16_to_f32(w.h[e]);
      s1 = fmaf(wv, gain[k], s1);
      if (bias) s2 = fmaf(wv, bias[k], s2);
    }
  }
  s1 = fold32(fold16(s1, Add()), Add());
  s2 = fold32(fold16(s2, Add()), Add());
  if (g == 0) {
    c1[nt * 16 + m] = s1;
    if (c2) c2[nt * 16 + m] = s2;
  }
}

int mfma_fold(float *c1, float *c2, const bf16_t *Wp, const float *gain, const float *bias, int n_out, int K,
              hipStream_t s) {
  hipLaunchKernelGGL(k_norm_fold, dim3(n_out / 16), dim3(64), 0, s, c1, bias ? c2 : nullptr, Wp, gain, bias, K / 32);
  PD_CHECK_HIP(hipGetLastError());
  return PD_OK;
}

int mfma_fold_norms(pd_ctx *c, hipStream_t s) {
  const pd_config &g = c->cfg;
  const int n_out = (g.ffn_kind == 1 ? 2 : 1) * g.d_ff;
  int rc;
  for (int l = 0; l < g.n_layer; ++l) {
    LayerPtrs &lp = c->layers[l];
    if ((rc = mfma_fold(lp.c1, lp.c2, lp.p_w1, lp.n2g, g.norm_kind == 0 ? lp.n2b : nullptr, n_out, g.d_model, s))) return rc;
    if ((rc = mfma_fold(lp.q1, lp.q2, lp.p_wqkv, lp.n1g, g.norm_kind == 0 ? lp.n1b : nullptr, 3 * g.d_model, g.d_model, s))) return rc;
  }
  return PD_OK;
}

// ---------------------------------------------------------------------------
// norm -> bf16 activations.  One block per row; rows without a token become zero.
// The row, its pending slices, gain and bias are read once into registers, every request in flight before anything is waited
// for, so that the kernel costs one memory round trip plus one block reduction (sum and sum of squares together: the variance
// is E[x^2] - mean^2, as in the projections that finish a norm).  The completed row is stored behind the last use.  With
// requests under conditions and a store between the slices' halves it took four round trips: 72 rows of width 1024, four
// slices 3.84 -> 3.32 us.
// Which of a launch's rows a block takes, P blocks to a tile of 16 rows: work-groups go to the XCDs round-robin, and the rows of
// a tile share the lines of the activations (16 bytes of every row in turn), which only meet in an L2 cache when one XCD writes
// them all.  Tiles beyond the last eight stay in order.  4096 rows of width 2048: gathered 46 -> 32 us, with two slices 41.3 -> 38.5, one 35.6 -> 34.6.
template <int P>
__device__ __forceinline__ int tile_on_one_xcd(int b, int R) {
  const int full = (((R + 15) >> 4) & ~7) * P, i = b >> 3;
  return b < full ? ((i / P) * 8 + (b & 7)) * P + i % P : b;
}

// EMB: the row is not read from x but gathered from the embedding tables (first norm of a step:
// x = E_tok[token] (+ E_pos[position]), zero for rows without a token) and written to x.
template <int NG, int NP, bool EMB>     // 8-value granules per thread: d <= 2048 * NG; NP pending slices
__global__ __launch_bounds__(256) void k_norm_bf16(const int32_t *flags, const void *src1, const void *src2, const float *g,
                                                   const float *b, int d, int R, int rows_pad, int kind,
                                                   const bf16_t *tok_emb, const bf16_t *pos_emb, float eps, float *xw,
                                                   bf16_t *xn, bf16_t *xn_lo) {
  // (the first 14 words arrive in registers: what the first requests need)
  const float *x = (const float *)src1, *ypart = (const float *)src2;            // rows and pending slices
  const size_t part_stride = (size_t)rows_pad * d;
  const int32_t *tok = (const int32_t *)src1, *pos = (const int32_t *)src2;      // EMB: token and position of a row
  const int r = tile_on_one_xcd<16>(blockIdx.x, R);
  int fl = 0;
  if (EMB) fl = r < R ? flags[r] : 0;
  // Every request goes out before anything is waited for, at clamped places and without a branch (a load under a condition
  // is waited for where its branch ends: four round trips instead of one).
  const float *bias = kind == 0 && b ? b : g;
  floatx4 xv[NG][2], tg[NG][2], tb[NG][2], y[NG][2][NP > 0 ? NP : 1];
  Frag et[EMB ? NG : 1], ep[EMB ? NG : 1];
  const bf16_t *te = nullptr, *pe = nullptr;
  if (EMB) {
    // (rows without a token hold an older one; the tables cover the padded rows)
    const int tk = tok[r], ps = pos[r];
    const bool has = fl & ROW_VALID;
    te = tok_emb + (has ? (size_t)tk * d : 0);
    pe = pos_emb ? pos_emb + (has ? (size_t)ps * d : 0) : te;
  }
  const float *xr = EMB ? nullptr : x + (size_t)r * d, *yr = NP > 0 ? ypart + (size_t)r * d : nullptr;
#pragma unroll
  for (int i = 0; i < NG; ++i) {
    const int c = min((int)(threadIdx.x + i * 256) * 8, d - 8);
    if (EMB) { et[i].u = *(const uint4 *)(te + c); ep[i].u = *(const uint4 *)(pe + c); }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (!EMB) xv[i][h] = *(const floatx4 *)(xr + c + 4 * h);
#pragma unroll
      for (int pp = 0; pp < NP; ++pp) y[i][h][pp] = *(const floatx4 *)(yr + pp * part_stride + c + 4 * h);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      tg[i][h] = *(const floatx4 *)(g + c + 4 * h);
      tb[i][h] = *(const floatx4 *)(bias + c + 4 * h);
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  if (!EMB) fl = r < R ? flags[r] : 0;
  const bool valid = fl & ROW_VALID;
  float v[NG][8];
#pragma unroll
  for (int i = 0; i < NG; ++i) {
    const bool in = (int)(threadIdx.x + i * 256) * 8 < d;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (EMB)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          xv[i][h][e] = valid ? bf16_to_f32(et[i].h[4 * h + e]) + (pos_emb ? bf16_to_f32(ep[i].h[4 * h + e]) : 0.f) : 0.f;
      // the pending split-K slices of the last projection
#pragma unroll
      for (int pp = 0; pp < NP; ++pp) xv[i][h] += y[i][h][pp];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[i][4 * h + e] = in ? xv[i][h][e] : 0.f;
    }
  }
  float s = 0.f, q = 0.f;
#pragma unroll
  for (int i = 0; i < NG; ++i)
#pragma unroll
    for (int e = 0; e < 8; ++e) { s += v[i][e]; q += v[i][e] * v[i][e]; }
  // one reduction for both sums (values beyond d are zero)
  s = fold_wave(s, Add());
  q = fold_wave(q, Add());
  __shared__ float2 sh2[4];
  if ((threadIdx.x & 63) == 0) sh2[threadIdx.x >> 6] = make_float2(s, q);
  __syncthreads();
  s = (sh2[0].x + sh2[1].x) + (sh2[2].x + sh2[3].x);
  q = (sh2[0].y + sh2[1].y) + (sh2[2].y + sh2[3].y);
  float mean = kind == 0 ? s / d : 0.f;
  float rstd = rsqrtf(fmaxf(q / d - mean * mean, 0.f) + eps);
#pragma unroll
  for (int i = 0; i < NG; ++i) {
    int c = (threadIdx.x + i * 256) * 8;
    if (c >= d) continue;
    float y[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float bias_e = kind == 0 && b ? tb[i][e >> 2][e & 3] : 0.f;
      y[e] = valid ? (v[i][e] - mean) * rstd * tg[i][e >> 2][e & 3] + bias_e : 0.f;
    }
    store8_split(xn, xn_lo, act_off(r, c, d), y);
    if ((EMB || NP > 0) && r < R) {
      *(float4 *)(xw + (size_t)r * d + c) = make_float4(v[i][0], v[i][1], v[i][2], v[i][3]);
      *(float4 *)(xw + (size_t)r * d + c + 4) = make_float4(v[i][4], v[i][5], v[i][6], v[i][7]);
    }
  }
}

// The same for launches of many rows (the context pass): a wave per row, up to four rows per block.  Lane l takes the
// 8-value granules l, l + 64, ... of its row, and the two sums are wave reductions (no barrier, no LDS).  A batch of
// granules, slices among them, is requested before any of it is waited for; gain and bias, up to width 2048, under the sums,
// beyond (a lane's registers are full) when they are used.  Requests under conditions, the completed halves stored between
// them, and four granules for every width up to 2048 took 6.2 us (192 rows of width 768, four slices; now 3.8), 11.6
// (2048 rows; 9.5, 4.6 TB/s).
template <int NGW, int NP, int WPB>     // granules per lane: d <= 512 * NGW; NP pending slices; rows per block
__global__ __launch_bounds__(64 * WPB) void k_norm_rows(const int32_t *flags, float *x, const float *ypart, const float *g,
                                                   const float *b, int d, int R, int rows_pad, int kind, float eps,
                                                   bf16_t *xn, bf16_t *xn_lo) {
  const size_t part_stride = (size_t)rows_pad * d;
  const int lane = threadIdx.x & 63, r = tile_on_one_xcd<16 / WPB>(blockIdx.x, R) * WPB + (threadIdx.x >> 6);
  float *xr = x + (size_t)r * d;
  const float *yr = ypart + (size_t)r * d;
  // granules of a batch: at most 20 requests of 32 bytes a lane, at clamped places and without a branch
  constexpr int GB = NGW * (1 + NP) <= 20 ? NGW : NGW * (1 + NP) <= 40 ? NGW / 2 : NGW * (1 + NP) <= 80 ? NGW / 4 : NGW / 8;
  float v[NGW][8];
  int fl = 0;
#pragma unroll
  for (int i0 = 0; i0 < NGW; i0 += GB) {
    floatx4 xv[GB][2], y[GB][2][NP > 0 ? NP : 1];
#pragma unroll
    for (int j = 0; j < GB; ++j) {
      const int c = min((lane + 64 * (i0 + j)) * 8, d - 8);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        xv[j][h] = *(const floatx4 *)(xr + c + 4 * h);
#pragma unroll
        for (int pp = 0; pp < NP; ++pp) y[j][h][pp] = *(const floatx4 *)(yr + pp * part_stride + c + 4 * h);
      }
    }
    if (i0 == 0) fl = flags[min(r, R - 1)];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < GB; ++j) {
      const bool in = (lane + 64 * (i0 + j)) * 8 < d;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int pp = 0; pp < NP; ++pp) xv[j][h] += y[j][h][pp];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[i0 + j][4 * h + e] = in ? xv[j][h][e] : 0.f;
      }
    }
  }
  const bool valid = r < R && (fl & ROW_VALID);
  // gain and bias, whose registers were the slices': asked for under the sums where a lane has room for them
  constexpr int NA = NGW <= 4 ? NGW : 1;
  const float *bias = kind == 0 && b ? b : g;
  floatx4 tg[NA][2], tb[NA][2];
  if (NGW <= 4) {
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const int c = min((lane + 64 * i) * 8, d - 8);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        tg[i][h] = *(const floatx4 *)(g + c + 4 * h);
        tb[i][h] = *(const floatx4 *)(bias + c + 4 * h);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  float s1 = 0.f;
#pragma unroll
  for (int i = 0; i < NGW; ++i)
#pragma unroll
    for (int e = 0; e < 8; ++e) s1 += v[i][e];
  s1 = fold_wave(s1, Add());
  const float mean = kind == 0 ? s1 / d : 0.f;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < NGW; ++i) {
    const bool in = (lane + 64 * i) * 8 < d;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float t = in ? v[i][e] - mean : 0.f;
      q += t * t;
    }
  }
  q = fold_wave(q, Add());
  const float rstd = rsqrtf(q / d + eps);
#pragma unroll
  for (int i = 0; i < NGW; ++i) {
    const int c = (lane + 64 * i) * 8;
    if (c >= d) continue;
    const int ia = NGW <= 4 ? i : 0;
    if (NGW > 4) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        tg[0][h] = *(const floatx4 *)(g + c + 4 * h);
        tb[0][h] = *(const floatx4 *)(bias + c + 4 * h);
      }
    }
    float y[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float bias_e = kind == 0 && b ? tb[ia][e >> 2][e & 3] : 0.f;
      y[e] = valid ? (v[i][e] - mean) * rstd * tg[ia][e >> 2][e & 3] + bias_e : 0.f;
    }
    store8_split(xn, xn_lo, act_off(r, c, d), y);
    if (NP > 0 && r < R) {
      *(float4 *)(xr + c) = make_float4(v[i][0], v[i][1], v[i][2], v[i][3]);
      *(float4 *)(xr + c + 4) = make_float4(v[i][4], v[i][5], v[i][6], v[i][7]);
    }
  }
}

int mfma_norm(pd_ctx *c, const float *gain, const float *bias, int R, hipStream_t s) {
  // packed pairs: rows 8-15 of the fragments belong to the low parts of rows 0-7
  int rows = c->packed ? 8 : (R + 15) / 16 * 16, d = c->cfg.d_model;
  bf16_t *xn = (bf16_t *)c->xn;
  const pd_config &g = c->cfg;
  PD_REQUIRE(d <= 2048 * 4, PD_EINVAL, "d_model %d too large for the norm kernel", d);
  if (rows > 128 && !c->embed_pending && !c->packed) {
    // (up to a row per compute unit a block of its own for each: 192 rows of width 768, four slices 4.2 us in blocks of four
    // rows, 3.8 in blocks of one; 400 rows 4.3 and 4.5)
#define PD_NORM_R(G, P)                                                                           \
  if (rows <= 256) PD_NORM_RW(G, P, 1); else PD_NORM_RW(G, P, 4)
#define PD_NORM_RW(G, P, WPB)                                                                     \
  hipLaunchKernelGGL((k_norm_rows<G, P, WPB>), dim3(rows / WPB), dim3(64 * WPB), 0, s, c->rows.flags, c->x, c->ypart, gain, bias, d, \
                     R, c->R_pad, g.norm_kind, g.norm_eps, xn, mfma_lo(c, xn, d))
#define PD_NORM_RP(G)                                                                            \
  switch (c->pend_parts) {                                                                       \
    case 0: PD_NORM_R(G, 0); break;                                                              \
    case 1: PD_NORM_R(G, 1); break;                                                              \
    case 2: PD_NORM_R(G, 2); break;                                                              \
    case 4: PD_NORM_R(G, 4); break;                                                              \
    default: pd_set_error("unsupported number of pending slices: %d", c->pend_parts); return PD_EINVAL; \
  }
    if (d <= 512) { PD_NORM_RP(1) } else if (d <= 1024) { PD_NORM_RP(2) } else if (d <= 2048) { PD_NORM_RP(4) }
    else if (d <= 4096) { PD_NORM_RP(8) } else { PD_NORM_RP(16) }
#undef PD_NORM_RP
#undef PD_NORM_R
#undef PD_NORM_RW
    PD_CHECK_HIP(hipGetLastError());
    c->pend_parts = 0;
    return PD_OK;
  }
#define PD_NORM(V, P, E)                                                                         \
  hipLaunchKernelGGL((k_norm_bf16<V, P, E>), dim3(rows), dim3(256), 0, s, c->rows.flags,                          \
                     E ? (const void *)c->rows.tok : c->x, E ? (const void *)c->rows.pos : c->ypart, gain, bias, d, R,    \
                     c->R_pad, g.norm_kind, (const bf16_t *)c->tok_emb, (const bf16_t *)c->pos_emb, g.norm_eps, c->x,  \
                     xn, mfma_lo(c, xn, d))
#define PD_NORM_P(V)                                                                             \
  if (c->embed_pending) { PD_NORM(V, 0, true); }                                                 \
  else switch (c->pend_parts) {                                                                  \
    case 0: PD_NORM(V, 0, false); break;                                                         \
    case 1: PD_NORM(V, 1, false); break;                                                         \
    case 2: PD_NORM(V, 2, false); break;                                                         \
    case 4: PD_NORM(V, 4, false); break;                                                         \
    default: pd_set_error("unsupported number of pending slices: %d", c->pend_parts); return PD_EINVAL; \
  }
  if (d <= 2048) { PD_NORM_P(1) } else if (d <= 4096) { PD_NORM_P(2) } else { PD_NORM_P(4) }
#undef PD_NORM_P
#undef PD_NORM
  PD_CHECK_HIP(hipGetLastError());
  c->pend_parts = 0;
  c->embed_pending = false;
  return PD_OK;
}

#endif

#ifdef PD_GEMM_EPI
#define PD_GEMM_CAT2(a, b) a##b
#define PD_GEMM_CAT(a, b) PD_GEMM_CAT2(a, b)
#define PD_GEMM_ENTRY PD_GEMM_CAT(mfma_gemm_epi, PD_GEMM_EPI)
#define PD_GEMM_ROWS_ENTRY PD_GEMM_CAT(mfma_gemm_rows_epi, PD_GEMM_EPI)

// ---------------------------------------------------------------------------
// skinny GEMM  y[r][n] = sum_k xn[r][k] W[n][k],  r < 16*RT rows (RT = 1, 2, 4, 5, 8); weights and
// activations both fragment-major.
// The matrix core computes the transposed tile: A = weight fragment (16 output columns x 32 k),
// B = activations (32 k x 16 rows), D[4g+j][r] = y[r][n0+4g+j].
// A block has NW_K waves that cut K between them; every wave owns the same NT column tiles and all
// RT row tiles, so the block requests every activation fragment of its K range exactly once and
// uses it for NT weight fragments.  The waves' partial tiles are summed through LDS.  The launch
// lives for a few microseconds up to a few tens: every load must be in flight from the first cycle
// on.  Per chunk of U k-tiles a wave requests everything first (the high- and low-part activation
// fragments of the row tiles, then the weight fragments of its tiles) into registers of their own;
// only then the multiplies run.  A share that is not a multiple of U ends with chunks of 4, 3, 2 and
// 1 k-tiles, so that no load is ever conditional.
// This file is compiled twice per epilogue (PD_GEMM_EPI = 0..6: kernels and launch code of that epilogue; with
// PD_GEMM_ROWS those of more than 128 rows and of the vocabulary projection of 33-128) and once without (weight packing,
// norm kernel, dispatcher).  Two units, because what else a unit holds decides how the compiler orders and allocates a
// kernel: in one unit with the others the QKV projection of 64 rows, width 4096, took 30.0 us instead of 29.1.
// ---------------------------------------------------------------------------
// epilogue of one 16-column tile: lane holds y[r][n0 + j], r = i*16 + m, n0 = nt*16 + 4g, j = 0..3
// Mean and reciprocal standard deviation of a row from the per-tile sums the producing projection
// left (EPI_RESID_NORM), stats[row][tile] = (sum, sum of squares).  The NW waves of a block share the
// work: wave w, lane (m, g) takes the tile pairs g + 4 (w + NW u) of row m, u = 0 .. PS-1, requested at
// kernel start so that they arrive with the first weights; what lies beyond (very wide models) is
// read when the sums are taken.  Fixed order, no atomics: deterministic.
constexpr int PS = 4;
__device__ __forceinline__ void stats_request(const float2 *stats, int npair, int lane, int w, int nw, float4 (&pre)[PS], int r0) {
  const int m = r0 + (lane & 15), g = lane >> 4;
  const float4 *sp = (const float4 *)stats + (size_t)m * npair;
#pragma unroll
  for (int u = 0; u < PS; ++u) {
    pre[u] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (4 * (w + nw * u) < npair) pre[u] = sp[min(g + 4 * (w + nw * u), npair - 1)];   // the same for the whole wave
  }
}
__device__ __forceinline__ float2 stats_partial(const float2 *stats, int npair, int lane, int w, int nw, const float4 (&pre)[PS], int r0) {
  const int m = r0 + (lane & 15), g = lane >> 4;
  const float4 *sp = (const float4 *)stats + (size_t)m * npair;
  float s1 = 0.f, s2 = 0.f;
#pragma unroll
  for (int u = 0; u < PS; ++u)
    if (g + 4 * (w + nw * u) < npair) { s1 += pre[u].x + pre[u].z; s2 += pre[u].y + pre[u].w; }
  for (int p = g + 4 * (w + nw * PS); p < npair; p += 4 * nw) {
    float4 v = sp[p];
    s1 += v.x + v.z; s2 += v.y + v.w;
  }
  s1 = fold32(fold16(s1, Add()), Add());
  s2 = fold32(fold16(s2, Add()), Add());
  return make_float2(s1, s2);
}
__device__ __forceinline__ float2 stats_finish(const GemmArgs &a, float2 s) {
  const float inv_d = 1.f / (float)a.norm_d;
  const float mean = a.norm_kind == 0 ? s.x * inv_d : 0.f;
  const float var = fmaxf(s.y * inv_d - mean * mean, 0.f);
  return make_float2(mean, rsqrtf(var + a.norm_eps));
}

// what the finishing wave of a tile asked for at kernel start (EPI_RESID_NORM): the residual rows
// and the next norm's gain at its columns
struct ResidPre { float4 x, g; };
// ... and for a projection that finishes a norm: c1 and c2 at the tile's columns
struct NormPre { float4 c1, c2; };

// EPI_LM: the best value of a row so far and its column, in every lane of the row
struct Winner { float best; int idx; };
constexpr int NO_WINNER = 0x7fffffff;

// t Phi(t) = max(t, 0) - |t| Phi(-|t|), Phi the normal distribution, by a polynomial for the logarithm of its tail
// (gelu_coefficient).  One form for every t, 14 instructions where erff has two branches of 42 together, and closer: over normal t of deviation 0.1, 1 and 4 the error is 3.1e-8, 2.7e-8 and 1.7e-8 (2-norm, relative), with 0.5 t (1 + erff) 3.8e-8,
// 3.8e-8 and 2.3e-8 (for t < 0 that sum cancels: 1e-5 at t = -3, here 8e-7).  4096 rows, 8192 columns,
// K 2048: 258 -> 237 us; 2048 rows, 3072 columns, K 768: 29.5 -> 26.0.
__device__ __forceinline__ float gelu(float t) {
  const float b = fabsf(t), a = b > 8.f ? 8.f : b;          // (NaN stays NaN)
  float r = gelu_coefficient(GELU_TERMS - 1);
#pragma unroll
  for (int i = GELU_TERMS - 2; i >= 0; --i) r = fmaf(r, a, gelu_coefficient(i));
  return fmaf(-0.5f * a, __builtin_amdgcn_exp2f(-(r * a)), t > 0.f ? t : 0.f);
}

// NORMED: instances that can finish a norm (nrm is looked at); the others carry none of its code
template <int RT, int EPI, bool NORMED = false>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs &a, int nt, const floatx4 (&acc_in)[RT],
                                              const int4 *kvi, int lane, int r0 = 0,
                                              const float2 *nrm = nullptr, const ResidPre *pre = nullptr,
                                              const NormPre *npre = nullptr, Winner *win = nullptr) {
  int m = lane & 15, g = lane >> 4;
  int n0 = nt * 16 + 4 * g;
  floatx4 acc[RT];
#pragma unroll
  for (int i = 0; i < RT; ++i) acc[i] = acc_in[i];
  if (NORMED && nrm) {
    // the activations were gain * x: finish the norm here (columns in the packed order of the weights)
    const float4 c1 = npre ? npre->c1 : *(const float4 *)(a.c1 + n0);
    const float4 c2 = npre ? npre->c2 : (a.c2 ? *(const float4 *)(a.c2 + n0) : make_float4(0.f, 0.f, 0.f, 0.f));
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      acc[i][0] = nrm[i].y * (acc[i][0] - nrm[i].x * c1.x) + c2.x;
      acc[i][1] = nrm[i].y * (acc[i][1] - nrm[i].x * c1.y) + c2.y;
      acc[i][2] = nrm[i].y * (acc[i][2] - nrm[i].x * c1.z) + c2.z;
      acc[i][3] = nrm[i].y * (acc[i][3] - nrm[i].x * c1.w) + c2.w;
    }
  }
  // rows at and beyond a.R are never stored: nobody reads them, and with packed activations their
  // slots hold the low parts of rows 0-7
  if (EPI == EPI_RESID) {
    // split-K slice blockIdx.y of y; the following norm kernel adds the slices to x
    float *yp = a.x + (size_t)blockIdx.y * a.part_stride;
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      int r = r0 + i * 16 + m;
      if (r >= a.R) continue;
      *(float4 *)(yp + (size_t)r * a.ld + n0) = make_float4(acc[i][0], acc[i][1], acc[i][2], acc[i][3]);
    }
  } else if (EPI == EPI_RESID_NORM) {
    const float4 gn = pre ? pre->g : *(const float4 *)(a.gain + n0);
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      int r = r0 + i * 16 + m;
      const bool in = r < a.R;
      float4 xo = make_float4(0.f, 0.f, 0.f, 0.f);
      if (in) xo = (pre && RT == 1) ? pre->x : *(const float4 *)(a.x_res + (size_t)r * a.ld + n0);
      float xn[4] = {xo.x + acc[i][0], xo.y + acc[i][1], xo.z + acc[i][2], xo.w + acc[i][3]};
      float s1 = 0.f, s2 = 0.f;
      if (in) {
        *(float4 *)(a.x_res + (size_t)r * a.ld + n0) = make_float4(xn[0], xn[1], xn[2], xn[3]);
        float z[4] = {gn.x * xn[0], gn.y * xn[1], gn.z * xn[2], gn.w * xn[3]};
        store4_split(a.out_bf, a.out_lo, act_off(r, n0, a.ld), z);
        s1 = (xn[0] + xn[1]) + (xn[2] + xn[3]);
        s2 = (xn[0] * xn[0] + xn[1] * xn[1]) + (xn[2] * xn[2] + xn[3] * xn[3]);
      }
      s1 = fold32(fold16(s1, Add()), Add());
      s2 = fold32(fold16(s2, Add()), Add());
      if (g == 0) a.stats_out[(size_t)r * a.n_tiles + nt] = make_float2(s1, s2);
    }
  } else if (EPI == EPI_GELU) {
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      int r = r0 + i * 16 + m;
      float y[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float t = acc[i][j];
        y[j] = a.act == 1 ? fmaxf(t, 0.f) : gelu(t);
      }
      if (r < a.R) store4_split(a.out_bf, a.out_lo, act_off(r, n0, a.ld), y);
    }
  } else if (EPI == EPI_SWIGLU) {
    // groups 0,1: gate of features nt*8 + 4g + j; groups 2,3: up of nt*8 + 4(g-2) + j
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      int r = r0 + i * 16 + m;
      float y[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const Halves<float> h = halves32(acc[i][j]);     // gate and up
        y[j] = h.lo / (1.f + __expf(-h.lo)) * h.hi;
      }
      if (g < 2 && r < a.R) store4_split(a.out_bf, a.out_lo, act_off(r, nt * 8 + 4 * g, a.ld), y);
    }
  } else if (EPI == EPI_QKV || EPI == EPI_QKV_ROPE) {
    int sec = n0 / a.d + a.sec0, nl = n0 % a.d, h = nl / a.hd;
    int half = a.hd >> 1;
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      int r = r0 + i * 16 + m;
      bool valid = r < a.R && (kvi[i].x & ROW_VALID);
      float y[4];
      int dim0;                                  // head-dim index of y[0]; y[j] is dim0 + j
      if (EPI == EPI_QKV_ROPE && sec < 2) {
        int th = (nl % a.hd) >> 4;
        int jj = th * 8 + 4 * (g & 1);           // rotation pair index of y[0]
        dim0 = jj + (g >= 2 ? half : 0);
        const float *cs = a.rope_cs + ((size_t)(valid ? kvi[i].w : 0) * half + jj) * 2;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const Halves<float> x = halves32(acc[i][j]);
          float cc = cs[2 * j], ss = cs[2 * j + 1];
          // low half: x1*c - x2*s ; high half: x2*c + x1*s
          y[j] = g < 2 ? x.lo * cc - x.hi * ss : x.hi * cc + x.lo * ss;
        }
      } else {
        dim0 = (nl % a.hd);
#pragma unroll
        for (int j = 0; j < 4; ++j) y[j] = acc[i][j];
      }
      if (!valid) continue;
      // keys and values beyond the largest half are stored saturated; count them so that the caller
      // can find out (practically never taken)
      if (sec != 0 && fmaxf(fmaxf(fabsf(y[0]), fabsf(y[1])), fmaxf(fabsf(y[2]), fabsf(y[3]))) > 65504.f)
        atomicAdd(a.kv_sat, (fabsf(y[0]) > 65504.f) + (fabsf(y[1]) > 65504.f) + (fabsf(y[2]) > 65504.f) +
                                (fabsf(y[3]) > 65504.f));
      if (sec == 0) {
        store4_split_h((f16_t *)a.out_bf, (f16_t *)a.out_lo, act_off(r, h * a.hd + dim0, a.d), y);
      } else {
        size_t head_base = ((size_t)kvi[i].y * a.H + h) * a.kv_cap * a.hd;
        int slot = kvi[i].z;
        if (sec == 1) {
          store4_split_h(a.kc, a.kc_lo, head_base + k_cache_off(slot, dim0, a.hd), y);
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            size_t o = head_base + v_cache_off(slot, dim0 + j, a.hd);
            f16_t hi = f32_to_f16_sat(y[j]);
            a.vc[o] = hi;
            if (a.vc_lo) a.vc_lo[o] = (f16_t)(y[j] - (float)hi);
          }
        }
      }
    }
  } else if (EPI == EPI_LM) {
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      int r = r0 + i * 16 + m;
      float best = -INFINITY;
      int bi = 0x7fffffff;
      float *dst = nullptr;
      if (a.logits && r < a.R) {
        const int4 qi = a.rt.qinfo[r];          // {flags, subsequence, limit, request}
        const int q = a.logits_A > 0 ? r / a.logits_A : qi.w;
        if (qi.x & ROW_VALID)
          dst = a.logits + ((size_t)q * a.logits_cap + (a.logits_A > 0 ? r - q * a.logits_A : qi.y - 1)) * a.ld_logits;
      }
      // (a row of logits starts at any multiple of 4 bytes: one 16-byte store, dword-aligned)
      if (dst && n0 + 3 < a.V) *(floatx4_a4 *)(dst + n0) = floatx4_a4{acc[i][0], acc[i][1], acc[i][2], acc[i][3]};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        int n = n0 + j;
        float t = acc[i][j];
        if (n < a.V) {
          if (dst && n0 + 3 >= a.V) dst[n] = t;
          if (t > best) { best = t; bi = n; }
        }
      }
      if (a.logits_A > 0) continue;           // (a training target selects no tokens)
      // across the 4 column groups of this row; lowest index wins ties
      best16(best, bi);
      best32(best, bi);
      keep_best(win[i].best, win[i].idx, best, bi);
    }
  }
}

// One winner per row and block: W waves of the block hold one each.  (One per 16-column tile: k_turn, one block per
// request, read 25 KB per row at 50265 words.)  Row-major [row][block]: it reads a row's winners as one run.
template <int RT, int W>
__device__ __forceinline__ void store_winners(const GemmArgs &a, const Winner (&win)[RT], int w, int lane, int r0) {
  if (a.logits_A > 0) return;           // the same for the whole launch
  __shared__ Winner sm_win[W > 1 ? W : 1][RT * 16];
  if (W > 1) {
    if (w < W && lane < 16)
#pragma unroll
      for (int i = 0; i < RT; ++i) sm_win[w][i * 16 + lane] = win[i];
    __syncthreads();
    const int q = threadIdx.x, r = r0 + q;
    if (q >= RT * 16 || r >= a.R) return;
    Winner best = sm_win[0][q];
#pragma unroll
    for (int v = 1; v < W; ++v) keep_best(best.best, best.idx, sm_win[v][q].best, sm_win[v][q].idx);
    a.part_val[(size_t)r * a.n_win + blockIdx.x] = best.best;
    a.part_idx[(size_t)r * a.n_win + blockIdx.x] = best.idx;
  } else if (w == 0 && lane < 16) {
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      const int r = r0 + i * 16 + lane;
      if (r >= a.R) continue;
      a.part_val[(size_t)r * a.n_win + blockIdx.x] = win[i].best;
      a.part_idx[(size_t)r * a.n_win + blockIdx.x] = win[i].idx;
    }
  }
}

// SW: the weight fragments are loaded with the non-temporal hint.  A step reads every weight once; when the
// step's bytes exceed the last-level cache nothing of them is left there a step later, and keeping them out
// of the caches' way makes the streams faster (cfg4 1.35 -> 1.31 ms per step, cfg5 6.27 -> 6.09); a model
// that fits the cache is served from it step after step and loses with the hint (cfg2 0.187 -> 0.202).
template <bool SW>
__device__ __forceinline__ bf16x8 ld_w(const uint4 *p) {
  return SW ? __builtin_nontemporal_load((const bf16x8 *)p) : *(const bf16x8 *)p;
}

template <int RT, int NT, int U, bool SPLIT, int NA, bool SW>
__device__ __forceinline__ void gemm_chunk(floatx4 (&acc)[NT][RT][NA], const uint4 *wp, const uint4 *xp,
                                           const uint4 *xl, size_t KT, const int (&tile)[NT], int kt) {
  Frag wa[NT][U], xh[RT][U], xo[SPLIT ? RT : 1][U];
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int u = 0; u < U; ++u) {
      xh[i][u].u = xp[((size_t)i * KT + kt + u) * 64];
      if (SPLIT) xo[i][u].u = xl[((size_t)i * KT + kt + u) * 64];
    }
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int u = 0; u < U; ++u) wa[t][u].v = ld_w<SW>(&wp[((size_t)tile[t] * KT + kt + u) * 64]);
  __builtin_amdgcn_sched_barrier(0);          // every request above is issued before the first multiply
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int i = 0; i < RT; ++i) {
        // small tiles keep two accumulators per tile (NA = 2) so that the high- and low-part products
        // do not wait for each other; large tiles have enough independent accumulators anyway
        acc[t][i][0] = mfma16(wa[t][u], xh[i][u], acc[t][i][0]);
        if (SPLIT) acc[t][i][NA - 1] = mfma16(wa[t][u], xo[i][u], acc[t][i][NA - 1]);
      }
}

// What a launch needs before it can ask for its first byte comes as scalars in front of GemmArgs: compiled with
// -amdgpu-kernarg-preload-count the first 14 words of the arguments are in scalar registers when a wave starts.  Read from
// memory they cost every launch 0.25-0.35 us before its first request (they are new to every cache), twice where a pointer
// decides on the next read; a decode step is 30-270 such launches one after the other.
#define PD_GEMM_HOT_PARAMS                                                                                        \
  const bf16_t *hot_w, const bf16_t *hot_x, const void *hot_a, const void *hot_b, const void *hot_c, uint32_t hot_lo, \
      uint32_t hot_k, uint32_t hot_share, uint32_t hot_n
struct GemmHot {
  const bf16_t *w, *x;        // weights, activations
  const void *a, *b, *c;      // EPI_RESID_NORM: x_res, gain, sums_before; finishing a norm: stats_in (else NULL), c1; EPI_QKV*: c = kvinfo
  GemmWords n;
};
template <int EPI>
static GemmHot gemm_hot(const GemmArgs &a) {
  constexpr bool out = EPI == EPI_RESID_NORM;
  return GemmHot{a.W, a.xn, out ? (const void *)a.x_res : a.stats_in, out ? a.gain : a.c1, out ? (const void *)a.sums_before : a.rt.kvinfo,
                 out ? gemm_words_rows(a.xn_lo ? a.xn_lo - a.xn : 0, a.K, a.k_share, a.n_tiles, a.R)
                     : gemm_words(a.xn_lo ? a.xn_lo - a.xn : 0, a.K, a.k_share, a.n_tiles, a.c2 != nullptr, a.stats_tiles > a.K / 16)};
}
template <int EPI, typename Kernel>
static int launch_gemm_kernel(Kernel kernel, dim3 grid, int threads, GemmArgs a, hipStream_t s) {
  PD_REQUIRE(a.K / 32 <= WORDS_K_TILES, PD_EINVAL, "%d inner values", a.K);
  PD_REQUIRE(!a.stats_in || ((a.stats_tiles == a.K / 16 || a.stats_tiles == a.K / 8) && (!a.c2 || a.c2 == a.c1 + (size_t)a.n_tiles * 16)), PD_EINVAL,
             "a norm is finished over the whole rows, with c2 behind c1");
  PD_REQUIRE(EPI != EPI_RESID_NORM || (a.R <= 128 && a.n_tiles < 65536), PD_EINVAL, "%d rows of %d values cannot prepare a norm",
             a.R, a.n_tiles * 16);
  a.n_win = grid.x;
  if (EPI == EPI_LM) *a.win_out = grid.x;
  const GemmHot h = gemm_hot<EPI>(a);
  hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, s, h.w, h.x, h.a, h.b, h.c, h.n.lo, h.n.k, h.n.share, h.n.n, a);
  PD_CHECK_HIP(hipGetLastError());
  return PD_OK;
}

// PACK (one row tile, at most 8 rows): the activation fragment carries the high parts in rows 0-7
// and the low parts of the same 8 rows in rows 8-15, so one fragment and one multiply per k-tile
// do the work of two; the two halves of the output tile are added before the epilogue.
// FUSED_IN: the epilogue finishes a norm where a.stats_in is set.  The first FFN projections always carry the code; the
// QKV projections have instances of their own for it (in the ordinary ones it cost 0.7 us of 7.8 at width 2048).
constexpr bool norm_in_default(int rt, int epi) { return rt == 1 && (epi == EPI_GELU || epi == EPI_SWIGLU); }
// ZROWS: the block serves row tiles blockIdx.z * RT .. + RT - 1 only (launches that spread the row tiles of a
// step over blocks, see launch_gemm_zrows).
// SW: weights loaded with the non-temporal hint (see ld_w; chosen per context, never with ZROWS, whose row
// tiles re-read the weights through L2).
template <int RT, int NT, int NW_K, int U, int EPI, bool SPLIT, bool PACK, bool ZROWS = false, bool SW = false,
          bool FUSED_IN = norm_in_default(RT, EPI)>
__global__ __launch_bounds__(64 * NW_K) void k_gemm_s(PD_GEMM_HOT_PARAMS, GemmArgs a) {
  static_assert(!PACK || (RT == 1 && !SPLIT), "packed activations: one row tile, one fragment");
  const int rz = ZROWS ? (int)blockIdx.z * RT : 0;          // first row tile of this block
  __shared__ floatx4 red[NW_K > 1 ? NW_K * NT * RT * 64 : 1];
  const int wk = NW_K == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int nt0 = blockIdx.x * NT;
  const int m = lane & 15;
  constexpr bool OUT = EPI == EPI_RESID_NORM;
  const int KT = words_k_tiles(hot_k), k_share = words_k_tiles(hot_share), n_tiles = OUT ? words_tiles_rows(hot_n) : words_tiles(hot_n);
  // waves along K: NW_K in this block times gridDim.y blocks (EPI_RESID only)
  const int gk = blockIdx.y * NW_K + wk;
  const int kt0 = min(gk * k_share, KT), kt1 = min(kt0 + k_share, KT);
  int tile[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) tile[t] = min(nt0 + t, n_tiles - 1);   // tiles past the end repeat the last one
  const uint4 *wp = (const uint4 *)hot_w + lane;
  const uint4 *xp = (const uint4 *)hot_x + lane + (size_t)rz * KT * 64;
  const uint4 *xl = SPLIT ? xp + words_granules(hot_lo) : nullptr;
  // row data of the KV-append epilogue, requested now so that it arrives with the weights (where a row's logits go is
  // read by the epilogue that stores them: requested here it held 4 registers per row tile in every vocabulary launch)
  constexpr bool QKV = EPI == EPI_QKV || EPI == EPI_QKV_ROPE;
  int4 kvi[QKV ? RT : 1];
  if (QKV) {
#pragma unroll
    for (int i = 0; i < RT; ++i) kvi[i] = ((const int4 *)hot_c)[(rz + i) * 16 + m];
  }
  // one row tile: what the epilogue needs from memory is asked for now, so that it arrives with the weights
  static_assert(!FUSED_IN || RT == 1, "norms are finished per row tile");
  constexpr bool FUSED_OUT = RT == 1 && EPI == EPI_RESID_NORM;
  __shared__ float2 sm_stat[FUSED_IN ? NW_K : 1][16];
  float4 pre_s[PS];
  const bool fused_norm = FUSED_IN && hot_a != nullptr;               // the same for the whole launch
  const int npair = OUT ? 0 : KT << words_half_sums(hot_n);           // pairs of row sums
  NormPre pre_n;
  if (fused_norm) stats_request((const float2 *)hot_a, npair, lane, wk, NW_K, pre_s, rz * 16);
  if (fused_norm && wk < NT) {      // wave w < NT finishes tile nt0 + w
    const float *c1 = (const float *)hot_b + min(nt0 + wk, n_tiles - 1) * 16 + 4 * (lane >> 4);
    pre_n.c1 = *(const float4 *)c1;
    pre_n.c2 = words_c2(hot_n) ? *(const float4 *)(c1 + n_tiles * 16) : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  ResidPre pre_r;
  if (FUSED_OUT && wk < NT) {       // wave w < NT finishes tile nt0 + w
    const int n0 = min(nt0 + wk, n_tiles - 1) * 16 + 4 * (lane >> 4);
    pre_r.g = *(const float4 *)((const float *)hot_b + n0);
    // (rows beyond R read row R - 1 and are masked where the value is used, not here: touching the
    // value now would make the wave wait for it before it has asked for its weights)
    pre_r.x = *(const float4 *)((const float *)hot_a + (size_t)min(rz * 16 + m, words_last_row(hot_n)) * (n_tiles * 16) + n0);
  }
  constexpr int NA = (SPLIT && NT * RT <= 2) ? 2 : 1;
  floatx4 acc2[NT][RT][NA];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int i = 0; i < RT; ++i) acc2[t][i][0] = acc2[t][i][NA - 1] = floatx4{0.f, 0.f, 0.f, 0.f};
  int kt = kt0;
  while (kt + U <= kt1) { gemm_chunk<RT, NT, U, SPLIT, NA, SW>(acc2, wp, xp, xl, KT, tile, kt); kt += U; }
  if (U > 4 && kt + 4 <= kt1) { gemm_chunk<RT, NT, 4, SPLIT, NA, SW>(acc2, wp, xp, xl, KT, tile, kt); kt += 4; }
  if (U > 3 && kt + 3 <= kt1) { gemm_chunk<RT, NT, 3, SPLIT, NA, SW>(acc2, wp, xp, xl, KT, tile, kt); kt += 3; }
  if (U > 2 && kt + 2 <= kt1) { gemm_chunk<RT, NT, 2, SPLIT, NA, SW>(acc2, wp, xp, xl, KT, tile, kt); kt += 2; }
  if (U > 1 && kt < kt1) gemm_chunk<RT, NT, 1, SPLIT, NA, SW>(acc2, wp, xp, xl, KT, tile, kt);
  floatx4 acc[NT][RT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int i = 0; i < RT; ++i) acc[t][i] = NA == 2 ? acc2[t][i][0] + acc2[t][i][1] : acc2[t][i][0];
  if (PACK) {
    // output row m + 8 holds the product with the low parts of row m
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[t][0][j] += rotate16<8>(acc[t][0][j]);
  }
  Winner win[EPI == EPI_LM ? RT : 1];
  if (EPI == EPI_LM)
#pragma unroll
    for (int i = 0; i < RT; ++i) win[i] = Winner{-INFINITY, NO_WINNER};
  if (NW_K > 1) {
    // every wave leaves its partial tiles in LDS; wave w then sums and finishes column tiles w, w + NW_K, ...
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int i = 0; i < RT; ++i) red[((wk * NT + t) * RT + i) * 64 + lane] = acc[t][i];
    if (fused_norm) {
      float2 sp = stats_partial((const float2 *)hot_a, npair, lane, wk, NW_K, pre_s, rz * 16);
      if (lane < 16) sm_stat[wk][lane] = sp;
    }
    __syncthreads();
    float2 nrm[RT];
    if (fused_norm && wk < NT) {            // finishing waves: add the waves' shares in wave order
      float2 tot = sm_stat[0][m];
#pragma unroll
      for (int w = 1; w < NW_K; ++w) { tot.x += sm_stat[w][m].x; tot.y += sm_stat[w][m].y; }
      nrm[0] = stats_finish(a, tot);
    }
    for (int t = wk; t < NT && nt0 + t < n_tiles; t += NW_K) {
      floatx4 sum[RT];
#pragma unroll
      for (int i = 0; i < RT; ++i) sum[i] = red[((0 * NT + t) * RT + i) * 64 + lane];
#pragma unroll
      for (int w = 1; w < NW_K; ++w)
#pragma unroll
        for (int i = 0; i < RT; ++i) sum[i] += red[((w * NT + t) * RT + i) * 64 + lane];
      gemm_epilogue<RT, EPI, FUSED_IN>(a, nt0 + t, sum, kvi, lane, rz * 16, fused_norm ? nrm : nullptr,
                             (FUSED_OUT && t == wk) ? &pre_r : nullptr, (fused_norm && t == wk) ? &pre_n : nullptr, win);
    }
    if constexpr (EPI == EPI_LM) store_winners<RT, (NT < NW_K ? NT : NW_K)>(a, win, wk, lane, rz * 16);
  } else {
    float2 nrm[RT];
    if (fused_norm) nrm[0] = stats_finish(a, stats_partial((const float2 *)hot_a, npair, lane, 0, 1, pre_s, rz * 16));
#pragma unroll
    for (int t = 0; t < NT; ++t)
      if (nt0 + t < n_tiles)
        gemm_epilogue<RT, EPI, FUSED_IN>(a, nt0 + t, acc[t], kvi, lane, rz * 16, fused_norm ? nrm : nullptr,
                               (FUSED_OUT && t == 0) ? &pre_r : nullptr, (fused_norm && t == 0) ? &pre_n : nullptr, win);
    if constexpr (EPI == EPI_LM) store_winners<RT, 1>(a, win, 0, lane, rz * 16);
  }
}

#if PD_GEMM_EPI == 6 && !defined(PD_GEMM_ROWS)     // EPI_RESID_NORM
// The same product for a projection that completes at most 16 rows and prepares the next norm, which is not cut along K over
// blocks: a block takes half of a column tile, 8 columns, so that twice as many compute units draw its weights.  One request
// brings the 8 columns of two k-tiles (lanes m < 8 of the first, the others of the second: the fragments' granules
// half a line at a time), and the one register pair is multiplied with the activations of either k-tile: output rows 0-7 of the
// first product and 8-15 of the second are sums to keep, the other halves meet the wrong k-tile and are dropped.  As many
// multiplies as with whole tiles, half the weights per compute unit, the same activations.  Row sums are left per 8 columns.
// Bound by what a compute unit draws, twice as many activations as weights (width 2048, 8192 inner values from the caches 7.8 us,
// cut along K 7.0 with 3.3 for the norm kernel behind it; from memory 10.9 against 7.4 + 3.2: see ffn2_handover).
// MEAN: for a norm that subtracts the mean, rows are handed over less the mean of their first 128 values in front of the FFN (from the
// sums that the output projection left).  The norm does not change when a row is shifted, and what is rounded to bf16 pairs
// is about as small as what a norm kernel rounds.  With the mean in it the relative error of the projection behind, at means of 0 /
// 1 / 3 / 10 / 36 deviations, was 2.4e-6 / 3.5e-6 / 7.7e-6 / 2.6e-5 / 1.0e-4, where a norm kernel's is 2.4e-6.
template <int NW, bool PACK, bool SW, bool MEAN>
__global__ __launch_bounds__(64 * NW) void k_gemm_half(PD_GEMM_HOT_PARAMS, GemmArgs a) {
  __shared__ floatx4 red[NW][32];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
  const int tile = blockIdx.x >> 1, half = blockIdx.x & 1;
  const int KT = words_k_tiles(hot_k), share = words_k_tiles(hot_share), n_tiles = words_tiles_rows(hot_n);      // (KT, share even)
  const int kt0 = min(w * share, KT), kt1 = min(kt0 + share, KT);
  const uint4 *wp = (const uint4 *)hot_w + ((size_t)tile * KT + (m >> 3)) * 64 + g * 16 + half * 8 + (m & 7);
  const uint4 *xp = (const uint4 *)hot_x + lane, *xl = PACK ? nullptr : xp + words_granules(hot_lo);
  const int n0 = tile * 16 + half * 8 + 4 * (g & 1);
  ResidPre pre;
  float4 sums;
  if (w == 0) {                         // (rows beyond the last read it and are masked where the value is used)
    pre.g = *(const float4 *)((const float *)hot_b + n0);
    pre.x = *(const float4 *)((const float *)hot_a + (size_t)min(m, words_last_row(hot_n)) * (n_tiles * 16) + n0);
    if (MEAN) sums = ((const float4 *)hot_c)[(size_t)m * (n_tiles / 2) + g];       // of two tiles each
  }
  floatx4 acc[2][PACK ? 1 : 2];         // k-tiles of either parity; high and low parts
#pragma unroll
  for (int p = 0; p < 2; ++p) acc[p][0] = acc[p][PACK ? 0 : 1] = floatx4{0.f, 0.f, 0.f, 0.f};
  auto chunk = [&](int kt, auto u_) {
    constexpr int U = decltype(u_)::value;
    Frag wa[U / 2], xh[U], xo[PACK ? 1 : U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      xh[u].u = xp[(size_t)(kt + u) * 64];
      if (!PACK) xo[u].u = xl[(size_t)(kt + u) * 64];
    }
#pragma unroll
    for (int u = 0; u < U / 2; ++u) wa[u].v = ld_w<SW>(&wp[(size_t)(kt + 2 * u) * 64]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      acc[u & 1][0] = mfma16(wa[u / 2], xh[u], acc[u & 1][0]);
      if (!PACK) acc[u & 1][PACK ? 0 : 1] = mfma16(wa[u / 2], xo[u], acc[u & 1][PACK ? 0 : 1]);
    }
  };
  int kt = kt0;
  constexpr int U = PACK ? 12 : 6;      // (16 waves leave 128 registers)
  for (; kt + U <= kt1; kt += U) chunk(kt, std::integral_constant<int, U>());
  if (PACK && kt + 8 <= kt1) { chunk(kt, std::integral_constant<int, 8>()); kt += 8; }
  if (PACK && kt + 6 <= kt1) { chunk(kt, std::integral_constant<int, 6>()); kt += 6; }
  if (kt + 4 <= kt1) { chunk(kt, std::integral_constant<int, 4>()); kt += 4; }
  if (kt < kt1) chunk(kt, std::integral_constant<int, 2>());
  floatx4 y;                            // lanes 0-31: columns 4 g .. + 3 of row m
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float first = acc[0][0][j], second = acc[1][0][j];
    if (!PACK) { first += acc[0][PACK ? 0 : 1][j]; second += acc[1][PACK ? 0 : 1][j]; }
    y[j] = first + halves32(second).hi;
    if (PACK) y[j] += rotate16<8>(y[j]);              // rows 8-15 hold the products with the low parts of 0-7
  }
  if (lane < 32) red[w][lane] = y;
  __syncthreads();
  if (w != 0) return;
  y = red[0][lane & 31];
#pragma unroll
  for (int v = 1; v < NW; ++v) y += red[v][lane & 31];
  const bool in = m < a.R && lane < 32;
  const float mean = MEAN ? fold32(fold16(sums.x + sums.z, Add()), Add()) * (1.f / 128.f) : 0.f;
  float s1 = 0.f, s2 = 0.f;
  if (in) {
    float x[4] = {pre.x.x + y[0], pre.x.y + y[1], pre.x.z + y[2], pre.x.w + y[3]};
    *(float4 *)(a.x_res + (size_t)m * a.ld + n0) = make_float4(x[0], x[1], x[2], x[3]);
    if (MEAN)
#pragma unroll
      for (int j = 0; j < 4; ++j) x[j] -= mean;
    const float z[4] = {pre.g.x * x[0], pre.g.y * x[1], pre.g.z * x[2], pre.g.w * x[3]};
    store4_split(a.out_bf, a.out_lo, act_off(m, n0, a.ld), z);
    s1 = (x[0] + x[1]) + (x[2] + x[3]);
    s2 = (x[0] * x[0] + x[1] * x[1]) + (x[2] * x[2] + x[3] * x[3]);
  }
  s1 = fold16(s1, Add());
  s2 = fold16(s2, Add());
  if (g == 0) a.stats_out[(size_t)m * (2 * a.n_tiles) + blockIdx.x] = make_float2(s1, s2);
}

template <int NW>
static int launch_gemm_half(GemmArgs a, hipStream_t s) {
  PD_REQUIRE(a.R <= 16 && a.K % 64 == 0, PD_EINVAL, "%d rows of %d inner values in halves of column tiles", a.R, a.K);
  PD_REQUIRE(!a.sums_before || (a.n_tiles >= 8 && a.n_tiles % 2 == 0), PD_EINVAL, "means of %d column tiles", a.n_tiles);
  a.k_share = (a.K / 64 + NW - 1) / NW * 2;
  const dim3 grid(2 * a.n_tiles);
#define PD_HALF(P, M) (a.stream_w ? launch_gemm_kernel<EPI_RESID_NORM>(k_gemm_half<NW, P, true, M>, grid, 64 * NW, a, s)    \
                                  : launch_gemm_kernel<EPI_RESID_NORM>(k_gemm_half<NW, P, false, M>, grid, 64 * NW, a, s))
  if (a.sums_before) return a.packed ? PD_HALF(true, true) : PD_HALF(false, true);
  return a.packed ? PD_HALF(true, false) : PD_HALF(false, false);
#undef PD_HALF
}
#endif

// ---------------------------------------------------------------------------
// launch
// ---------------------------------------------------------------------------
#ifndef PD_GEMM_ROWS
int PD_GEMM_ROWS_ENTRY(const GemmArgs &a, int rows, hipStream_t s);
int mfma_gemm_rows_epi5(const GemmArgs &a, int rows, hipStream_t s);

// 1 row tile.  Two column tiles per wave when that still leaves 128 or more blocks: the
// activation fragments (2 KiB per k-tile with the low parts) are then requested once for 2 KiB of
// weights instead of 1 KiB, and the vector-memory pipeline of a compute unit, which every request
// occupies for the same time whether it is served by HBM or by L2, has a third less to do.  A
// wave's share of K is at most 8 k-tiles (two requests of 4), less when the launch would
// otherwise have fewer than about 1500 waves; up to 16 waves along K per block are summed
// through LDS and, for the residual projections, K is also cut into slices over blocks that the
// next norm kernel sums.
template <int RT, int NT, int EPI, bool SPLIT, bool PACK>
static int launch_gemm_small_nt(GemmArgs a, int ks, hipStream_t s) {
  constexpr int U = 4;
  int KT = a.K / 32, groups = (a.n_tiles + NT - 1) / NT;
  int per_block = (KT + ks - 1) / ks;          // k-tiles of one block
  int nwk = NT;
  while (nwk < 16 && (per_block + nwk - 1) / nwk > 8) nwk *= 2;
  while (nwk < 16 && (long)groups * ks * nwk < 1500 && (per_block + nwk - 1) / nwk > 2) nwk *= 2;
  a.k_share = (per_block + nwk - 1) / nwk;
  dim3 grid(groups, ks);
  // a projection that completes the rows is not cut over blocks; with 6 k-tiles per wave (packed rows: also 8) it asks for
  // all of them at once instead of in two batches (K 3072, width 768: in two batches it cost more than the norm kernel it
  // replaces).  Shares of 5 and 7 take two batches, 4 + 1 and 4 + 3 k-tiles: the last ones are short, and
  // whole steps at d_ff 2560 and 3584 are no slower than with the norm kernel (widths 512-1024, 8 and 12 rows).
  if constexpr (EPI == EPI_RESID_NORM && NT == 1) {
    constexpr int UL = SPLIT ? 6 : 8;
    if (nwk == 16 && a.k_share > 4 && a.k_share <= UL) {
#define PD_LAUNCH_U(UU)                                                                                               \
  (a.stream_w ? launch_gemm_kernel<EPI>(k_gemm_s<RT, NT, 16, UU, EPI, SPLIT, PACK, false, true>, grid, 1024, a, s)    \
              : launch_gemm_kernel<EPI>(k_gemm_s<RT, NT, 16, UU, EPI, SPLIT, PACK>, grid, 1024, a, s))
      return a.k_share <= 6 ? PD_LAUNCH_U(6) : PD_LAUNCH_U(UL);
#undef PD_LAUNCH_U
    }
  }
  constexpr bool QKV_NORM = RT == 1 && (EPI == EPI_QKV || EPI == EPI_QKV_ROPE);
  constexpr bool DEF = norm_in_default(RT, EPI);
  int rc;
#define PD_LAUNCH_F(NWK, SWX, FI)                                                                                    \
  rc = launch_gemm_kernel<EPI>(k_gemm_s<RT, NT, (NWK < NT ? NT : NWK), U, EPI, SPLIT, PACK, false, SWX, FI>, grid,   \
                               64 * (NWK < NT ? NT : NWK), a, s)
#define PD_LAUNCH(NWK)                                                                                               \
  do {                                                                                                               \
    if (QKV_NORM && a.stats_in) {                                                                                    \
      if (a.stream_w) PD_LAUNCH_F(NWK, true, (QKV_NORM || DEF));                                                     \
      else PD_LAUNCH_F(NWK, false, (QKV_NORM || DEF));                                                               \
    } else if (a.stream_w) PD_LAUNCH_F(NWK, true, DEF);                                                              \
    else PD_LAUNCH_F(NWK, false, DEF);                                                                               \
  } while (0)
  switch (nwk) {
    case 1: PD_LAUNCH(1); break;
    case 2: PD_LAUNCH(2); break;
    case 4: PD_LAUNCH(4); break;
    case 8: PD_LAUNCH(8); break;
    default: PD_LAUNCH(16); break;
  }
#undef PD_LAUNCH
#undef PD_LAUNCH_F
  if (rc) return rc;
  if (EPI == EPI_RESID && a.parts_out) *a.parts_out = ks;
  return PD_OK;
}

template <int RT, int EPI, bool SPLIT, bool PACK>
static int launch_gemm_small(const GemmArgs &a, hipStream_t s) {
  int KT = a.K / 32, ks = 1;
  if (EPI == EPI_RESID)    // slices while the launch has fewer than 256 blocks and a slice keeps 8 k-tiles
    while (ks < a.max_parts && ((a.n_tiles + 1) / 2) * ks < 256 && KT / (2 * ks) >= 8) ks *= 2;
  if (RT == 1 && ((a.n_tiles + 1) / 2) * ks >= 128) return launch_gemm_small_nt<RT, 2, EPI, SPLIT, PACK>(a, ks, s);
  return launch_gemm_small_nt<RT, 1, EPI, SPLIT, PACK>(a, ks, s);
}

// 2, 4, 5 or 8 row tiles (many rows per request, many requests at once, prefill chunks).  Here the activation fragments of a
// block (32-128 rows x K, high and low parts) outweigh its weights, every block has to request all
// of them, and a compute unit's vector-memory pipeline is the limit, so what counts is how many
// requests the busiest compute unit issues: rounds of 256 blocks x k-tiles per block x (NT weight
// + 2 RT activation requests per k-tile).  The launch takes the column tiles per wave NT (and, for
// the residual projections, the K slices over blocks) that minimise this count -- typically the
// pair that makes exactly 256 blocks, one per compute unit: measured 29 us against 42 us for the
// QKV projection of cfg5 with 256 instead of 384 blocks.  Blocks are 4 waves along K (one wave per
// SIMD: registers for up to 8 x 4 accumulator tiles) and keep the compute unit to themselves.
template <int RT, int NT, int EPI, bool SPLIT>
static int launch_gemm_wide_nt(GemmArgs a, int ks, hipStream_t s) {
  constexpr int NWK = 4;
  constexpr int U = (NT + 2 * RT) <= 16 ? 4 : 2;
  int KT = a.K / 32, groups = (a.n_tiles + NT - 1) / NT;
  a.k_share = ((KT + ks - 1) / ks + NWK - 1) / NWK;
  const dim3 grid(groups, ks);
  const int rc = a.stream_w ? launch_gemm_kernel<EPI>(k_gemm_s<RT, NT, NWK, U, EPI, SPLIT, false, false, true>, grid, 64 * NWK, a, s)
                            : launch_gemm_kernel<EPI>(k_gemm_s<RT, NT, NWK, U, EPI, SPLIT, false>, grid, 64 * NWK, a, s);
  if (rc) return rc;
  if (EPI == EPI_RESID && a.parts_out) *a.parts_out = ks;
  return PD_OK;
}

template <int RT, int EPI, bool SPLIT>
static int launch_gemm_wide(const GemmArgs &a, hipStream_t s) {
  // 4 * NT * RT KiB of LDS, at most 128-160; with 2 row tiles more than 4 column tiles measured slower
  // (7 only with 5 row tiles: the vocabulary projection of a 72-row step without low parts then makes 449 blocks,
  // two rounds of one block per compute unit, instead of 524 with 6, where 12 blocks run a third round alone)
  constexpr int NT_MAX = RT <= 2 ? 4 : (RT <= 4 ? 8 : (RT == 5 ? 7 : 4));
  static const int nts[] = {1, 2, 3, 4, 6, 7, 8};
  int KT = a.K / 32, best_nt = 1, best_ks = 1;
  long best = -1;
  for (int ks = 1; ks <= (EPI == EPI_RESID ? a.max_parts : 1); ks *= 2) {
    if (ks > 1 && KT / ks < 8) break;
    for (int nt : nts) {
      if (nt > NT_MAX) break;
      if (nt == 7 && RT != 5) continue;
      long blocks = (long)((a.n_tiles + nt - 1) / nt) * ks;
      long rounds = (blocks + 255) / 256;
      long cost = rounds * ((KT + ks - 1) / ks) * (nt + 2 * RT);
      if (best < 0 || cost < best) { best = cost; best_nt = nt; best_ks = ks; }
    }
  }
  switch (best_nt) {
    case 1: return launch_gemm_wide_nt<RT, 1, EPI, SPLIT>(a, best_ks, s);
    case 2: return launch_gemm_wide_nt<RT, 2, EPI, SPLIT>(a, best_ks, s);
    case 3: return launch_gemm_wide_nt<RT, 3, EPI, SPLIT>(a, best_ks, s);
    case 4: return launch_gemm_wide_nt<RT, 4, EPI, SPLIT>(a, best_ks, s);
    case 6: return launch_gemm_wide_nt<RT, (NT_MAX >= 6 ? 6 : NT_MAX), EPI, SPLIT>(a, best_ks, s);
    case 7: return launch_gemm_wide_nt<RT, (RT == 5 ? 7 : 1), EPI, SPLIT>(a, best_ks, s);
    default: return launch_gemm_wide_nt<RT, (NT_MAX >= 8 ? 8 : NT_MAX), EPI, SPLIT>(a, best_ks, s);
  }
}


// 17-128 rows against a small weight matrix (at most 16 MB: what the L2 caches hold with room to spare).  One
// row tile and four column tiles per block instead of all row tiles and one column tile: a k-tile then costs a
// wave 4 weight + 2 activation requests for 4 output tiles, not 1 + 2 RT for RT, so the busiest compute unit
// issues about half the requests (its vector-memory pipeline is what bounds these launches), all requests
// of a wave go out in one batch, and 5 x 48 blocks fill the chip where 192 did not.  The weights are read
// once per row tile; block ids that differ by a multiple of 8 run on the same XCD (work-groups go to the
// XCDs round-robin), so with a number of column groups that is a multiple of 8 the row tiles of a group
// share one L2 and the repeats stay out of HBM.  Measured at 72 rows, width 1024 (cfg3): QKV 10.9 -> 6.9 us, first
// FFN projection 11.5 -> 9.5, output projection 4.0 (K slices of 8 k-tiles), second FFN projection 8.4 -> 7.7;
// 0.83 -> 0.76 ms per step.
// A projection that completes the residual rows and prepares the next norm (never cut along K over blocks)
// takes one column tile per block, so that the launch still has a block per compute unit: 64 x 5 at width 1024.
template <int EPI, bool SPLIT, int NT = 4>
static int launch_gemm_zrows(GemmArgs a, int rows, hipStream_t s) {
  constexpr int U = 4;
  const int KT = a.K / 32, groups = (a.n_tiles + NT - 1) / NT, rts = (rows + 15) / 16;
  // the residual projections also cut K into slices over blocks (summed by the next norm kernel) until the
  // launch has a block per compute unit
  int ks = 1;
  if (EPI == EPI_RESID)
    while (ks < a.max_parts && groups * rts * ks < 256 && KT / (2 * ks) >= 4) ks *= 2;
  const int per_block = (KT + ks - 1) / ks;
  // 4 or 8 waves along K (16 would leave a wave 128 registers, too few for 4 x 4 weight fragments in flight):
  // one batch of 4 k-tiles per wave up to K = 1024 per slice, two up to 2048.  A block of 8 waves has a compute
  // unit to itself; a launch of more than 256 blocks therefore takes 4 waves per block (two batches per wave),
  // so that all its blocks are resident at once instead of a few left over for a second round (320 blocks at
  // width 1024, 72 rows: first FFN projection 10.3 -> 9.3 us, second 8.1 -> 7.7)
  const int nwk = (per_block > 16 && (per_block > 64 || (long)groups * ks * rts <= 256)) ? 8 : 4;
  a.k_share = (per_block + nwk - 1) / nwk;
  dim3 grid(groups, ks, rts);
  constexpr bool DEF = norm_in_default(1, EPI), QKV_NORM = EPI == EPI_QKV || EPI == EPI_QKV_ROPE;
#define PD_LAUNCH(NWK, FI) launch_gemm_kernel<EPI>(k_gemm_s<1, NT, NWK, U, EPI, SPLIT, false, true, false, FI>, grid, 64 * NWK, a, s)
  int rc;
  if (QKV_NORM && a.stats_in) rc = nwk == 4 ? PD_LAUNCH(4, (QKV_NORM || DEF)) : PD_LAUNCH(8, (QKV_NORM || DEF));
  else rc = nwk == 4 ? PD_LAUNCH(4, DEF) : PD_LAUNCH(8, DEF);
#undef PD_LAUNCH
  if (rc) return rc;
  if (EPI == EPI_RESID && a.parts_out) *a.parts_out = ks;
  return PD_OK;
}

template <int EPI, bool SPLIT>
static int launch_gemm_split(const GemmArgs &a, int rows, hipStream_t s) {
  constexpr bool zrows = EPI != EPI_LM;
  if (zrows && mfma_gemm_row_tile_blocks(a.n_tiles, a.K, rows, EPI == EPI_RESID ? a.max_parts : 1))
    return launch_gemm_zrows<EPI, SPLIT, (EPI == EPI_RESID_NORM ? 1 : 4)>(a, rows, s);
  if (EPI == EPI_RESID_NORM || a.stats_in)
    PD_REQUIRE(rows <= 16, PD_EINVAL, "a projection of this shape cannot prepare or finish a norm for %d rows", rows);
  if (EPI == EPI_LM && SPLIT && vocab_shares_row_tiles(a.n_tiles, a.K / 32, rows)) return mfma_gemm_rows_epi5(a, rows, s);
  switch (mfma_gemm_row_tiles(rows)) {
    case 16: return launch_gemm_small<1, EPI, SPLIT, false>(a, s);
    case 32: return launch_gemm_wide<2, EPI, SPLIT>(a, s);
    case 64: return launch_gemm_wide<4, EPI, SPLIT>(a, s);
    case 80: return launch_gemm_wide<5, EPI, SPLIT>(a, s);
    default: return launch_gemm_wide<8, EPI, SPLIT>(a, s);
  }
}

template <int EPI>
static int launch_gemm(const GemmArgs &a, int rows, hipStream_t s) {
#if PD_GEMM_EPI == 6
  if (a.half_tiles) return launch_gemm_half<16>(a, s);
#endif
  if (EPI == EPI_RESID_NORM || a.stats_in)
    PD_REQUIRE(rows <= 128 && a.R <= 128, PD_EINVAL,
               "projections that prepare or finish a norm take at most 128 rows (%d)", rows);
  if constexpr (EPI != EPI_RESID_NORM) {
    if (rows > 128) {
      PD_REQUIRE(!a.packed, PD_EINVAL, "packed activations hold at most 8 rows (%d)", rows);
      return PD_GEMM_ROWS_ENTRY(a, rows, s);
    }
  }
  if (a.packed) {
    PD_REQUIRE(rows <= 8 && a.R <= 8, PD_EINVAL, "packed activations hold at most 8 rows (%d)", rows);
    return launch_gemm_small<1, EPI, false, true>(a, s);
  }
  return a.xn_lo ? launch_gemm_split<EPI, true>(a, rows, s) : launch_gemm_split<EPI, false>(a, rows, s);
}

int PD_GEMM_ENTRY(const GemmArgs &a, int rows, hipStream_t s) { return launch_gemm<PD_GEMM_EPI>(a, rows, s); }

#else   // ---- more than 128 rows, and the vocabulary projection of 33-128 -------------------------

// ---------------------------------------------------------------------------
// More than 128 rows against matrices that make the multiplies the bound (the context pass, large teacher-forced
// passes; also the vocabulary projection of 33-128 rows, see launch_gemm_vocab): grid (column groups, K slices, groups
// of 16 RT rows).  A block is NW = 8 waves (two per SIMD: a single wave issues a 16x16x32 multiply every 29 clocks, two
// or more every 19) that own NT column tiles each and share the RT row tiles of their row group: per k-tile every wave
// requests its share of the activation fragments (high and low parts) and its own weight fragments, two k-tiles ahead;
// the activation fragments pass through LDS (two buffers), and every wave multiplies all of them with its weights.
// One barrier per k-tile, in the middle of its multiplies: the fragments of a k-tile go from LDS to the matrix cores
// in groups of GS, the group after next is requested when a group has been multiplied, and behind the barrier that
// request already goes to the next k-tile's buffer.  So a wave never stands between a barrier and its first multiply
// waiting for LDS (with the barrier in front of the k-tile's first LDS read the same launches took: QKV, 2048 rows,
// width 4096, 327 us, now 310; QKV, 4096 rows, width 2048, 182 -> 173; second FFN projection there 204 -> 198).
// At these sizes the multiplies run at 1.1-1.4 PFLOP/s (high and low parts counted), what a large library product
// reaches on this device: with operands of zeros the same launches are 20-30 % faster, so it is the power limit
// that holds the rate, and 32x32x16 multiplies (half the operand reads) measured no better (239 against 226 us).
// ---------------------------------------------------------------------------
template <int RT, int NT, int EPI, bool SPLIT, bool SW = false>
__global__ __launch_bounds__(512, 1) void k_gemm_t(PD_GEMM_HOT_PARAMS, GemmArgs a) {
  constexpr int NW = 8, NA = SPLIT ? 2 * RT : RT;     // activation fragments of a k-tile
  constexpr int NAW = (NA + NW - 1) / NW;             // staged by one wave (no multiple of the waves: some twice, same bytes)
  constexpr int GS = RT == 5 ? 5 : 4, NG = NA / GS;
  static_assert(NA % GS == 0 && (NG == 1 || NG % 2 == 0), "fragment groups alternate between two register sets");
  __shared__ bf16x8 sm_x[2][NA][64];   // (vector types throughout: struct copies would keep xr in scratch memory)
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int m = lane & 15;
  const int KT = words_k_tiles(hot_k), per_slice = words_k_tiles(hot_share), n_tiles = words_tiles(hot_n);
  const int kt0 = min((int)blockIdx.y * per_slice, KT), kt1 = min(kt0 + per_slice, KT);
  const int rt0 = blockIdx.z * RT, r0 = rt0 * 16;
  const int nt0 = (blockIdx.x * NW + w) * NT;
  floatx4 acc[NT][RT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int i = 0; i < RT; ++i) acc[t][i] = floatx4{0.f, 0.f, 0.f, 0.f};
  const bf16x8 *wsrc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)          // tiles past the end repeat the last one
    wsrc[t] = (const bf16x8 *)hot_w + (size_t)min(nt0 + t, n_tiles - 1) * KT * 64 + lane;
  // this wave's share of the activation fragments: fragment f is row tile f % RT of the high (f < RT) or low parts
  const bf16x8 *xsrc[NAW];
#pragma unroll
  for (int i = 0; i < NAW; ++i) {
    const int f = (w * NAW + i) % NA;
    xsrc[i] = (const bf16x8 *)hot_x + (SPLIT && f >= RT ? words_granules(hot_lo) : 0) + (size_t)(rt0 + f % RT) * KT * 64 + lane;
  }
  const int len = kt1 - kt0;
  bf16x8 xr[2][NAW], wr[2][NT];         // k-tiles in flight, slot = k-tile index mod 2; past the end: the last one again
  auto load_x = [&](int s, int j) {
    const size_t k = (size_t)(kt0 + min(j, len - 1)) * 64;
#pragma unroll
    for (int i = 0; i < NAW; ++i) xr[s][i] = xsrc[i][k];
  };
  auto load_w = [&](int s, int j) {
    const size_t k = (size_t)(kt0 + min(j, len - 1)) * 64;
#pragma unroll
    for (int t = 0; t < NT; ++t) wr[s][t] = ld_w<SW>((const uint4 *)(wsrc[t] + k));
  };
  auto put_x = [&](int s) {
#pragma unroll
    for (int i = 0; i < NAW; ++i) sm_x[s][(w * NAW + i) % NA][lane] = xr[s][i];
  };
  if (len > 0) {                        // the same for the whole block
    load_x(0, 0); load_w(0, 0);
    load_x(1, 1); load_w(1, 1);
    put_x(0);
    load_x(0, 2);
    __syncthreads();
    Frag xg[2][GS];
#pragma unroll
    for (int h = 0; h < (NG == 1 ? 1 : 2); ++h)
#pragma unroll
      for (int u = 0; u < GS; ++u) xg[h][u].v = sm_x[0][h * GS + u][lane];
    for (int j0 = 0; j0 < len; j0 += 2) {
#pragma unroll
      for (int d = 0; d < 2; ++d) {
        const int j = j0 + d;
        if (j < len) {                  // the same for every wave of the block
          // k-tile j + 1 goes to the other buffer (its last readers, of k-tile j - 1, are behind the barrier of
          // k-tile j - 1); the slots are refilled two k-tiles on
          put_x(d ^ 1);
          load_x(d ^ 1, j + 3);
          Frag wc[NT];
#pragma unroll
          for (int t = 0; t < NT; ++t) wc[t].v = wr[d][t];
          load_w(d, j + 2);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int gi = 0; gi < NG; ++gi) {
#pragma unroll
            for (int u = 0; u < GS; ++u)
#pragma unroll
              for (int t = 0; t < NT; ++t)
                acc[t][(gi * GS + u) % RT] = mfma16(wc[t], xg[gi & 1][u], acc[t][(gi * GS + u) % RT]);
            __builtin_amdgcn_sched_barrier(0);
            if (gi == (NG == 1 ? 0 : NG - 2)) {
              __syncthreads();          // k-tile j + 1 is in LDS, nobody reads k-tile j there any more
              __builtin_amdgcn_sched_barrier(0);
            }
            const int gn = NG == 1 ? 1 : gi + 2;      // the group that takes this one's registers
#pragma unroll
            for (int u = 0; u < GS; ++u)
              xg[gi & 1][u].v = gn < NG ? sm_x[d][gn * GS + u][lane] : sm_x[d ^ 1][(gn - NG) * GS + u][lane];
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
    }
  }
  // row data of the epilogue (asked for here: it would cost the loop 4 RT registers)
  constexpr bool QKV = EPI == EPI_QKV || EPI == EPI_QKV_ROPE;
  int4 kvi[QKV ? RT : 1];
  if (QKV) {
#pragma unroll
    for (int i = 0; i < RT; ++i) kvi[i] = ((const int4 *)hot_c)[r0 + i * 16 + m];
  }
  Winner win[EPI == EPI_LM ? RT : 1];
  if (EPI == EPI_LM)
#pragma unroll
    for (int i = 0; i < RT; ++i) win[i] = Winner{-INFINITY, NO_WINNER};
#pragma unroll
  for (int t = 0; t < NT; ++t)
    if (nt0 + t < n_tiles) gemm_epilogue<RT, EPI>(a, nt0 + t, acc[t], kvi, lane, r0, nullptr, nullptr, nullptr, win);
  if constexpr (EPI == EPI_LM) store_winners<RT, NW>(a, win, w, lane, r0);
}

template <int RT, int NT, int EPI, bool SPLIT>
static int launch_gemm_t(GemmArgs a, int rows, int ks, hipStream_t s) {
  dim3 grid((a.n_tiles + 8 * NT - 1) / (8 * NT), ks, (rows + 16 * RT - 1) / (16 * RT));
  a.k_share = (a.K / 32 + ks - 1) / ks;
  const int rc = launch_gemm_kernel<EPI>(k_gemm_t<RT, NT, EPI, SPLIT>, grid, 512, a, s);
  if (rc) return rc;
  if (EPI == EPI_RESID && a.parts_out) *a.parts_out = ks;
  return PD_OK;
}

// The waves of a block cut K (k_gemm_s), RT row tiles and NT column tiles per block.
template <int RT, int NT, int NWK, int EPI, bool SPLIT>
static int launch_gemm_cut(GemmArgs a, int rows, int ks, hipStream_t s) {
  a.k_share = ((a.K / 32 + ks - 1) / ks + NWK - 1) / NWK;
  dim3 grid((a.n_tiles + NT - 1) / NT, ks, (rows + 16 * RT - 1) / (16 * RT));
  const int rc = launch_gemm_kernel<EPI>(k_gemm_s<RT, NT, NWK, 4, EPI, SPLIT, false, true>, grid, 64 * NWK, a, s);
  if (rc) return rc;
  if (EPI == EPI_RESID && a.parts_out) *a.parts_out = ks;
  return PD_OK;
}

// The tiling is the candidate that should end first (row_tiling).  Small tiles whose waves cut K keep no barrier in their loop
// and fill the chip: 192 rows, K 768, N 3072 5.7 us against 28 with 128 x 256 tiles (24 blocks), 512 rows 9.9 against 28;
// from about 1024 rows the requests for their operands outweigh (2048 rows: 32 against 26).
template <int EPI, bool SPLIT>
static int launch_gemm_rows(const GemmArgs &a, int rows, hipStream_t s) {
  constexpr RowOutput OUT = EPI == EPI_RESID ? ROWS_SLICES : EPI == EPI_LM ? ROWS_VOCAB
                          : EPI == EPI_SWIGLU ? ROWS_GATED : ROWS_STORED;
  const RowTiling t = row_tiling(a.n_tiles, a.K / 32, rows, a.max_parts, SPLIT, OUT);
  if (t.cut) {
    if (t.nt == 6) return launch_gemm_cut<2, 6, 4, EPI, SPLIT>(a, rows, t.ks, s);
    if (t.nt == 4) return launch_gemm_cut<2, 4, 8, EPI, SPLIT>(a, rows, t.ks, s);
    return launch_gemm_cut<2, 2, 4, EPI, SPLIT>(a, rows, t.ks, s);
  }
  if (t.rt == 8) {
    if (t.nt == 4) return launch_gemm_t<8, 4, EPI, SPLIT>(a, rows, t.ks, s);
    if (t.nt == 3) return launch_gemm_t<8, 3, EPI, SPLIT>(a, rows, t.ks, s);
    return launch_gemm_t<8, 2, EPI, SPLIT>(a, rows, t.ks, s);
  }
  switch (t.nt) {
    case 1: return launch_gemm_t<4, 1, EPI, SPLIT>(a, rows, t.ks, s);
    case 2: return launch_gemm_t<4, 2, EPI, SPLIT>(a, rows, t.ks, s);
    case 3: return launch_gemm_t<4, 3, EPI, SPLIT>(a, rows, t.ks, s);
    default: return launch_gemm_t<4, 4, EPI, SPLIT>(a, rows, t.ks, s);
  }
}

#if PD_GEMM_EPI == 5     // EPI_LM
// Vocabulary projection of 33-128 rows: the same kernel with all rows in one group and one or two column tiles per
// wave.  Cut along K over 4 waves (launch_gemm_wide) every wave requests a few k-tiles, waits for all of them, multiplies,
// and the blocks end with a sum through LDS; one stream of k-tiles per block hides both.  One layer + vocabulary, us per
// step, before -> after: 72 rows, width 1024, 50265 words 83.3 -> 73.3 (the projection itself 40.7 -> 31), 128 rows
// 113 -> 83, 120000 words 190 -> 138; 64 rows, width 512, 32000 words 55.6 -> 52.2; width 4096, 100000 words 315 -> 276.
// From which sizes on: vocab_shares_row_tiles.  Two column tiles per wave where one makes more than a round of blocks and a
// block's multiplies cover its requests (64 rows, width 1024, 50265 words 67.2 with one, 72.7 with two; 72 rows of width
// 768 66.6 and 65.3; 128 rows of width 2048 148 and 139); three, or four k-tiles ahead instead of two, measured no better.
// Steps of 17-32 rows differ by less than 5 % either way and stay.
template <int RT, int NT>
static int launch_gemm_vocab(GemmArgs a, int rows, hipStream_t s) {
  PD_REQUIRE(rows <= 16 * RT, PD_EINVAL, "%d rows in %d row tiles", rows, RT);
  const dim3 grid((a.n_tiles + 8 * NT - 1) / (8 * NT));
  a.k_share = a.K / 32;
  return a.stream_w ? launch_gemm_kernel<EPI_LM>(k_gemm_t<RT, NT, EPI_LM, true, true>, grid, 512, a, s)
                    : launch_gemm_kernel<EPI_LM>(k_gemm_t<RT, NT, EPI_LM, true, false>, grid, 512, a, s);
}

static int launch_gemm_vocab_rows(const GemmArgs &a, int rows, hipStream_t s) {
  const int rt = mfma_gemm_row_tiles(rows) / 16, KT = a.K / 32;
  const bool two = a.n_tiles > 2048 && (rt * KT >= 160 || a.n_tiles > 4096);
  if (rt == 4) return two ? launch_gemm_vocab<4, 2>(a, rows, s) : launch_gemm_vocab<4, 1>(a, rows, s);
  if (rt == 5) return two ? launch_gemm_vocab<5, 2>(a, rows, s) : launch_gemm_vocab<5, 1>(a, rows, s);
  return two ? launch_gemm_vocab<8, 2>(a, rows, s) : launch_gemm_vocab<8, 1>(a, rows, s);
}
#endif

int PD_GEMM_ROWS_ENTRY(const GemmArgs &a, int rows, hipStream_t s) {
  constexpr int EPI = PD_GEMM_EPI;
#if PD_GEMM_EPI == 5
  if (rows <= 128) return launch_gemm_vocab_rows(a, rows, s);
#endif
  return a.xn_lo ? launch_gemm_rows<EPI, true>(a, rows, s) : launch_gemm_rows<EPI, false>(a, rows, s);
}

#endif

#else   // ---- common part: dispatcher ----------------------------------------------------------

// 17-128 rows against a weight matrix of at most 16 MB (17-32 rows: 64 MB; the blocks of both row tiles are then
// resident together and the second reader of a weight line finds it in L2) and a K that 8 waves (times the K
// slices over blocks) cover in batches of 4 k-tiles: the launch gives every row tile blocks of its own
// (launch_gemm_zrows)
bool mfma_gemm_row_tile_blocks(int n_tiles, int K, int rows, int k_slices) {
  const size_t bytes = (size_t)n_tiles * 16 * K * 2;
  return rows > 16 && rows <= 128 && (bytes <= ((size_t)16 << 20) || (rows <= 32 && bytes <= ((size_t)64 << 20))) &&
         K / 32 <= 64 * k_slices;
}

int mfma_gemm_row_tiles(int rows) {
  int rt = (rows + 15) / 16;
  return (rt <= 1 ? 1 : rt <= 2 ? 2 : rt <= 4 ? 4 : rt <= 5 ? 5 : 8) * 16;
}

int mfma_gemm_epi0(const GemmArgs &a, int rows, hipStream_t s);
int mfma_gemm_epi1(const GemmArgs &a, int rows, hipStream_t s);
int mfma_gemm_epi2(const GemmArgs &a, int rows, hipStream_t s);
int mfma_gemm_epi3(const GemmArgs &a, int rows, hipStream_t s);
int mfma_gemm_epi4(const GemmArgs &a, int rows, hipStream_t s);
int mfma_gemm_epi5(const GemmArgs &a, int rows, hipStream_t s);
int mfma_gemm_epi6(const GemmArgs &a, int rows, hipStream_t s);

int mfma_gemm(int epi, const GemmArgs &a, int rows, hipStream_t s) {
  switch (epi) {
    case EPI_QKV: return mfma_gemm_epi0(a, rows, s);
    case EPI_QKV_ROPE: return mfma_gemm_epi1(a, rows, s);
    case EPI_RESID: return mfma_gemm_epi2(a, rows, s);
    case EPI_GELU: return mfma_gemm_epi3(a, rows, s);
    case EPI_SWIGLU: return mfma_gemm_epi4(a, rows, s);
    case EPI_LM: return mfma_gemm_epi5(a, rows, s);
    case EPI_RESID_NORM: return mfma_gemm_epi6(a, rows, s);
  }
  pd_set_error("unknown epilogue %d", epi);
  return PD_EINVAL;
}

#endif
