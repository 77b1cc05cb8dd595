// fp32-activation kernels.  They serve dtype 0 (fp32 weights and KV cache) and, for bf16 weights whose
// shapes the bf16 matrix-core kernels do not cover, dtype 1 with fp32 activations.
// KV cache layout on this path: K [B][H][kv_cap][hd], V [B][H][hd][kv_cap] (a lane's four values of either are then
// consecutive in the order in which the products want them).
//
// All products run on the matrix cores in fp32 (16x16x4, fp32 operands and accumulators: a chain of fused
// multiply-adds, no reduced precision anywhere).  A lane holds four consecutive contraction values of one row of
// either operand (one 16-byte load) and feeds them to four instructions; which contraction value meets which
// instruction does not matter as long as both operands agree.
// The models of this path are small, so a decode step is a chain of launches of a few microseconds each and their
// number decides: five per layer (QKV with the norm in front of it and the KV append behind it, attention, output
// projection, the two FFN projections, the first with its norm), the embedding read by the first of them and the
// argmax left as one winner per 16-column tile for k_turn.
#include "launch_rules.h"
#include "pd_internal.h"

#include <algorithm>
#include <type_traits>

typedef float floatx4 __attribute__((ext_vector_type(4)));

// four consecutive values as fp32 (the address is aligned to the four of them)
__device__ __forceinline__ floatx4 ld4(const float *p) { return *(const floatx4 *)p; }
__device__ __forceinline__ floatx4 ld4(const bf16_t *p) {
  const uint2 u = *(const uint2 *)p;
  return floatx4{__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16),
                 __uint_as_float(u.y & 0xffff0000u)};
}
__device__ __forceinline__ floatx4 ld4(const f16_t *p) {
  union { uint2 u; f16_t h[4]; } v;
  v.u = *(const uint2 *)p;
  return floatx4{(float)v.h[0], (float)v.h[1], (float)v.h[2], (float)v.h[3]};
}
// values k .. k+3 of a row of n; VEC: n is a multiple of 4 and the row aligned.  Beyond the row: the values at the
// nearest place that exists (the caller multiplies them by zero or masks them).
template <bool VEC, typename T>
__device__ __forceinline__ floatx4 ld_row4(const T *row, int k, int n) {
  if (VEC) return ld4(row + min(k, n - 4));
  floatx4 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = ld_f32(row, (size_t)min(k + e, n - 1));
  return v;
}

__device__ __forceinline__ floatx4 mfma_f32(float a, float b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// ---------------------------------------------------------------------------
// norm: xn[r] = LayerNorm(x[r]) or RMSNorm(x[r]); one block per row
// ---------------------------------------------------------------------------
__device__ __forceinline__ float block_sum(float v, float *sh) {
  v = fold_wave(v, Add());
  int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[w] = v;
  __syncthreads();
  float t = 0.f;
  for (int i = 0; i < nw; ++i) t += sh[i];
  return t;
}

__global__ void k_norm_f32(float *xn, const float *x, const float *g, const float *b, int d,
                           int kind, float eps, const int32_t *flags) {
  __shared__ float sh[16];
  int r = blockIdx.x;
  if (!(flags[r] & ROW_VALID)) return;
  const float *xr = x + (size_t)r * d;
  float s = 0.f;
  for (int c = threadIdx.x; c < d; c += blockDim.x) s += xr[c];
  float mean = kind == 0 ? block_sum(s, sh) / d : 0.f;
  float v = 0.f;
  for (int c = threadIdx.x; c < d; c += blockDim.x) { float t = xr[c] - mean; v += t * t; }
  float rstd = rsqrtf(block_sum(v, sh) / d + eps);
  for (int c = threadIdx.x; c < d; c += blockDim.x) {
    float t = (xr[c] - mean) * rstd * g[c];
    if (kind == 0 && b) t += b[c];
    xn[(size_t)r * d + c] = t;
  }
}

// ---------------------------------------------------------------------------
// linear: y[r][n] = sum_k u(x)[r][k] * W[n][k], u = identity or the norm of the row
// ---------------------------------------------------------------------------
enum { LIN_STORE = 0, LIN_RESID = 1, LIN_GELU = 2, LIN_SWIGLU = 3, LIN_QKV = 4, LIN_HEAD = 5, LIN_SLICE = 6 };
constexpr int SLICES = 4;      // LIN_SLICE: cuts of K over blocks

struct LinArgs {
  const float *x;                     // [R][K]
  const void *W, *W2;                 // row-major [N][K]; W2: the up matrix of LIN_SWIGLU
  int R, N, K;
  const float *ng, *nb; int norm_kind; float eps;   // NORM launches: gain, bias (or NULL)
  // rows gathered instead of read (first layer): x = tok_emb[tok] (+ pos_emb[pos]); LIN_RESID: the residual, not x
  const void *tok_emb, *pos_emb;      // tok_emb NULL: rows of x
  RowTables rt;
  float *out; int ldo;
  const float *res;                   // LIN_RESID (may be out itself)
  // slices [SLICES][slice_stride] that the rows of x (of the residual) still lack, or NULL; LIN_SLICE: where its own go
  const float *pend; size_t slice_stride;
  void *kc, *vc, *kc_lo, *vc_lo; int d, H, hd, kv_cap; int32_t *kv_sat;   // LIN_QKV
  int sec0;                           // ... section of the first column (0: Q, K, V follow; 1: K, V only)
  float *logits; int S;               // LIN_HEAD: NULL, or [B][S][N] addressed by a row's request and subsequence
  float *part_val; int32_t *part_idx; int n_tiles;
};

// Where the rows that a launch normalises (LIN_RESID: adds to) come from: a buffer, a buffer and the slices it still lacks, or the
// embedding tables.  A part of the kernel's type: decided at run time, every row was read in branches of its own, each waited
// for before the next row was asked for (8 rows of width 64 from the tables: QKV 6.6 -> 5.2 us, from the buffer FFN 5.2 -> 4.4).
enum { SRC_ROWS = 0, SRC_SLICES = 1, SRC_GATHER = 2 };
constexpr int row_parts(int src) { return src == SRC_SLICES ? 1 + SLICES : src == SRC_GATHER ? 2 : 1; }
struct RowState { bool valid, learned; };            // SRC_GATHER: the row carries a token; positions are learned

// first: buffer or token table; second: slices or position table
template <typename WT, int SRC>
struct RowSrc {
  const float *x; size_t stride; const WT *te, *pe; RowState state;
  __device__ __forceinline__ RowSrc(const LinArgs &a, const void *first, const void *second, int r, int ld)
      : x(nullptr), stride(0), te(nullptr), pe(nullptr), state{true, true} {
    if (SRC == SRC_GATHER) {
      gather(first, second, a.rt.flags[r], a.rt.tok[r], a.rt.pos[r], ld);     // (independent reads)
    } else {
      x = (const float *)first + (size_t)r * ld;
      if (SRC == SRC_SLICES) { pe = (const WT *)((const float *)second + (size_t)r * ld); stride = a.slice_stride; }
    }
  }
  __device__ __forceinline__ RowSrc(const void *first, const void *second, int fl, int tok, int pos, int ld) : x(nullptr), stride(0) {
    gather(first, second, fl, tok, pos, ld);
  }
  __device__ __forceinline__ void gather(const void *first, const void *second, int fl, int tok, int pos, int ld) {
    // (places are masked, not chosen: a choice would put a read into a branch)
    const int has = -(fl & ROW_VALID), lp = second ? -1 : 0;
    static_assert(ROW_VALID == 1, "a mask by negation");
    state = RowState{has != 0, lp != 0};
    te = (const WT *)first + (size_t)(tok & has) * ld;
    pe = (const WT *)(second ? second : first) + (size_t)(((pos & lp) | (tok & ~lp)) & has) * ld;    // (no positions: the token's again)
  }
  // in two parts: the second waits for the argument struct where there are slices
  template <bool VEC> __device__ __forceinline__ void ask(floatx4 (&q)[row_parts(SRC)], int k, int n) const {
    q[0] = SRC == SRC_GATHER ? ld_row4<VEC>(te, k, n) : ld_row4<VEC>(x, k, n);
  }
  template <bool VEC> __device__ __forceinline__ void ask_rest(floatx4 (&q)[row_parts(SRC)], int k, int n) const {
#pragma unroll
    for (int i = 1; i < row_parts(SRC); ++i)
      q[i] = SRC == SRC_GATHER ? ld_row4<VEC>(pe, k, n) : ld_row4<VEC>((const float *)pe + (i - 1) * stride, k, n);
  }
};
template <int SRC>
__device__ __forceinline__ floatx4 row_value(const floatx4 (&q)[row_parts(SRC)], RowState state) {
  constexpr int N = row_parts(SRC) - 1;
  if (SRC == SRC_ROWS) return q[0];
  if (SRC == SRC_SLICES) return q[0] + ((q[min(1, N)] + q[min(2, N)]) + (q[min(3, N)] + q[N]));
  floatx4 y;
#pragma unroll
  for (int e = 0; e < 4; ++e) y[e] = state.valid ? (state.learned ? q[0][e] + q[N][e] : q[0][e]) : 0.f;
  return y;
}

// A block owns one 16-column tile and RT tiles of 16 rows; its NW waves cut K in steps of 16, the partial tiles are
// summed through LDS.  VPL > 0: the rows are normalised first (K <= 256 VPL).  Every wave reads 16 / NW rows once,
// whole (VPL quads per lane), takes mean and variance in registers (two passes) and leaves the normalised row in LDS;
// the first weights are requested before that (by the leading arguments, which arrive in registers).  Bound by latency at the
// sizes of this path: enough waves that each has one or two batches of requests (512 x 2048, 12 rows: 13.5 us with a wave per
// column, 6-7 so), and every request of the first batch in flight before anything is waited for, as far as registers go: 16
// waves have 128 each, and beyond that everything in flight goes through scratch memory (rows of four quads with their slices beside
// gain, bias and weights; two matrices beside two sets of rows; a place for every value of a scalar load.  us per step of 4
// layers with spills / without: width 768, 12 rows 175.8 / 157.7, 1024 193.9 / 174.4, gated 1280 337.7 / 320.3, scalar
// loads 650 346 / 310, gated 371 / 319).
template <typename WT, typename KT, int EPI, int NW, int RT, int VPL, bool VEC, int SRC>
__global__ __launch_bounds__(64 * NW) void k_lin(const void *hot_x, const void *hot_w, const void *hot_w2, const float *hot_g,
                                                   const float *hot_b, const int4 *hot_info, int R, int K, LinArgs a) {
  // (hot_x: the rows or, of normed gathered ones, the token table; hot_w2: the second matrix of LIN_SWIGLU, else RowSrc's second)
  const int N = a.N;
  constexpr bool NORM = VPL > 0;
  constexpr int NT = EPI == LIN_SWIGLU ? 2 : 1, U = VEC || NT == 1 ? 4 : 2;
  constexpr int XLD = NORM ? 256 * VPL + 4 : 4;      // (+ 4: the 16 rows of a step lie in different banks)
  static_assert(!NORM || RT == 1, "row statistics are taken for one row tile");
  static_assert(SRC == SRC_ROWS || (EPI != LIN_SWIGLU && (NORM || EPI == LIN_RESID)), "rows put together: normed, or the residual");
  __shared__ floatx4 red[NW][NT * RT][64];
  __shared__ float sm_x[NORM ? 16 : 1][XLD];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
  const int r0 = blockIdx.y * 16 * RT, n0 = blockIdx.x * 16;
  const int all = (K + 15) >> 4, steps = EPI == LIN_SLICE ? (all + SLICES - 1) / SLICES : all, share = (steps + NW - 1) / NW;
  const int b0 = EPI == LIN_SLICE ? min((int)blockIdx.z * steps, all) : 0, b1 = min(b0 + steps, all);
  const int s0 = min(b0 + w * share, b1), s1 = min(s0 + share, b1);
  const WT *wrow[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) wrow[t] = (const WT *)(t ? hot_w2 : hot_w) + (size_t)min(n0 + m, N - 1) * K;
  // weights of U steps (beyond the share: the last place again, not multiplied)
  auto load_w = [&](floatx4 (&wv)[NT][U], int s) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int u = 0; u < U; ++u) wv[t][u] = ld_row4<VEC>(wrow[t], min(s + u, max(s1 - 1, 0)) * 16 + 4 * g, K);
  };
  floatx4 wv[NT][U];
  constexpr int RPW = NORM ? 16 / NW : 1, VP = NORM ? VPL : 1;      // rows per wave, quads per lane
  constexpr int NSRC = NORM ? SRC : SRC_ROWS, RSRC = EPI == LIN_RESID ? SRC : SRC_ROWS;
  static_assert(VP < 4 || RPW == 1, "a wave holds one row of four quads a lane");
  floatx4 xq[RPW][VP][row_parts(NSRC)], gv[VP], bv[VP];
  RowState xs[RPW];
  // (rows before weights: the number of columns is in the argument struct, which is still on its way)
  // a batch's rows are requested with its weights, or when it begins where two matrices or scalar loads leave no registers
  constexpr bool AHEAD = !NORM && RT == 1 && NT == 1 && VEC;
  floatx4 xv[RT][U];
  auto load_x = [&](floatx4 (&xv)[RT][U], int s) {
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      const float *row = (const float *)hot_x + (size_t)min(r0 + i * 16 + m, R - 1) * K;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = min(s + u, max(s1 - 1, 0)) * 16 + 4 * g;
        if constexpr (NORM) xv[i][u] = *(const floatx4 *)&sm_x[m][min(k, XLD - 4)];
        else xv[i][u] = ld_row4<VEC>(row, k, K);
      }
    }
  };
  // gain and bias: with everything else or, where rows of four quads and their slices fill a wave's registers, under the sums
  // (scalar loads: such rows and slices in two halves, more than 63 requests wait for each other)
  constexpr bool LATE_GAIN = NORM && VPL == 4 && SRC == SRC_SLICES;
  constexpr int QB = LATE_GAIN && !VEC ? VP / 2 : VP;
  auto load_gain = [&]() {
#pragma unroll
    for (int v = 0; v < VP; ++v) {
      gv[v] = ld_row4<VEC>(hot_g, 4 * (lane + 64 * v), K);
      bv[v] = ld_row4<VEC>(hot_b ? hot_b : hot_g, 4 * (lane + 64 * v), K);
    }
  };
  if (AHEAD) load_x(xv, s0);
  if constexpr (!NORM) load_w(wv, s0);
  if constexpr (NORM) {
    auto row = [&](int i) { return RowSrc<WT, NSRC>(a, hot_x, hot_w2, min(r0 + w * RPW + i, R - 1), K); };
    if (SRC != SRC_GATHER)
#pragma unroll
      for (int i = 0; i < RPW; ++i)
#pragma unroll
        for (int v = 0; v < QB; ++v) row(i).template ask<VEC>(xq[i][v], 4 * (lane + 64 * v), K);
    if (!LATE_GAIN) load_gain();
    int fl = 0, tok = 0, pos = 0;         // lane i: of row i (read one by one they were waited for one by one)
    if (SRC == SRC_GATHER) {
      const int rl = min(r0 + w * RPW + lane % RPW, R - 1);
      fl = a.rt.flags[rl]; tok = a.rt.tok[rl]; pos = a.rt.pos[rl];
    }
    load_w(wv, s0);
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
      const RowSrc<WT, NSRC> src = SRC == SRC_GATHER
          ? RowSrc<WT, NSRC>(hot_x, hot_w2, __builtin_amdgcn_readlane(fl, i), __builtin_amdgcn_readlane(tok, i), __builtin_amdgcn_readlane(pos, i), K)
          : row(i);
      xs[i] = src.state;
#pragma unroll
      for (int v = 0; v < QB; ++v) {
        if (SRC == SRC_GATHER) src.template ask<VEC>(xq[i][v], 4 * (lane + 64 * v), K);
        src.template ask_rest<VEC>(xq[i][v], 4 * (lane + 64 * v), K);
      }
    }
  }
  // what the finishing waves need from memory: the residual rows, where a row's results go
  const int rf = min(r0 + min(w, RT - 1) * 16 + m, R - 1);
  floatx4 rq[row_parts(RSRC)];
  RowState rs{true, true};
  if constexpr (EPI == LIN_RESID) {
    if (w < RT) {                       // (asked for by every wave, five quads each of 16 rows: 8.1 us where 4.4 will do)
      const RowSrc<WT, RSRC> src(a, SRC == SRC_GATHER ? a.tok_emb : (const void *)a.res, hot_w2, rf, N);
      rs = src.state;
      if (VEC && N % 4 == 0) {
        src.template ask<true>(rq, n0 + 4 * g, N);
        src.template ask_rest<true>(rq, n0 + 4 * g, N);
      } else {
        src.template ask<false>(rq, n0 + 4 * g, N);
        src.template ask_rest<false>(rq, n0 + 4 * g, N);
      }
    }
  }
  int4 info = make_int4(0, 0, 0, 0);                                // {flags, req, slot, pos}; {flags, sub, lim, req}
  if ((EPI == LIN_QKV || EPI == LIN_HEAD) && !LATE_GAIN) info = hot_info[rf];
  if constexpr (NORM) {
    __builtin_amdgcn_sched_barrier(0);
    floatx4 nx[RPW][VPL];
    float s[RPW], q[RPW];
#pragma unroll
    for (int i = 0; i < RPW; ++i)
#pragma unroll
      for (int v = 0; v < QB; ++v) nx[i][v] = row_value<NSRC>(xq[i][v], xs[i]);
    if constexpr (QB < VP) {
      __builtin_amdgcn_sched_barrier(0);
      const RowSrc<WT, NSRC> src(a, hot_x, hot_w2, min(r0 + w, R - 1), K);
#pragma unroll
      for (int v = 0; v < QB; ++v) {
        src.template ask<VEC>(xq[0][v], 4 * (lane + 64 * (QB + v)), K);
        src.template ask_rest<VEC>(xq[0][v], 4 * (lane + 64 * (QB + v)), K);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int v = 0; v < QB; ++v) nx[0][QB + v] = row_value<NSRC>(xq[0][v], xs[0]);
    }
    if (LATE_GAIN) {
      __builtin_amdgcn_sched_barrier(0);
      load_gain();
      if (EPI == LIN_QKV || EPI == LIN_HEAD) info = hot_info[rf];
    }
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
      s[i] = 0.f;
      if (a.norm_kind == 0)
#pragma unroll
        for (int v = 0; v < VPL; ++v)
#pragma unroll
          for (int e = 0; e < 4; ++e) s[i] += 4 * (lane + 64 * v) + e < K ? nx[i][v][e] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < RPW; ++i) s[i] = fold_wave(s[i], Add());
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
      s[i] /= K;
      q[i] = 0.f;
#pragma unroll
      for (int v = 0; v < VPL; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e) { const float t = nx[i][v][e] - s[i]; q[i] += 4 * (lane + 64 * v) + e < K ? t * t : 0.f; }
    }
#pragma unroll
    for (int i = 0; i < RPW; ++i) q[i] = fold_wave(q[i], Add());
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
      const float rstd = rsqrtf(q[i] / K + a.eps);
#pragma unroll
      for (int v = 0; v < VPL; ++v) {
        floatx4 y;
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = 4 * (lane + 64 * v) + e < K ? (nx[i][v][e] - s[i]) * rstd * gv[v][e] + (hot_b ? bv[v][e] : 0.f) : 0.f;
        *(floatx4 *)&sm_x[w * RPW + i][4 * (lane + 64 * v)] = y;
      }
    }
    __syncthreads();
  }
  floatx4 acc[NT][RT][4];       // one per value of a lane's quad: short chains of additions
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[t][i][e] = floatx4{0.f, 0.f, 0.f, 0.f};
  // one batch of U steps; `more`: the next one's weights (and rows) are requested before it is multiplied (a copy of the body without that
  // for the last: where a branch decided on it, the wait for this batch's values counted on its not having been made)
  auto batch = [&](int s, auto more_) {
    constexpr bool more = decltype(more_)::value;
    if (!AHEAD) load_x(xv, s);
    floatx4 wn[NT][U], xn[RT][U];
    if (more && AHEAD) load_x(xn, s + U);
    if (more) load_w(wn, s + U);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (!more && s + u >= s1) break;          // the same for the whole wave
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) wv[t][u][e] = (s + u) * 16 + 4 * g + e < K ? wv[t][u][e] : 0.f;
#pragma unroll
      for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int t = 0; t < NT; ++t) acc[t][i][e] = mfma_f32(wv[t][u][e], xv[i][u][e], acc[t][i][e]);
    }
    if (more)
#pragma unroll
      for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int t = 0; t < NT; ++t) wv[t][u] = wn[t][u];
        if (AHEAD) xv[0][u] = xn[0][u];
      }
  };
  int st = s0;
  for (; st + U < s1; st += U) batch(st, std::true_type());
  if (st < s1) batch(st, std::false_type());
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int i = 0; i < RT; ++i) red[w][t * RT + i][lane] = (acc[t][i][0] + acc[t][i][1]) + (acc[t][i][2] + acc[t][i][3]);
  __syncthreads();
  // wave i finishes row tile i: lane (m, g) holds y[r][n .. n + 3], r = r0 + 16 i + m, n = n0 + 4 g
  static_assert(RT <= NW, "one row tile per finishing wave");
  if (w < RT) {
    const int i = w;
    floatx4 y = red[0][i][lane], y2 = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int v = 1; v < NW; ++v) y += red[v][i][lane];
    if (EPI == LIN_SWIGLU) {
      y2 = red[0][RT + i][lane];
#pragma unroll
      for (int v = 1; v < NW; ++v) y2 += red[v][RT + i][lane];
    }
    const int r = r0 + i * 16 + m, n = n0 + 4 * g;
    const bool in = r < R;
    if (EPI == LIN_HEAD) {
      float best = -INFINITY;
      int bi = 0x7fffffff;
      float *dst = a.logits && in && (info.x & ROW_VALID) ? a.logits + ((size_t)info.w * a.S + (info.y - 1)) * N : nullptr;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (n + j < N) {
          if (dst) dst[n + j] = y[j];
          if (y[j] > best) { best = y[j]; bi = n + j; }
        }
      best16(best, bi);                               // the tile's winner, lowest index on ties
      best32(best, bi);
      if (g == 0 && in) {
        a.part_val[(size_t)r * a.n_tiles + blockIdx.x] = best;
        a.part_idx[(size_t)r * a.n_tiles + blockIdx.x] = bi;
      }
      return;
    }
    if (!in) return;
    if (EPI == LIN_QKV) {
      if (!(info.x & ROW_VALID)) return;
      // (heads of whole quads: one quad is of one section and head; divisions by a variable are chains of 30 instructions)
      const bool quads = a.hd % 4 == 0;
      int sec = 0, c = 0, h = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (n + j >= N) continue;
        if (j == 0 || !quads) {
          const int s_in = (n + j) / a.d;
          sec = s_in + a.sec0; c = (n + j) - s_in * a.d; h = c / a.hd;
        }
        const int cj = quads ? c + j : c;
        if (sec == 0) { a.out[(size_t)r * a.ldo + n + j] = y[j]; continue; }
        const size_t slab = ((size_t)info.y * a.H + h) * a.kv_cap * a.hd, dim = cj - h * a.hd;
        const size_t o = slab + (sec == 1 ? (size_t)info.z * a.hd + dim : dim * a.kv_cap + info.z);
        KT *cache = (KT *)(sec == 1 ? a.kc : a.vc), *low = (KT *)(sec == 1 ? a.kc_lo : a.vc_lo);
        if (sizeof(KT) == 2 && fabsf(y[j]) > 65504.f) atomicAdd(a.kv_sat, 1);   // stored saturated
        st_f32(cache, o, y[j]);
        if (low) {            // what the rounding of the store above left out
          KT t;
          st_f32(&t, 0, y[j]);
          st_f32(low, o, y[j] - ld_f32(&t, 0));
        }
      }
      return;
    }
    float *dst = a.out + (size_t)r * a.ldo + n + (EPI == LIN_SLICE ? blockIdx.z * a.slice_stride : 0);
    if constexpr (EPI == LIN_RESID) y += row_value<RSRC>(rq, rs);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (n + j >= N) continue;
      float v = y[j];
      if (EPI == LIN_GELU) v = 0.5f * v * (1.f + erff(v * 0.70710678118654752f));
      if (EPI == LIN_SWIGLU) v = v / (1.f + expf(-v)) * y2[j];
      dst[j] = v;
    }
  }
}

template <typename WT, typename KT, int EPI, int NW, int RT, int VPL, int SRC = SRC_ROWS>
static void launch_lin(const LinArgs &a, int n_tiles, bool vec, hipStream_t s) {
  const dim3 grid(n_tiles, (a.R + 16 * RT - 1) / (16 * RT), EPI == LIN_SLICE ? SLICES : 1);
  const int4 *info = EPI == LIN_QKV ? a.rt.kvinfo : a.rt.qinfo;
  const void *x = VPL > 0 && SRC == SRC_GATHER ? a.tok_emb : a.x;
  const void *second = SRC == SRC_GATHER ? a.pos_emb : SRC == SRC_SLICES ? (const void *)a.pend : a.W2;
  auto kernel = vec ? k_lin<WT, KT, EPI, NW, RT, VPL, true, SRC> : k_lin<WT, KT, EPI, NW, RT, VPL, false, SRC>;
  hipLaunchKernelGGL(kernel, grid, dim3(64 * NW), 0, s, x, a.W, second, a.ng, a.nb, info, a.R, a.K, a);
}

// rows from where they are (see SRC_ROWS)
template <typename WT, typename KT, int EPI, int NW, int VPL>
static void launch_lin_from(const LinArgs &a, int n_tiles, bool vec, hipStream_t s) {
  constexpr bool GATHERS = EPI == LIN_RESID || EPI == LIN_QKV || EPI == LIN_STORE, ADDS = GATHERS || EPI == LIN_HEAD;
  if constexpr (GATHERS)
    if (a.tok_emb) return launch_lin<WT, KT, EPI, NW, 1, VPL, SRC_GATHER>(a, n_tiles, vec, s);
  if constexpr (ADDS)
    if (a.pend) return launch_lin<WT, KT, EPI, NW, 1, VPL, SRC_SLICES>(a, n_tiles, vec, s);
  launch_lin<WT, KT, EPI, NW, 1, VPL>(a, n_tiles, vec, s);
}

// Wide loads where the rows allow them: K a multiple of 4 and every matrix aligned.  Waves along K: 16 steps each up
// to K = 1024, 16 waves beyond; 8 with two or four row tiles per block (lin_row_tiles).
template <typename WT, typename KT, int EPI>
static int run_lin(const LinArgs &a, int n_tiles, hipStream_t s) {
  const uintptr_t mis = (uintptr_t)a.W | (uintptr_t)a.W2 | (uintptr_t)a.tok_emb | (uintptr_t)a.pos_emb;
  const uintptr_t misv = (uintptr_t)a.ng | (uintptr_t)a.nb;
  const bool vec = a.K % 4 == 0 && mis % (4 * sizeof(WT)) == 0 && misv % 16 == 0;
  if constexpr (EPI == LIN_SLICE) {
    launch_lin<WT, KT, EPI, 8, 1, 0>(a, n_tiles, vec, s);
    PD_CHECK_HIP(hipGetLastError());
    return PD_OK;
  }
  if constexpr (EPI != LIN_RESID) {
    if (a.ng) {
      if (a.K <= 256) launch_lin_from<WT, KT, EPI, 4, 1>(a, n_tiles, vec, s);
      else if (a.K <= 512) launch_lin_from<WT, KT, EPI, 8, 2>(a, n_tiles, vec, s);
      else launch_lin_from<WT, KT, EPI, 16, 4>(a, n_tiles, vec, s);
      PD_CHECK_HIP(hipGetLastError());
      return PD_OK;
    }
  }
  // (only the rows of at most 32, of up to 1024 values, are gathered or lack slices: norm_inside)
  const int rt = lin_row_tiles(n_tiles, a.K, a.R);
  if constexpr (EPI == LIN_RESID) {
    if (a.tok_emb || a.pend) {
      PD_REQUIRE(rt == 1 && a.K <= 1024, PD_EINVAL, "rows put together by launches of one row tile (%d rows of %d values)", a.R, a.K);
      if (a.K <= 256) launch_lin_from<WT, KT, EPI, 4, 0>(a, n_tiles, vec, s);
      else launch_lin_from<WT, KT, EPI, 8, 0>(a, n_tiles, vec, s);
      PD_CHECK_HIP(hipGetLastError());
      return PD_OK;
    }
  }
  if (rt == 4) launch_lin<WT, KT, EPI, 8, 4, 0>(a, n_tiles, vec, s);
  else if (rt == 2) launch_lin<WT, KT, EPI, 8, 2, 0>(a, n_tiles, vec, s);
  else if (a.K <= 256) launch_lin<WT, KT, EPI, 4, 1, 0>(a, n_tiles, vec, s);
  else if (a.K <= 1024) launch_lin<WT, KT, EPI, 8, 1, 0>(a, n_tiles, vec, s);
  else launch_lin<WT, KT, EPI, 16, 1, 0>(a, n_tiles, vec, s);
  PD_CHECK_HIP(hipGetLastError());
  return PD_OK;
}

template <int EPI>
static int linear(pd_ctx *c, LinArgs a, const void *W, const void *W2, int R, int N, int K, hipStream_t s,
                  int n_tiles = 0) {
  a.W = W; a.W2 = W2; a.R = R; a.N = N; a.K = K;
  if (!n_tiles) n_tiles = (N + 15) / 16;
  return c->cfg.dtype == 0 ? run_lin<float, float, EPI>(a, n_tiles, s) : run_lin<bf16_t, f16_t, EPI>(a, n_tiles, s);
}

// ---------------------------------------------------------------------------
// rotary + KV append: q (in place) and k rotated by the row's position; k, v
// written to the row's slot of the request's cache.
// ---------------------------------------------------------------------------
template <typename KT>
__global__ void k_qkv_post(float *qkv, KT *kc, KT *vc, KT *kc_lo, KT *vc_lo, RowTables rt,
                           const float *rope_cs, int d, int H, int hd, int kv_cap, int32_t *kv_sat) {
  int r = blockIdx.x;
  if (!(rt.flags[r] & ROW_VALID)) return;
  float *row = qkv + (size_t)r * 3 * d;
  int half = hd / 2;
  const size_t base = (size_t)rt.req[r] * H * kv_cap * hd, slot = rt.slot[r];
  const float *cs = rope_cs + (size_t)rt.pos[r] * half * 2;
  for (int i = threadIdx.x; i < H * half; i += blockDim.x) {
    int h = i / half, j = i % half;
    float q1 = row[h * hd + j], q2 = row[h * hd + j + half];
    float k1 = row[d + h * hd + j], k2 = row[d + h * hd + j + half];
    float cc = cs[2 * j], ss = cs[2 * j + 1];
    float a = q1 * cc - q2 * ss, b = q2 * cc + q1 * ss;
    q1 = a; q2 = b;
    a = k1 * cc - k2 * ss; b = k2 * cc + k1 * ss;
    k1 = a; k2 = b;
    row[h * hd + j] = q1; row[h * hd + j + half] = q2;
    const size_t o = base + ((size_t)h * kv_cap + slot) * hd, ov = base + ((size_t)h * hd + j) * kv_cap + slot;
    const size_t ov2 = ov + (size_t)half * kv_cap;
    float v1 = row[2 * d + h * hd + j], v2 = row[2 * d + h * hd + j + half];
    if (sizeof(KT) == 2) {   // half cache: count what is stored saturated
      int n_sat = (fabsf(k1) > 65504.f) + (fabsf(k2) > 65504.f) + (fabsf(v1) > 65504.f) + (fabsf(v2) > 65504.f);
      if (n_sat) atomicAdd(kv_sat, n_sat);
    }
    st_f32(kc, o + j, k1); st_f32(kc, o + j + half, k2);
    st_f32(vc, ov, v1); st_f32(vc, ov2, v2);
    if (kc_lo) {      // low halves: what the rounding of the stores above left out
      st_f32(kc_lo, o + j, k1 - ld_f32(kc, o + j)); st_f32(kc_lo, o + j + half, k2 - ld_f32(kc, o + j + half));
      st_f32(vc_lo, ov, v1 - ld_f32(vc, ov)); st_f32(vc_lo, ov2, v2 - ld_f32(vc, ov2));
    }
  }
}

// ---------------------------------------------------------------------------
// attention: block = (head, request and group of 16 of its rows), its waves take tiles of 16 keys in turn and are
// merged through LDS.  Key j of the row's request is visible when j < lim[r] (context part) or when it is a
// generated-side slot (j >= L, j < n) whose subsequence index is <= the row's (Section 3.2).
// Per key tile: S^T (16 keys x 16 queries) from the keys' rows and the queries, mask, online softmax per query,
// O^T += V^T P^T; the score tile's registers are the operand of the second product.  Keys and values are requested
// together, before either is used.  Bound by its chain, queries and keys to scores to values to the merge of the waves (6-7 us
// however few the keys), then by the one or two compute units that draw a unit's keys and values (10.6 us per 1000 keys of 64 dims in
// two blocks, of which 5 are the products: 24 of 32 clocks per key tile), so 16 waves and a tile or two each, and two blocks
// per unit where that pays (attn_f32_halves; 12 rows, 16 units of 64 dims, 330 keys: 8.7 us, 11.7 with one block, 12 more with all waves
// merging and expf; a thread per key over uncoalesced key rows took 31; requesting the next tile ahead costs the registers of half
// the waves, 13-17 us).
// ---------------------------------------------------------------------------
struct AttnF32Args {
  float *out; const float *qkv;
  const void *kc, *vc, *kc_lo, *vc_lo;
  RowTables rt; const int32_t *kv_len; const uint16_t *gen_sub;
  int kv_override, d, H, hd, kv_cap, gen_stride, L, A, nqg, req0;
  float scale;
  int keys;                 // (host) keys of the launch, of a step those of the middle of its run
};

// e^x for x <= 0 (or NaN) as 2^n 2^f, n the whole part of x log2 e and f the rest.  The rounded product h = x log2 e is taken
// apart exactly (h - n, which must not become a multiply-add), its rounding error and the low part of the constant are added
// back in one rounding: over every float of [-87, 0] the errors are those of the library's function (largest 8.4e-8; root mean
// square 1.9e-8 to 2.6e-8) without its checks.  Below -150 the result is 0, and with an unbounded x the rounding error would be
// no fraction any more: beyond 2.5e9 it passes 128 and 2^f is infinite.
__device__ __forceinline__ float exp_f32(float x) {
#pragma clang fp contract(off)
  x = x < -150.f ? -150.f : x;          // (NaN stays NaN)
  const float h = x * 1.44269504f, n = rintf(h);
  const float f = (h - n) + fmaf(x, 1.92596300e-8f, fmaf(x, 1.44269504f, -h));
  return ldexpf(__builtin_amdgcn_exp2f(f), (int)n);
}

// NHB: 16-dim blocks of a head (hd <= 16 NHB); PAIR: low halves; VS: blocks that share a unit, each with all scores and its part of
// the values' dims (nothing to merge)
template <typename KT, int NHB, int NW, bool VEC, bool PAIR, int VS>
__global__ __launch_bounds__(64 * NW) void k_attn_f32(const float *hot_qkv, const void *hot_k, const void *hot_v,
                                                      const int4 *hot_qinfo, const int32_t *hot_kv_len, uint32_t hot_hda, int kv_cap,
                                                      int H, int hot_req0, AttnF32Args a) {
  constexpr int NV = NHB / VS;          // 16-dim blocks of the values here
  static_assert(NHB % VS == 0, "whole 16-dim blocks");
  __shared__ floatx4 sm_o[NW][NV][64];
  __shared__ float sm_m[NW][16], sm_l[NW][16];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
  // (one grid dimension: the others end at 65535, and a batch may have more requests)
  const int hd = hot_hda & 0xffff, A = hot_hda >> 16, nqg = (A + 15) >> 4, unit = blockIdx.x / H, h = blockIdx.x - unit * H;
  int reqi = unit, qg = 0;
  if (nqg > 1) { reqi = unit / nqg; qg = unit - reqi * nqg; }
  const int req = hot_req0 + reqi, d = H * hd;
  const int hb0 = VS > 1 ? (int)blockIdx.y * NV : 0;
  const int qa = qg * 16 + m;
  const int r = reqi * A + min(qa, A - 1);              // clamped: loads stay in bounds
  const int4 qi = hot_qinfo[r];                         // {flags, sub, lim, req}
  int n = 0;
  if (hot_kv_len) n = hot_kv_len[req];                  // NULL: the number is an argument
  floatx4 q[NHB];
#pragma unroll
  for (int c = 0; c < NHB; ++c) q[c] = ld_row4<VEC>(hot_qkv + (size_t)r * 3 * d + h * hd, 16 * c + 4 * g, hd);
  // the first keys and values are requested before anything is known about the rows (what lies behind the last key is
  // masked; it is allocated and holds finite numbers)
  const size_t base = ((size_t)req * H + h) * kv_cap * hd;
  const KT *K = (const KT *)hot_k + base, *V = (const KT *)hot_v + base;
  floatx4 kf[NHB], vf[NV];              // key m, dims 16 c + 4 g .. + 3;  dim 16 (hb0 + i) + m, keys 4 g .. + 3
  auto load = [&](int t) {
    const size_t krow = (size_t)min(t * 16 + m, kv_cap - 1) * hd;
#pragma unroll
    for (int c = 0; c < NHB; ++c) kf[c] = ld_row4<VEC>(K + krow, 16 * c + 4 * g, hd);
#pragma unroll
    for (int i = 0; i < NV; ++i)        // (kv_cap is a multiple of 64)
      vf[i] = ld_row4<true>(V + (size_t)min(16 * (hb0 + i) + m, hd - 1) * kv_cap, t * 16 + 4 * g, kv_cap);
  };
  load(w);
  __builtin_amdgcn_sched_barrier(0);
  const KT *Kl = PAIR ? (const KT *)a.kc_lo + base : nullptr, *Vl = PAIR ? (const KT *)a.vc_lo + base : nullptr;
  const uint16_t *gs = a.gen_sub + (size_t)req * a.gen_stride;
  const int L8 = a.L & ~7;            // entry of key slot j >= L is j - L8
  // tags of the lane's 4 keys: 8 aligned bytes (clamped: context keys read entry 0 and never use it)
  uint2 tg;
  auto load_tags = [&](int t) { tg = *(const uint2 *)(gs + min(max(t * 16 + 4 * g - L8, 0), a.gen_stride - 4)); };
  load_tags(w);
  if (!hot_kv_len) n = a.kv_override;
  const bool valid = qa < A && (qi.x & ROW_VALID);
  const int lim = valid ? min(qi.z, n) : 0, sub = valid ? qi.y : -1;
  // keys some query of the group sees
  int reach = valid ? (n > a.L && sub >= 1 ? n : lim) : 0;
  reach = fold_row(reach, Max());
  const int tiles = __builtin_amdgcn_readfirstlane((reach + 15) >> 4);
#pragma unroll
  for (int c = 0; c < NHB; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) q[c][e] = 16 * c + 4 * g + e < hd ? q[c][e] : 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  floatx4 o_acc[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) o_acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
  for (int t = w; t < tiles; t += NW) {
    const int key0 = t * 16, key = key0 + 4 * g;
    if (PAIR) {
      // (scalar loads: their places are computed here, held over the loop they spill; 160 units of head size 50, 700 keys
      // 297 -> 281 us per step of 4 layers, of size 66 397 -> 372; of size 150 slower)
      int ml = m, gl = g;
      if (!VEC && NHB <= 8) asm volatile("" : "+v"(ml), "+v"(gl));
      const size_t krow = (size_t)min(key0 + ml, kv_cap - 1) * hd;
#pragma unroll
      for (int c = 0; c < NHB; ++c) kf[c] += ld_row4<VEC>(Kl + krow, 16 * c + 4 * gl, hd);
      if (!VEC && NHB == 4) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < NV; ++i) vf[i] += ld_row4<true>(Vl + (size_t)min(16 * (hb0 + i) + ml, hd - 1) * kv_cap, key, kv_cap);
    }
    const int tag[4] = {(int)(tg.x & 0xffff), (int)(tg.x >> 16), (int)(tg.y & 0xffff), (int)(tg.y >> 16)};
    floatx4 se[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) se[e] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < NHB; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) se[e] = mfma_f32(kf[c][e], q[c][e], se[e]);      // (dims past the head meet a zero query)
    floatx4 s = (se[0] + se[1]) + (se[2] + se[3]);
    // lane (query m, g), register j  <->  key key0 + 4 g + j
    float mloc = -INFINITY;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int key = key0 + 4 * g + j;
      const bool vis = (key < lim) | ((key >= a.L) & (key < n) & (tag[j] <= sub));
      s[j] = vis ? s[j] * a.scale : -INFINITY;
      mloc = fmaxf(mloc, s[j]);
    }
    mloc = fold32(fold16(mloc, Max()), Max());
    const float m_new = fmaxf(m_run, mloc);
    const float m_ref = m_new == -INFINITY ? 0.f : m_new;      // nothing visible yet: exp(-inf) = 0, never NaN
    const float alpha = exp_f32(m_run - m_ref);
    float p[4], psum = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) { p[j] = exp_f32(s[j] - m_ref); psum += p[j]; }
    l_run = l_run * alpha + psum;
    m_run = m_new;
    if (__any(alpha != 1.f))
#pragma unroll
      for (int i = 0; i < NV; ++i) o_acc[i] *= alpha;
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < NV; ++i)        // (slots past the last key hold what an earlier request left there)
        o_acc[i] = mfma_f32(key0 + 4 * g + e < n ? vf[i][e] : 0.f, p[e], o_acc[i]);
    if (t + NW < tiles) { load(t + NW); load_tags(t + NW); }   // the same for the whole wave
  }
  l_run = fold32(fold16(l_run, Add()), Add());
  if (g == 0) { sm_m[w][m] = m_run; sm_l[w][m] = l_run; }
#pragma unroll
  for (int i = 0; i < NV; ++i) sm_o[w][i][lane] = o_acc[i];
  __syncthreads();
  if (w >= NV) return;                 // a wave per 16 dims merges (all 16 doing the weights took 2.7 us)
  float M = -INFINITY, f[NW], l = 0.f;
#pragma unroll
  for (int v = 0; v < NW; ++v) M = fmaxf(M, sm_m[v][m]);
#pragma unroll
  for (int v = 0; v < NW; ++v) {
    f[v] = exp_f32(sm_m[v][m] - M);     // (a wave without a key, -inf: 0; a query without one is not stored)
    l += f[v] * sm_l[v][m];
  }
  if (!valid) return;
  // lane (query m, g) of dim block i: dims 16 (hb0 + i) + 4 g .. + 3
  for (int i = w; i < NV; i += NW) {
    floatx4 o = f[0] * sm_o[0][i][lane];
#pragma unroll
    for (int v = 1; v < NW; ++v) o += f[v] * sm_o[v][i][lane];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (16 * (hb0 + i) + 4 * g + j < hd) a.out[(size_t)r * d + h * hd + 16 * (hb0 + i) + 4 * g + j] = o[j] / l;
  }
}

template <typename KT>
static int attention_f32(const AttnF32Args &a, int nreq, hipStream_t s) {
  const int units = a.H * nreq * a.nqg;
  const int32_t *kv_len = a.kv_override >= 0 ? nullptr : a.kv_len;
  PD_REQUIRE(a.A < 65536, PD_EINVAL, "%d rows per request", a.A);        // (a step has at most 1024, a context pass too)
  const uint32_t hda = (uint32_t)a.hd | (uint32_t)a.A << 16;
  constexpr bool LOW = sizeof(KT) == 2; // (only half caches have low halves)
  const bool vec = a.hd % 4 == 0;       // rows of q, keys and values then start at multiples of 16 (half: 8) bytes
  const bool halves = attn_f32_halves(a.hd, units, a.keys);
#define PD_ATTN_F32_VS(NHB, NW, VS)                                                                           \
  do {                                                                                                        \
    auto kernel = a.kc_lo ? (vec ? k_attn_f32<KT, NHB, NW, true, LOW, VS> : k_attn_f32<KT, NHB, NW, false, LOW, VS>)  \
                          : (vec ? k_attn_f32<KT, NHB, NW, true, false, VS> : k_attn_f32<KT, NHB, NW, false, false, VS>); \
    hipLaunchKernelGGL(kernel, dim3(units, VS), dim3(64 * NW), 0, s, a.qkv, a.kc, a.vc, a.rt.qinfo, kv_len, hda, a.kv_cap, a.H,  \
                       a.req0, a);                                                                            \
  } while (0)
#define PD_ATTN_F32(NHB, NW)                                                                                  \
  do {                                                                                                        \
    if (halves) PD_ATTN_F32_VS(NHB, NW, (NHB > 2 ? 2 : 1));                                                   \
    else PD_ATTN_F32_VS(NHB, NW, 1);                                                                          \
  } while (0)
  // waves per block: what the registers of a wave leave room for
  if (a.hd <= 16) PD_ATTN_F32(1, 16);
  else if (a.hd <= 32) PD_ATTN_F32(2, 16);
  else if (a.hd <= 64) PD_ATTN_F32(4, 16);
  else if (a.hd <= 128) PD_ATTN_F32(8, 8);
  else PD_ATTN_F32(16, 4);
#undef PD_ATTN_F32
#undef PD_ATTN_F32_VS
  PD_CHECK_HIP(hipGetLastError());
  return PD_OK;
}

// ---------------------------------------------------------------------------
// one transformer layer / the head, as sequences of launches
// ---------------------------------------------------------------------------
// At most 32 rows (decode steps) of up to 1024 values: the norms are taken inside the projections that follow them and the first layer
// gathers its rows from the embedding tables.  With more rows a norm kernel of its own and tiles of 32 or 64 rows per
// block are faster (every block would take the statistics of its rows again).
// The second FFN projection of such a step is cut along K over SLICES blocks where that saves more than it costs the readers
// (ffn2_in_slices; width 512, d_ff 2048, 12 rows: 32 blocks 10.4 us, 128 blocks 4.4).  The slices are added where the rows are
// read next, by the norms inside the projections (QKV 6.4 -> 7.7, head of 8192 words 9.0 -> 12.0) and the output projection,
// which completes the residual.
static bool norm_inside(const pd_ctx *c, int R) { return R <= 32 && c->cfg.d_model <= 1024; }

bool simple_embeds(const pd_ctx *c, int R) { return !norm_inside(c, R); }

static int normed(pd_ctx *c, LinArgs &a, const float *gain, const float *bias, int R, hipStream_t s) {
  const pd_config &g = c->cfg;
  if (norm_inside(c, R)) {
    a.x = c->x; a.ng = gain; a.nb = g.norm_kind == 0 ? bias : nullptr; a.norm_kind = g.norm_kind; a.eps = g.norm_eps;
    return PD_OK;
  }
  hipLaunchKernelGGL(k_norm_f32, dim3(R), dim3(256), 0, s, (float *)c->xn, c->x, gain, bias, g.d_model, g.norm_kind,
                     g.norm_eps, c->rows.flags);
  PD_CHECK_HIP(hipGetLastError());
  a.x = (const float *)c->xn;
  return PD_OK;
}

int simple_layer(pd_ctx *c, int l, int R, int A, int nreq, int req0, int kv_override,
                 hipStream_t s) {
  const pd_config &g = c->cfg;
  const LayerPtrs &lw = c->layers[l];
  const int d = g.d_model, ff = g.d_ff, H = g.n_head, hd = g.head_dim;
  int rc;
  LinArgs base;
  memset(&base, 0, sizeof(base));
  base.rt = c->rows; base.d = d; base.H = H; base.hd = hd; base.kv_cap = c->kv_cap; base.kv_sat = c->kv_sat;
  base.slice_stride = (size_t)c->R_pad * d;
  const float *pend = c->pend_parts ? c->ypart : nullptr;        // what the layer before left out of x
  const bool gather = l == 0 && norm_inside(c, R);
  LinArgs a = base;
  if ((rc = normed(c, a, lw.n1g, lw.n1b, R, s))) return rc;
  if (gather) { a.tok_emb = c->tok_emb; a.pos_emb = c->pos_emb; }
  a.pend = pend;
  // context pass, last layer: only its keys and values are ever used, and only they are projected
  const bool last = kv_override >= 0 && l == g.n_layer - 1;
  const int n0 = last ? d : 0;
  const void *wqkv = (const char *)lw.wqkv + (size_t)n0 * d * (g.dtype == 0 ? sizeof(float) : sizeof(bf16_t));
  a.out = c->qkv32 + n0; a.ldo = 3 * d; a.sec0 = last ? 1 : 0;
  if (g.pos_kind == 1) {
    // (the rotation also turns the queries of a pass before where this one has none; nobody reads them)
    if ((rc = linear<LIN_STORE>(c, a, wqkv, nullptr, R, 3 * d - n0, d, s))) return rc;
    if (g.dtype == 0)
      hipLaunchKernelGGL(k_qkv_post<float>, dim3(R), dim3(256), 0, s, c->qkv32, (float *)lw.kc, (float *)lw.vc,
                         (float *)nullptr, (float *)nullptr, c->rows, c->rope_cs, d, H, hd, c->kv_cap, c->kv_sat);
    else
      hipLaunchKernelGGL(k_qkv_post<f16_t>, dim3(R), dim3(256), 0, s, c->qkv32, (f16_t *)lw.kc, (f16_t *)lw.vc,
                         (f16_t *)lw.kc_lo, (f16_t *)lw.vc_lo, c->rows, c->rope_cs, d, H, hd, c->kv_cap, c->kv_sat);
    PD_CHECK_HIP(hipGetLastError());
  } else {
    a.kc = lw.kc; a.vc = lw.vc; a.kc_lo = lw.kc_lo; a.vc_lo = lw.vc_lo;
    if ((rc = linear<LIN_QKV>(c, a, wqkv, nullptr, R, 3 * d - n0, d, s))) return rc;
  }
  if (last) return PD_OK;
  AttnF32Args t;
  memset(&t, 0, sizeof(t));
  t.out = (float *)c->att; t.qkv = c->qkv32; t.kc = lw.kc; t.vc = lw.vc; t.kc_lo = lw.kc_lo; t.vc_lo = lw.vc_lo;
  t.rt = c->rows; t.kv_len = c->sch.kv_len; t.gen_sub = c->sch.gen_sub; t.kv_override = kv_override; t.d = d; t.H = H;
  t.hd = hd; t.kv_cap = c->kv_cap; t.gen_stride = c->gen_stride; t.L = c->L; t.A = A; t.nqg = (A + 15) / 16;
  t.req0 = req0; t.scale = 1.0f / sqrtf((float)hd);
  t.keys = kv_override >= 0 ? kv_override : c->L + c->S * (c->M + 1) / 2;
  if ((rc = g.dtype == 0 ? attention_f32<float>(t, nreq, s) : attention_f32<f16_t>(t, nreq, s))) return rc;
  a = base;
  a.x = (const float *)c->att; a.out = c->x; a.res = c->x; a.ldo = d;
  LinArgs o = a;
  if (gather) { o.tok_emb = c->tok_emb; o.pos_emb = c->pos_emb; }
  o.pend = pend;                        // the residual is completed here
  c->pend_parts = 0;
  if ((rc = linear<LIN_RESID>(c, o, lw.wo, nullptr, R, d, d, s))) return rc;
  LinArgs f = base;
  if ((rc = normed(c, f, lw.n2g, lw.n2b, R, s))) return rc;
  f.out = (float *)c->hb; f.ldo = ff;
  rc = g.ffn_kind == 0 ? linear<LIN_GELU>(c, f, lw.w1, nullptr, R, ff, d, s)
                       : linear<LIN_SWIGLU>(c, f, lw.w1, lw.w_up, R, ff, d, s);
  if (rc) return rc;
  a.x = (const float *)c->hb;
  if (norm_inside(c, R) && ffn2_in_slices(d, ff, R, l + 1 < g.n_layer ? (3 * d + 15) / 16 : c->vocab_pad / 16)) {
    a.out = c->ypart;
    c->pend_parts = SLICES;
    return linear<LIN_SLICE>(c, a, lw.w2, nullptr, R, d, ff, s);
  }
  return linear<LIN_RESID>(c, a, lw.w2, nullptr, R, d, ff, s);
}

// leaves one winner per 16-column tile; k_turn picks the winner of each row
int simple_head(pd_ctx *c, int R, float *logits, hipStream_t s) {
  const pd_config &g = c->cfg;
  LinArgs a;
  memset(&a, 0, sizeof(a));
  int rc;
  a.rt = c->rows;
  a.slice_stride = (size_t)c->R_pad * g.d_model;
  if ((rc = normed(c, a, c->fng, c->fnb, R, s))) return rc;
  if (c->pend_parts) a.pend = c->ypart;
  c->pend_parts = 0;
  a.logits = logits; a.S = c->S; a.part_val = c->lm_part_val; a.part_idx = c->lm_part_idx; a.n_tiles = c->vocab_pad / 16;
  c->lm_win = a.n_tiles;
  return linear<LIN_HEAD>(c, a, c->lm_head, nullptr, R, g.vocab, g.d_model, s, a.n_tiles);
}
