// Masked multi-query attention of the pipelined decode step on the matrix cores.
//
// Dependency rule (paper Section 3.2): the row of subsequence i sees every context
// key and the generated-side keys of subsequences i' <= i fed so far, this step's
// included.  In the cache every generated-side slot is tagged with its subsequence,
// so the rule is one integer compare per key.  Prefill rows use the same kernel
// with a causal limit instead (key index < lim).
//
// grid (split, head, request * query-group); block = 4 or 8 waves.  The 32-key blocks of one
// (request, head) are dealt round-robin to the waves of all splits that serve it, so the
// first block of every wave is known at launch and its K/V fragments are requested
// before anything else is read.  Per block of 32 keys: 2*(hd/32) K fragments and hd/16 V fragments
// (1 KiB each, contiguous), two 16-key score tiles S^T = K Q^T, mask, online
// softmax (running max / sum per query), O^T += V^T P^T.  Up to 16 query rows of a
// request share every key/value byte read.  Waves are merged through LDS; blocks
// write (max, sum, O) partials that a second, tiny kernel merges by log-sum-exp.
#include "mfma_common.h"

#include <hip/hip_ext.h>

#include <algorithm>
#include <type_traits>

struct AttnArgs {
  const f16_t *q, *q_lo;    // [rows][d] fp16 high / low parts (q_lo NULL: high part only)
  const f16_t *kc, *vc;     // packed fp16 caches of this layer
  const f16_t *kc_lo, *vc_lo;   // low halves of the same layout (PAIR kernels only)
  bf16_t *out, *out_lo;     // [rows][d] high / low parts (out_lo NULL: high part only)
  RowTables rt;
  const int32_t *kv_len;
  const uint16_t *gen_sub;  // subsequence tag of key slot j >= L at [req][j - (L & ~7)]
  int kv_override;          // >= 0: number of keys to consider (prefill), else kv_len[req]
  float *part;
  int d, H, kv_cap, gen_stride, L, A, nqg, req0, nsplit, nblk_static;
  float scale_log2;         // log2(e) / sqrt(hd)
  // BIAS kernels: every key slot j carries a grid coordinate, coord[req * coord_req_stride + j - coord_off]
  // = (tau - 1) + (i - 1) for a generated-side token (the encoder: its position), and a query has
  // c_q = pos[r] - pos0.
  //  * relative-position bias of the encoder-decoder form (Section 4.3): the score gets
  //    bias[h][clamp(c_q - coord[j] + bias_off, 0, bias_len - 1)] (already times log2(e));
  //  * a generated-side key is visible only if it is not later than the query, tau_k <= tau_q, beside
  //    the subsequence rule.  In a decode step that holds for every key in the cache; in the one-pass
  //    teacher-forced forward (Fig. 3b) all of the target's keys are there at once and this is the
  //    time half of the matrix.  tau - 2 = coordinate - subsequence tag on both sides.
  const float *bias; const uint16_t *coord;
  int bias_len, bias_off, coord_stride, coord_req_stride, coord_off, pos0;
  // QP kernels: the projection in front; stats != NULL: it finishes a norm without mean and bias
  const bf16_t *W, *xn; uint32_t xn_lo;
  const float2 *stats; float norm_eps;
};
constexpr int BIAS_MAX = 264;   // entries of one head's bias table that the kernel keeps in LDS

// PAIR: the layer keeps keys and values as high + low halves.  Scores add q_hi K_lo (q_lo K_lo is
// below the rounding of everything else), outputs add P V_lo; the kernel holds twice the fragments
// and is built for one block per compute unit.
// STREAM: keys and values are loaded with the non-temporal hint.  In a decode step every key/value byte is read
// once per launch and nothing reads it again before the caches have turned over, so keeping it out of the
// caches' way pays (cfg4: 15.9 -> 15.0 us per launch, cfg5: 60.5 -> 52.8); in the context pass the 16-query
// groups of a chunk re-read the same keys from L2, and there the hint costs a third of the pass.
template <bool STREAM>
__device__ __forceinline__ f16x8 ld_kv(const uint4 *p) {
  return STREAM ? __builtin_nontemporal_load((const f16x8 *)p) : *(const f16x8 *)p;
}

// Tags and coordinates stay in one piece until they are used: taken apart or copied at their load, at the end of the block
// before, they made every block wait there for the loads it should overlap (256 units of head size 32, 107 blocks:
// 51 us per layer and step, 57 with it).
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void pin(u32x4 &u) { asm volatile("" : "+v"(u)); }

// VS = 2: two blocks per (request, head, query group), each with half of the dims of the values: both take all scores, so
// that nothing is merged and a compute unit draws three quarters of the bytes.  The second block's number is higher by the units
// of the launch: where these are a multiple of 8, both run on one XCD and the second finds the keys in the L2 cache they
// share; with 12 heads they do not, and the keys (QP: and the weights) come from behind L2 for both.
// QP: the block projects its queries itself from the rows in xn (the attention over the encoder states, whose queries are a
// projection of their own): a launch and its way through memory less for a share of 16 HD weights rows per block.  The waves
// cut K as in the projection kernels; PK: rows of at most 8, high and low parts as one fragment.  Width 768, 8 rows, 512
// keys: 4.4 us (projection) + 4.5 -> 6.9.  With keys and values of the step projected here too a block's share of the weights is three
// times as large and one compute unit draws it slower than 144 blocks do: width 768 12.2 us against 10.2, with few keys 9.4
// against 8.6, width 1024 21.8 against 21.0; taken out.
template <int HD, bool SPLIT, bool PAIR, bool BIAS = false, bool STREAM = false, int NW = 4, int VS = 1, bool QP = false, bool PK = false>
__global__ __launch_bounds__(64 * NW, PAIR ? 1 : NW == 4 ? 3 : NW / 4)
void k_attn_mfma(const f16_t *hot_q, const int4 *hot_qinfo, const f16_t *hot_kc, const int32_t *hot_kv_len, uint32_t hot_q_lo,
                 uint32_t hot_v, int hot_kv_cap, uint32_t hot_ha, uint32_t hot_nb, int hot_req0, AttnArgs a) {
  // (QP: hot_q is xn, hot_q_lo the way to its low parts, hot_qinfo the weights, hot_kv_len the row sums of the norm or NULL)
  constexpr int NC = HD / 32, NHB = HD / 16 / VS, PSTR = HD + 2;   // partial: m, l, O[HD] per query
  static_assert(HD / 16 % VS == 0 && (VS == 1 || !PAIR), "whole 16-dim blocks; pair layers keep theirs together");
  __shared__ float sm_m[NW][16], sm_l[NW][16];
  __shared__ float sm_bias[BIAS ? BIAS_MAX : 1];
  constexpr int T = QP ? HD / 16 : 0;                         // column tiles projected
  static_assert(!QP || (SPLIT && !PAIR && !BIAS && VS == 2 && NW == 8), "projecting launches: halves, 8 waves, low parts");
  __shared__ floatx4 sm_raw[NW * (T > NHB ? T : NHB)][64];   // partial tiles of the projection, later the waves' outputs
  floatx4 (*sm_o)[NHB][64] = (floatx4 (*)[NHB][64])sm_raw;
  __shared__ float sm_stat[QP ? NW : 1][16];
  __shared__ uint4 sm_q[(SPLIT ? 2 : 1) * NC][64];
  const int H = word_heads(hot_ha), A = word_rows(hot_ha), nqg = (A + 15) >> 4, d = H * HD;
  const int nsplit = hot_nb >> 20, nblk_static = hot_nb & 0xfffff;
  // (halves: heads, groups, halves of the dims; no splits)
  const int split = VS == 1 ? blockIdx.x : 0, h = VS == 1 ? blockIdx.y : blockIdx.x, z = VS == 1 ? blockIdx.z : blockIdx.y;
  const int hb0 = VS == 1 ? 0 : (int)blockIdx.z * NHB;        // first 16-dim block of this block
  int reqi = z, qg = 0;
  if (nqg > 1) { reqi = z / nqg; qg = z - reqi * nqg; }
  const int req = hot_req0 + reqi;
  int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  int n = lane & 15, g = lane >> 4;

  // The rows and their queries are requested first (a few lines that sit in the L2 cache), then the first key/value
  // block, all by arguments that arrive in registers (the first 14 words; read from memory they cost 0.25-0.35 us before
  // the first request); the wait for the row data does not wait for the key/value block behind it.
  int qa = qg * 16 + n;                       // query index inside the request
  bool in_req = qa < A;
  int r = reqi * A + (in_req ? qa : 0);     // row (clamped: loads stay in bounds)
  int4 qi;                                   // {flags, sub, lim, req}
  int n_keys = 0;
  if (!QP) qi = hot_qinfo[r];
  if (!QP && hot_kv_len) n_keys = hot_kv_len[req];   // NULL: the number is an argument
  // Query fragments (high and low parts) go to LDS, in operand order: the waves share them,
  // and keeping them out of the registers leaves room for three waves per SIMD.  Rows without a
  // token keep whatever finite numbers their q slots hold: all their keys are masked below, and
  // their output is never written.
  const size_t q_off = act_off(r, h * HD + g * 8, d);
  static_assert(NC <= 4, "one query fragment (and its low part) per wave");
  uint4 qh, qlo;
  if (!QP) {
    const int c = min(wave, NC - 1);
    size_t off = q_off + (size_t)c * 512;     // the next 32 dims are the next fragment
    qh = *(const uint4 *)(hot_q + off);
    if (SPLIT) qlo = *((const uint4 *)(hot_q + off) + words_granules(hot_q_lo));
  }

  const uint4 *Kp = (const uint4 *)(hot_kc + ((size_t)req * H + h) * hot_kv_cap * HD) + lane;
  const uint4 *Vp = Kp + (size_t)hot_v * 16 + hb0 * 64;      // (in units of 256 bytes, to which caches are aligned)
  const uint4 *Kl = PAIR ? (const uint4 *)(a.kc_lo + ((size_t)req * H + h) * hot_kv_cap * HD) + lane : nullptr;
  const uint4 *Vl = PAIR ? (const uint4 *)(a.vc_lo + ((size_t)req * H + h) * hot_kv_cap * HD) + lane : nullptr;
  // 32-key blocks are dealt round-robin to the NW*nsplit waves that serve this (request, head):
  // whatever the current key count, no wave gets more than one block above the average
  const int stride = NW * nsplit;
  int kb = split * NW + wave;
  Frag kf[2][NC], vf[NHB];
  Frag kl[PAIR ? 2 : 1][PAIR ? NC : 1], vl[PAIR ? NHB : 1];
  union { u32x4 u; uint16_t s[8]; } tg, kco;
  auto load_k = [&](int kbx) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        kf[t][c].hv = ld_kv<STREAM>(&Kp[((size_t)(kbx * 2 + t) * NC + c) * 64]);
        if (PAIR) kl[t][c].hv = ld_kv<STREAM>(&Kl[((size_t)(kbx * 2 + t) * NC + c) * 64]);
      }
  };
  auto load_v = [&](int kbx) {
#pragma unroll
    for (int i = 0; i < NHB; ++i) {
      vf[i].hv = ld_kv<STREAM>(&Vp[((size_t)kbx * (NHB * VS) + i) * 64]);
      if (PAIR) vl[i].hv = ld_kv<STREAM>(&Vl[((size_t)kbx * NHB + i) * 64]);
    }
  };
  // ---- projection: k-tiles wave, wave + NW, ... of the block's T column tiles, two at a time ----
  const int KT = d >> 5;
  floatx4 pacc[T > 0 ? T : 1];
  const uint4 *wq = (const uint4 *)hot_qinfo + lane, *px = nullptr;
  constexpr int TA = T > 0 ? T : 1;
  Frag pw[TA][2], pxh[2], pxl[2];
  auto project_request = [&](int kt, int u) {
    pxh[u].u = px[(size_t)kt * 64];
    if (!PK) pxl[u].u = px[(size_t)kt * 64 + words_granules(hot_q_lo)];
#pragma unroll
    for (int j = 0; j < T; ++j) pw[j][u].hv = ld_kv<STREAM>(&wq[((size_t)(h * T + j) * KT + kt) * 64]);
  };
  auto project_multiply = [&](int u) {
#pragma unroll
    for (int j = 0; j < T; ++j) {
      pacc[j] = mfma16(pw[j][u], pxh[u], pacc[j]);
      if (!PK) pacc[j] = mfma16(pw[j][u], pxl[u], pacc[j]);
    }
  };
  if constexpr (QP) {
    const int pr = reqi * A + min(PK ? n & 7 : n, A - 1);               // (PK: lanes 8-15 of a row of 16 hold the low parts of 0-7)
    px = (const uint4 *)hot_q + ((size_t)(pr >> 4) * KT * 64 + g * 16 + (pr & 15)) + (PK && n >= 8 ? words_granules(hot_q_lo) : 0);
#pragma unroll
    for (int j = 0; j < T; ++j) pacc[j] = floatx4{0.f, 0.f, 0.f, 0.f};
    if (wave < KT) project_request(wave, 0);                            // the same for the whole wave
    if (wave + NW < KT) project_request(wave + NW, 1);
    __builtin_amdgcn_sched_barrier(0);
  }

  // requested unconditionally (a wave beyond the last block fetches that block and ignores it), so
  // that the wait for the query rows above never has to wait for these
  load_k(min(kb, nblk_static - 1));
  load_v(min(kb, nblk_static - 1));
  __builtin_amdgcn_sched_barrier(0);          // (arguments that are not in registers yet are waited for behind these requests)
  // subsequence tags of the generated-side slots, 8 keys (16 bytes) per lane group
  const uint16_t *gs = a.gen_sub + (size_t)req * a.gen_stride;
  const int L8 = a.L & ~7;
  const uint16_t *kcp = BIAS ? a.coord + (size_t)req * a.coord_req_stride : nullptr;
  // tags of the lane's 8 keys (clamped: context blocks read entry 0 and never use it)
  auto load_tags = [&](int kbx) {
    tg.u = *(const u32x4 *)(gs + min(max(kbx * 32 + 8 * g - L8, 0), a.gen_stride - 8));
    if (BIAS) kco.u = *(const u32x4 *)(kcp + min(max(kbx * 32 + 8 * g - a.coord_off, 0), a.coord_stride - 8));
  };
  load_tags(min(kb, nblk_static - 1));
  if (!QP && !hot_kv_len) n_keys = a.kv_override;
  int q_pos = 0;
  float bias_pre[2] = {0.f, 0.f};
  if (BIAS) {
    q_pos = a.rt.pos[r] - a.pos0;
    bias_pre[0] = a.bias[(size_t)h * a.bias_len + min((int)threadIdx.x, a.bias_len - 1)];
    bias_pre[1] = a.bias[(size_t)h * a.bias_len + min((int)threadIdx.x + 64 * NW, a.bias_len - 1)];
  }
  if constexpr (QP) {
    qi = a.rt.qinfo[r];
    n_keys = a.kv_override >= 0 ? a.kv_override : a.kv_len[req];
    // the sums of squares: wave w, lane (n, g) takes the tile pairs g + 4 w, + 4 NW, ... of its row (fixed order)
    const bool normed = hot_kv_len != nullptr;                          // the same for the whole launch
    if (normed) {
      const float4 *sp = (const float4 *)hot_kv_len + (size_t)r * KT;   // (sum, sum of squares) of two tiles
      float sq = 0.f;
      for (int p = g + 4 * wave; p < KT; p += 4 * NW) { const float4 v = sp[p]; sq += v.y + v.w; }
      sq = fold32(fold16(sq, Add()), Add());
      if (lane < 16) sm_stat[wave][lane] = sq;
    }
    for (int kt = wave; kt < KT; kt += 2 * NW) {
      if (kt >= 2 * NW) {
        project_request(kt, 0);
        if (kt + NW < KT) project_request(kt + NW, 1);
        __builtin_amdgcn_sched_barrier(0);
      }
      project_multiply(0);
      if (kt + NW < KT) project_multiply(1);
    }
#pragma unroll
    for (int j = 0; j < T; ++j) sm_raw[wave * T + j][lane] = pacc[j];
    __syncthreads();
    if (wave < T) {                                                     // wave j finishes tile j
      floatx4 y = sm_raw[wave][lane];
#pragma unroll
      for (int w = 1; w < NW; ++w) y += sm_raw[w * T + wave][lane];
      if (PK)
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] += rotate16<8>(y[e]);
      if (normed) {
        float tot = sm_stat[0][n];
#pragma unroll
        for (int w = 1; w < NW; ++w) tot += sm_stat[w][n];
        y *= rsqrtf(tot * (1.f / (float)d) + a.norm_eps);
      }
      // queries in operand order: y[e] is dim 16 wave + 4 g + e (lanes beyond the rows hold copies, finite as those are)
      const int dim0 = wave * 16 + 4 * g;
      float yv[4] = {y[0], y[1], y[2], y[3]};
      f16_t *dst = (f16_t *)&sm_q[dim0 >> 5][((dim0 & 31) >> 3) * 16 + n] + (dim0 & 7);
      store4_split_h(dst, dst + (size_t)NC * 64 * 8, 0, yv);
    }
    __syncthreads();
  }
  // (waves beyond the fragment count store a copy of the last fragment: same bytes, same place)
  if (!QP) {
    const int c = min(wave, NC - 1);
    sm_q[c][lane] = qh;
    if (SPLIT) sm_q[NC + c][lane] = qlo;
  }
  if (BIAS && !QP) {
    if (threadIdx.x < BIAS_MAX) sm_bias[threadIdx.x] = bias_pre[0];
    if (threadIdx.x + 64 * NW < BIAS_MAX) sm_bias[threadIdx.x + 64 * NW] = bias_pre[1];
  }
  if (!QP) __syncthreads();

  bool qvalid = in_req && (qi.x & ROW_VALID);
  int q_sub = qvalid ? qi.y : -1, q_lim = qvalid ? qi.z : 0;
  // keys any query of this group can see
  int reach = qvalid ? (n_keys > a.L && q_sub >= 1 ? n_keys : min(q_lim, n_keys)) : 0;
  reach = fold_row(reach, Max());
  const int end = __builtin_amdgcn_readfirstlane(min(nblk_static, (reach + 31) >> 5));
  // keys below lim_all are visible to every query of the group that has a token (the others are
  // never written, whatever they compute): blocks below it skip the per-key test
  int lim_q = qvalid ? min(q_lim, a.L) : 0x7fffffff;
  lim_q = fold_row(lim_q, Min());
  const int lim_all = __builtin_amdgcn_readfirstlane(lim_q);

  float m_run = -INFINITY, l_run = 0.f;
  floatx4 o_acc[NHB];
#pragma unroll
  for (int i = 0; i < NHB; ++i) o_acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};

  // One block per wave is resident in registers.  The key fragments of the wave's next block are
  // requested as soon as the score products have consumed the current ones, the value fragments
  // (and tags) as soon as the output products have: the loads of block i+1 overlap the softmax
  // and the output products of block i without a second set of registers.  The wave's last block is a copy of the
  // loop's body without requests: where a branch decides on a request, the wait for the values counts on its not
  // having been made, and every block waited for the next one's keys.
  auto block = [&](auto more_) {
    constexpr bool more = decltype(more_)::value;
    floatx4 s[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};
    // the query fragments are re-read from LDS for every block (the empty asm keeps the compiler
    // from hoisting the reads out of the loop, which would put them back into 32 registers)
    int ql_lane = lane;
    asm volatile("" : "+v"(ql_lane));
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      Frag qf;
      qf.u = sm_q[c][ql_lane];
      s[0] = mfma16h(kf[0][c], qf, s[0]);
      s[1] = mfma16h(kf[1][c], qf, s[1]);
      if (PAIR) {
        s[0] = mfma16h(kl[0][PAIR ? c : 0], qf, s[0]);
        s[1] = mfma16h(kl[PAIR ? 1 : 0][PAIR ? c : 0], qf, s[1]);
      }
      if (SPLIT) {
        qf.u = sm_q[NC + c][ql_lane];
        s[0] = mfma16h(kf[0][c], qf, s[0]);
        s[1] = mfma16h(kf[1][c], qf, s[1]);
      }
    }
    const int kn = kb + stride;
    if (more) load_k(kn);
    // lane (n, g), tile t, register j  <->  key kb*32 + 8g + 4t + j
    const int key0 = kb * 32 + 8 * g;
    float sv[8];
    float bv[8];
    if (BIAS) {
      pin(kco.u);
      const int q_off = q_pos + a.bias_off, last = a.bias_len - 1;
#pragma unroll
      for (int e = 0; e < 8; ++e) bv[e] = sm_bias[min(max(q_off - (int)kco.s[e], 0), last)];
    }
    if (kb * 32 + 32 <= lim_all) {
      // every query of the group sees the whole block (the same for all lanes of the wave)
#pragma unroll
      for (int e = 0; e < 8; ++e) sv[e] = BIAS ? s[e >> 2][e & 3] * a.scale_log2 + bv[e] : s[e >> 2][e & 3] * a.scale_log2;
    } else {
      pin(tg.u);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        int key = key0 + e;
        bool vis = (key < q_lim) | ((key >= a.L) & (key < n_keys) & ((int)tg.s[e] <= q_sub) &
                                    (!BIAS || (int)kco.s[e] - (int)tg.s[e] <= q_pos - q_sub));
        sv[e] = vis ? (BIAS ? s[e >> 2][e & 3] * a.scale_log2 + bv[e] : s[e >> 2][e & 3] * a.scale_log2) : -INFINITY;
      }
    }
    float mloc = fmaxf(fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3])), fmaxf(fmaxf(sv[4], sv[5]), fmaxf(sv[6], sv[7])));
    mloc = fold32(fold16(mloc, Max()), Max());
    const float m_new = fmaxf(m_run, mloc);
    // while nothing is visible yet the reference is 0 instead of -inf: every exponential below is
    // then exp2(-inf) = 0 and never exp2(NaN)
    const float m_ref = m_new == -INFINITY ? 0.f : m_new;
    const float alpha = __builtin_amdgcn_exp2f(m_run - m_ref);
    float p[8], psum = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      p[e] = __builtin_amdgcn_exp2f(sv[e] - m_ref);
      psum += p[e];
    }
    l_run = l_run * alpha + psum;
    m_run = m_new;
    // probabilities enter the matrix core as fp16 (the same 11 significant bits as the values they multiply)
    Frag pf, pl;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      pf.hh[e] = (f16_t)p[e];
      if (PAIR) pl.hh[e] = (f16_t)(p[e] - (float)pf.hh[e]);
    }
    if (__any(alpha != 1.f)) {                // the running maximum of some query moved: rescale
#pragma unroll
      for (int i = 0; i < NHB; ++i) o_acc[i] *= alpha;
    }
#pragma unroll
    for (int i = 0; i < NHB; ++i) {
      o_acc[i] = mfma16h(vf[i], pf, o_acc[i]);
      if (PAIR) {
        o_acc[i] = mfma16h(vl[PAIR ? i : 0], pf, o_acc[i]);
        o_acc[i] = mfma16h(vf[i], pl, o_acc[i]);
      }
    }
    if (more) { load_tags(kn); load_v(kn); }
    kb = kn;
  };
  while (kb + stride < end) block(std::true_type());
  if (kb < end) block(std::false_type());
  l_run = fold32(fold16(l_run, Add()), Add());

  // ---- merge the waves of the block (log-sum-exp) ----
  // every wave stores its accumulators as 16-byte quads (lane order: conflict-free); after the
  // barrier wave w owns the 16-dim blocks w, w + NW, ... and sums the NW copies of each
  if (g == 0) { sm_m[wave][n] = m_run; sm_l[wave][n] = l_run; }
#pragma unroll
  for (int i = 0; i < NHB; ++i) sm_o[wave][i][lane] = o_acc[i];
  __syncthreads();
  if (wave >= NHB) return;                    // no block of dims left to finish
  float mw[NW], M = -INFINITY;
#pragma unroll
  for (int w = 0; w < NW; ++w) { mw[w] = sm_m[w][n]; M = fmaxf(M, mw[w]); }
  float fw[NW], lsum = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    fw[w] = mw[w] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mw[w] - M);
    lsum += fw[w] * sm_l[w][n];
  }
  if (!qvalid) return;                        // lane (n, g) writes for query n only
  // partial of this block: m[16], l[16], then O as [dim / 4][query][4 dims]: a wave's store of one
  // 16-dim block is 1 KiB of consecutive bytes
  size_t unit = (size_t)z * H + h;
  float *pp = a.part + (unit * nsplit + split) * (size_t)(PSTR * 16);
  if (nsplit > 1 && wave == 0 && g == 0) { pp[n] = M; pp[16 + n] = lsum; }
  const float inv = 1.f / lsum;
  for (int i = wave; i < NHB; i += NW) {
    floatx4 o = fw[0] * sm_o[0][i][lane];
#pragma unroll
    for (int w = 1; w < NW; ++w) o += fw[w] * sm_o[w][i][lane];
    if (nsplit == 1) {
      float y[4] = {o[0] * inv, o[1] * inv, o[2] * inv, o[3] * inv};
      store4_split(a.out, a.out_lo, act_off(r, h * HD + (hb0 + i) * 16 + 4 * g, d), y);
    } else {
      *(floatx4 *)(pp + 32 + ((i * 4 + g) * 16 + n) * 4) = o;
    }
  }
}

// Merge of the split partials by log-sum-exp.  Block = (unit, 16-dim block), 4 waves; wave w merges
// the splits w, w + 4, ... online (running max, sum and 4 output dims per lane), 8 splits' loads in
// flight at a time; the four running states are then combined through LDS.
template <int HD>
__global__ __launch_bounds__(256) void k_attn_merge(const float *part, const int32_t *flags, bf16_t *out, bf16_t *out_lo,
                                                    uint32_t ha, int nsplit) {
  constexpr int PSTR = HD + 2, U = 8;
  __shared__ float sm_M[4][64], sm_L[4][64];
  __shared__ floatx4 sm_O[4][64];
  const int H = word_heads(ha), A = word_rows(ha), nqg = (A + 15) >> 4;
  int unit = blockIdx.x, i = blockIdx.y, z = unit / H, h = unit - z * H;
  int reqi = z, qg = 0;
  if (nqg > 1) { reqi = z / nqg; qg = z - reqi * nqg; }
  int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
  int qa = qg * 16 + n, r = reqi * A + min(qa, A - 1);
  int fl = flags[r];
  const size_t sstr = (size_t)PSTR * 16;
  const float *pb = part + (size_t)unit * nsplit * sstr;
  const int o_off = 32 + ((i * 4 + g) * 16 + n) * 4;
  float M = -INFINITY, l = 0.f;
  floatx4 o = floatx4{0.f, 0.f, 0.f, 0.f};
  for (int s0 = wave; s0 < nsplit; s0 += 4 * U) {
    float mv[U], lv[U];
    floatx4 ov[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float *ps = pb + (size_t)min(s0 + 4 * u, nsplit - 1) * sstr;   // clamped: masked below
      mv[u] = ps[n];
      lv[u] = ps[16 + n];
      ov[u] = *(const floatx4 *)(ps + o_off);
    }
    float Mn = M;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s0 + 4 * u >= nsplit) mv[u] = -INFINITY;
      Mn = fmaxf(Mn, mv[u]);
    }
    if (Mn != -INFINITY) {
      float sc = exp2f(M - Mn);               // M == -inf: 0, and l, o are 0 anyway
      l *= sc; o *= sc;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float w = mv[u] == -INFINITY ? 0.f : exp2f(mv[u] - Mn);
        l += w * lv[u];
        o += w * ov[u];
      }
      M = Mn;
    }
  }
  sm_M[wave][lane] = M; sm_L[wave][lane] = l; sm_O[wave][lane] = o;
  __syncthreads();
  if (wave != 0) return;
  float Mt = fmaxf(fmaxf(sm_M[0][lane], sm_M[1][lane]), fmaxf(sm_M[2][lane], sm_M[3][lane]));
  float lt = 0.f;
  floatx4 ot = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    float f = sm_M[w][lane] == -INFINITY ? 0.f : exp2f(sm_M[w][lane] - Mt);
    lt += f * sm_L[w][lane];
    ot += f * sm_O[w][lane];
  }
  if (qa >= A || !(fl & ROW_VALID)) return;
  float inv = 1.f / lt;
  float y[4] = {ot[0] * inv, ot[1] * inv, ot[2] * inv, ot[3] * inv};
  store4_split(out, out_lo, act_off(r, h * HD + i * 16 + 4 * g, H * HD), y);
}

template <int HD, bool SPLIT, bool PAIR, bool BIAS, bool STREAM, int NW, int VS = 1>
static void launch_attn_nw(dim3 grid, hipStream_t s, hipEvent_t e0, hipEvent_t e1, const AttnArgs &a) {
  const uint32_t q_lo = a.q_lo ? (uint32_t)((a.q_lo - a.q) / 64) : 0u, v = (uint32_t)((a.vc - a.kc) / 128);
  const uint32_t ha = heads_rows(a.H, a.A), nb = (uint32_t)a.nblk_static | (uint32_t)a.nsplit << 20;
  const int32_t *kv_len = a.kv_override >= 0 ? nullptr : a.kv_len;
  auto kernel = k_attn_mfma<HD, SPLIT, PAIR, BIAS, STREAM, NW, VS>;
  if (e0 || e1)
    hipExtLaunchKernelGGL(kernel, grid, dim3(64 * NW), 0, s, e0, e1, 0, a.q, a.rt.qinfo, a.kc, kv_len, q_lo, v, a.kv_cap, ha, nb, a.req0, a);
  else
    hipLaunchKernelGGL(kernel, grid, dim3(64 * NW), 0, s, a.q, a.rt.qinfo, a.kc, kv_len, q_lo, v, a.kv_cap, ha, nb, a.req0, a);
}

template <int HD, bool SPLIT, bool PAIR, bool BIAS, bool STREAM>
static void launch_attn(dim3 grid, int nw, bool halves, hipStream_t s, hipEvent_t e0, hipEvent_t e1, const AttnArgs &a) {
  if constexpr (!PAIR && HD / 16 % 2 == 0) {
    const dim3 grid2(grid.y, grid.z, 2);
    if (halves && nw == 8) return launch_attn_nw<HD, SPLIT, PAIR, BIAS, STREAM, 8, 2>(grid2, s, e0, e1, a);
    if (halves) return launch_attn_nw<HD, SPLIT, PAIR, BIAS, STREAM, 4, 2>(grid2, s, e0, e1, a);
  }
  if constexpr (!PAIR) {
    if (nw == 8) return launch_attn_nw<HD, SPLIT, PAIR, BIAS, STREAM, 8>(grid, s, e0, e1, a);
  }
  launch_attn_nw<HD, SPLIT, PAIR, BIAS, STREAM, 4>(grid, s, e0, e1, a);
}

// Ordinary loads also where a step takes the non-temporal hint (PD_OPT_STREAM_LOADS), which the projection launch in front had
// for its weights: with the hint on weights, keys and values 76 models (12 layers of width 256-1024, 1-8 requests, 20 and 512
// input tokens) take 0.93-1.07 times as long per step, 1.016 on average.
template <int HD>
static void launch_attn_proj(int nreq, hipStream_t s, const AttnArgs &a) {
  const uint32_t v = (uint32_t)((a.vc - a.kc) / 128), ha = heads_rows(a.H, a.A), nb = (uint32_t)a.nblk_static | 1u << 20;
  auto kernel = a.A <= 8 ? k_attn_mfma<HD, true, false, false, false, 8, 2, true, true>
                         : k_attn_mfma<HD, true, false, false, false, 8, 2, true, false>;
  hipLaunchKernelGGL(kernel, dim3(a.H, nreq, 2), dim3(512), 0, s, (const f16_t *)a.xn, (const int4 *)a.W, a.kc,
                     (const int32_t *)a.stats, a.xn_lo, v, a.kv_cap, ha, nb, a.req0, a);
}

int mfma_attention(pd_ctx *c, const LayerPtrs &lw, int A, int nreq, int req0, int kv_override,
                   hipStream_t s, const AttnMode *mode, const AttnProj *proj) {
  const pd_config &g = c->cfg;
  if (kv_override >= 0 && !mode && c->opt_profile == 0) {     // context pass: many rows per request
    int rc = mfma_attention_ctx(c, lw, A, nreq, req0, kv_override, s);
    if (rc != 1) return rc;
  }
  AttnArgs a;
  memset(&a, 0, sizeof(a));
  a.q = (const f16_t *)c->q; a.q_lo = (const f16_t *)mfma_lo(c, c->q, g.d_model);
  a.out_lo = mfma_lo(c, c->att, g.d_model); a.kc = (const f16_t *)lw.kc; a.vc = (const f16_t *)lw.vc;
  a.kc_lo = (const f16_t *)lw.kc_lo; a.vc_lo = (const f16_t *)lw.vc_lo;
  a.out = (bf16_t *)c->att; a.rt = c->rows; a.kv_len = c->sch.kv_len; a.gen_sub = c->sch.gen_sub;
  a.kv_override = kv_override; a.part = c->att_part;
  a.d = g.d_model; a.H = g.n_head; a.kv_cap = c->kv_cap; a.gen_stride = c->gen_stride; a.L = c->L;
  a.A = A; a.nqg = (A + 15) / 16; a.req0 = req0;
  a.scale_log2 = 1.4426950408889634f / sqrtf((float)g.head_dim);
  if (mode) {
    PD_REQUIRE(!a.kc_lo, PD_EINVAL, "the encoder-decoder form keeps no pair layers");
    if (mode->kc) { a.kc = (const f16_t *)mode->kc; a.vc = (const f16_t *)mode->vc; }
    if (mode->qinfo) a.rt.qinfo = const_cast<int4 *>(mode->qinfo);
    a.L = mode->L;
    a.scale_log2 = 1.4426950408889634f * mode->scale;
    if (mode->bias) {
      PD_REQUIRE(mode->bias_len >= 1 && mode->bias_len <= BIAS_MAX && mode->coord && mode->coord_stride >= 8,
                 PD_EINVAL, "relative-position bias table of %d entries (at most %d)", mode->bias_len, BIAS_MAX);
      a.bias = mode->bias; a.coord = mode->coord; a.bias_len = mode->bias_len; a.bias_off = mode->bias_off;
      a.coord_stride = mode->coord_stride; a.coord_req_stride = mode->coord_req_stride;
      a.coord_off = mode->coord_off; a.pos0 = mode->pos0;
    }
  }
  int units = nreq * a.nqg * g.n_head;
  PD_REQUIRE(units <= c->part_units, PD_EINVAL, "too many (request, head, query group) units: %d", units);
  // the most keys this launch can meet: prefill knows it, decode takes the end of the run
  int n_keys = kv_override >= 0 ? kv_override : c->L + c->S * (c->M + 1);
  a.nblk_static = std::min((n_keys + 31) / 32, c->kv_cap / 32);
  // the shape fits the keys of the middle of the run (half of what it can generate)
  const int nblk = kv_override >= 0 ? a.nblk_static : std::min((c->L + c->S * (c->M + 1) / 2 + 31) / 32, a.nblk_static);
  const int cap = std::max(1, c->part_units / units);
  const AttnShape shape = c->opt_splits > 0 ? AttnShape{std::min(c->opt_splits, cap), 4}
                                            : attn_shape(g.head_dim, units, nblk, cap, kv_override < 0 || mode,
                                                         a.kc_lo != nullptr, c->stream_loads);
  const int nw = shape.waves;
  a.nsplit = shape.splits;
  PD_REQUIRE(a.H <= 256 && A < (1 << 24) && a.nblk_static < (1 << 20) && a.nsplit < (1 << 12) && a.vc > a.kc &&
                 (a.vc - a.kc) % 128 == 0,
             PD_EINVAL, "an attention launch over %d rows and %d key blocks is too large", A, a.nblk_static);
  const bool halves = attn_halves(shape, units, kv_override < 0 || mode, a.kc_lo != nullptr);
  if (proj) {
    if (!halves || A > 16 || (g.head_dim != 64 && g.head_dim != 32) || !a.q_lo || c->opt_profile || c->opt_splits > 0 ||
        g.d_model > 1024 || g.norm_kind != 1)
      return 1;
    a.W = proj->W; a.xn = (const bf16_t *)c->xn; a.xn_lo = (uint32_t)((mfma_lo(c, c->xn, g.d_model) - a.xn) / 64);
    if (proj->finish) { a.stats = c->nstats; a.norm_eps = g.norm_eps; }
    if (g.head_dim == 64) launch_attn_proj<64>(nreq, s, a);
    else launch_attn_proj<32>(nreq, s, a);
    PD_CHECK_HIP(hipGetLastError());
    if (proj->finish) c->norm_fused = false;
    return PD_OK;
  }
  dim3 grid(a.nsplit, g.n_head, nreq * a.nqg);
  // measurement: mode 1 attaches a start and a stop event to the dispatch of the main kernel itself
  // (their difference is the kernel's execution time), mode 2 records events before the main kernel
  // and after the merge kernel
  // mode 3 records nothing: it launches the main kernel one extra time first, on the cache of the layer half
  // the stack away (other bytes of the same size: no cache serves them) and with the same outputs, which the
  // real launch then overwrites.  Timing a run of steps with and without it gives the kernel's cost where it
  // runs, between its neighbours, without any event next to it.
  const bool twice = c->opt_profile == 3 && kv_override < 0 && !a.bias && !a.kc_lo;
  AttnArgs a_extra = a;
  if (twice) {
    const size_t n = c->layers.size(), l = (size_t)(&lw - c->layers.data());
    const LayerPtrs &other = c->layers[(l + n / 2) % n];
    a_extra.kc = (const f16_t *)other.kc; a_extra.vc = (const f16_t *)other.vc;
  }
  bool prof = (c->opt_profile == 1 || c->opt_profile == 2) && kv_override < 0 && !a.bias;   // (the instantiations with coordinates take no events)
  hipEvent_t ev0 = nullptr, ev1 = nullptr;
  if (prof) {
    while (c->ev_pool.size() < c->ev_used + 2) {
      hipEvent_t ev;
      PD_CHECK_HIP(hipEventCreate(&ev));
      c->ev_pool.push_back(ev);
    }
    ev0 = c->ev_pool[c->ev_used];
    ev1 = c->ev_pool[c->ev_used + 1];
    if (c->opt_profile == 2) PD_CHECK_HIP(hipEventRecord(ev0, s));
  }
  const bool attach = prof && c->opt_profile == 1;
  hipEvent_t pe0 = attach ? ev0 : nullptr, pe1 = attach ? ev1 : nullptr;
  // decode steps of the decoder-only form stream their keys and values (see STREAM); the context pass, the
  // teacher-forced forward and the encoder-decoder launches (small or re-read key sets) do not
  const bool stream = kv_override < 0 && !mode && c->stream_loads;
#define PD_ATTN_ONE(HDV, ARGS)                                                                         \
  do {                                                                                                 \
    const bool sp = a.q_lo != nullptr, pr = a.kc_lo != nullptr, bi = a.bias != nullptr;                \
    if (bi && sp) launch_attn<HDV, true, false, true, false>(grid, nw, halves, s, pe0, pe1, ARGS);                 \
    else if (bi) launch_attn<HDV, false, false, true, false>(grid, nw, halves, s, pe0, pe1, ARGS);                 \
    else if (pr && sp && stream) launch_attn<HDV, true, true, false, true>(grid, nw, halves, s, pe0, pe1, ARGS);   \
    else if (pr && sp) launch_attn<HDV, true, true, false, false>(grid, nw, halves, s, pe0, pe1, ARGS);            \
    else if (pr && stream) launch_attn<HDV, false, true, false, true>(grid, nw, halves, s, pe0, pe1, ARGS);        \
    else if (pr) launch_attn<HDV, false, true, false, false>(grid, nw, halves, s, pe0, pe1, ARGS);                 \
    else if (sp && stream) launch_attn<HDV, true, false, false, true>(grid, nw, halves, s, pe0, pe1, ARGS);        \
    else if (sp) launch_attn<HDV, true, false, false, false>(grid, nw, halves, s, pe0, pe1, ARGS);                 \
    else if (stream) launch_attn<HDV, false, false, false, true>(grid, nw, halves, s, pe0, pe1, ARGS);             \
    else launch_attn<HDV, false, false, false, false>(grid, nw, halves, s, pe0, pe1, ARGS);                        \
  } while (0)
#define PD_ATTN(HDV)                                                                                   \
  do {                                                                                                 \
    if (twice) PD_ATTN_ONE(HDV, a_extra);                                                              \
    PD_ATTN_ONE(HDV, a);                                                                               \
    if (a.nsplit > 1)                                                                                  \
      hipLaunchKernelGGL(k_attn_merge<HDV>, dim3(units, HDV / 16), dim3(256), 0, s, a.part, a.rt.flags, a.out, a.out_lo, \
                         heads_rows(a.H, A), a.nsplit);                                                        \
  } while (0)
  switch (g.head_dim) {
    case 32: PD_ATTN(32); break;
    case 64: PD_ATTN(64); break;
    case 96: PD_ATTN(96); break;
    case 128: PD_ATTN(128); break;
    default: pd_set_error("head_dim %d not supported by the MFMA attention", g.head_dim); return PD_EINVAL;
  }
#undef PD_ATTN
#undef PD_ATTN_ONE
  PD_CHECK_HIP(hipGetLastError());
  if (prof) {
    if (c->opt_profile != 1) PD_CHECK_HIP(hipEventRecord(c->ev_pool[c->ev_used + 1], s));
    c->ev_used += 2;
  }
  return PD_OK;
}
