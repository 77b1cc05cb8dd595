// Schedule and glue kernels: the integer bookkeeping of Algorithm 1 kept on the
// device (so that a decode step never waits for the host), embedding gather,
// rotary table.
#include "mfma_common.h"

// ---------------------------------------------------------------------------
// reset: t = 0, no subsequences, nothing generated (Algorithm 1, lines 1-2)
// ---------------------------------------------------------------------------
__global__ void k_reset_state(SchedState st, RowTables rt, int B, int S, int L, int R_cap) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < B) {
    st.step[i] = 0; st.k_open[i] = 0; st.done[i] = 0; st.steps[i] = 0;
    st.n_gen[i] = 0; st.kv_len[i] = L; st.n_rows[i] = 0;
  }
  if (i < B * S) {
    st.n_tok[i] = 0; st.n_fed[i] = 0; st.fin[i] = 0; st.step_tok[i] = -1; st.force[i] = -1;
    st.row_of[i] = -1;
  }
  if (i < R_cap) { rt.flags[i] = 0; rt.qinfo[i] = make_int4(0, -1, 0, 0); rt.kvinfo[i] = make_int4(0, 0, 0, 0); }
  if (i == 0) *st.all_done = 0;
}

int launch_reset_state(pd_ctx *c, hipStream_t s) {
  int n = c->B * c->S;
  if (n < c->R_cap) n = c->R_cap;
  hipLaunchKernelGGL(k_reset_state, dim3((n + 255) / 256), dim3(256), 0, s, c->sch, c->rows, c->B,
                     c->S, c->L, c->R_cap);
  PD_CHECK_HIP(hipGetLastError());
  return PD_OK;
}

// ---------------------------------------------------------------------------
// prefill rows: context tokens p0 .. p0+n-1 of each of nreq requests from b on, n rows per request.
// Row for position p sees the keys 0..p (causal prefix), nothing generated; with `bidir` (rows of a
// bidirectional encoder) all L keys.  Keys and values of the rows go to cache entry `b_cache` (+ the
// request's place among the nreq).
// ---------------------------------------------------------------------------
__global__ void k_prefill_rows(RowTables rt, const int32_t *ctx_tok, int b, int L, int p0, int n, int nreq,
                               int R_cap, int bidir, int b_cache) {
  int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= R_cap) return;
  if (r < n * nreq) {
    const int q = r / n, p = p0 + r - q * n;
    rt.req[r] = b + q; rt.sub[r] = 0; rt.tok[r] = ctx_tok[(size_t)(b + q) * L + p]; rt.pos[r] = p;
    const int lim = bidir ? L : p + 1;
    rt.slot[r] = p; rt.lim[r] = lim; rt.flags[r] = ROW_VALID;
    rt.qinfo[r] = make_int4(ROW_VALID, 0, lim, b_cache + q);
    rt.kvinfo[r] = make_int4(ROW_VALID, b_cache + q, p, p);
  } else {
    rt.flags[r] = 0;
    rt.qinfo[r] = make_int4(0, -1, 0, b);
    rt.kvinfo[r] = make_int4(0, b, 0, 0);
  }
}

int launch_prefill_rows(pd_ctx *c, int b, int p0, int n, hipStream_t s, int L, int bidir, int b_cache, int nreq) {
  hipLaunchKernelGGL(k_prefill_rows, dim3((c->R_cap + 255) / 256), dim3(256), 0, s, c->rows,
                     c->ctx_tok, b, L, p0, n, nreq, c->R_cap, bidir, b_cache);
  PD_CHECK_HIP(hipGetLastError());
  return PD_OK;
}

// ---------------------------------------------------------------------------
// teacher-forced rows (Section 3.3, Fig. 3b): every token of a request's training target as one row,
// subsequence-major (row of token j of subsequence i: the lengths before i, plus j), at the grid
// coordinate Algorithm 1 would feed it, tau = (i-1) dt + 1 + j.  tgt: [B][S][ML] token ids, -1 behind a
// subsequence's last token.  A rows per request, requests b0 + blockIdx.x: row t of a request is row
// blockIdx.x A + t of the launch and writes key slot L + t with its subsequence tag and coordinate;
// next_tok[r] is the token that follows it (-1 behind the last one: a key, but no loss term).  Rows behind
// the request's last token carry nothing, and their key slots the tag 65535, which no query reaches.
// One block per request; its schedule state is used as scratch and is reset by the caller afterwards.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void k_teacher_rows(RowTables rt, SchedState st, uint16_t *gen_coord,
                                                       int32_t *next_tok, const int32_t *tgt, int b0, int S, int ML,
                                                       int A, int dt, int L, int gen_cap, int gen_stride, int R_cap,
                                                       int4 *qinfo_x, int Lx) {
  const int b = b0 + blockIdx.x, r0 = blockIdx.x * A, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int32_t *tb = tgt + (size_t)b * S * ML;
  int32_t *len = st.n_tok + (size_t)b * S, *off = st.n_fed + (size_t)b * S;
  // a wave per subsequence finds its length 64 tokens at a time
  for (int i = wave; i < S; i += blockDim.x >> 6) {
    int n = 0;
    for (;;) {
      const bool tok = n + lane < ML && tb[(size_t)i * ML + n + lane] >= 0;
      const unsigned long long m = __ballot(tok);
      if (m != ~0ull) { n += __ffsll(~m) - 1; break; }
      n += 64;
    }
    if (lane == 0) len[i] = n;
  }
  __syncthreads();
  __shared__ int s_total;
  if (threadIdx.x == 0) {
    int acc = 0;
    for (int i = 0; i < S; ++i) { off[i] = acc; acc += len[i]; }
    s_total = min(acc, A);
  }
  __syncthreads();
  const int total = s_total;
  for (int t = threadIdx.x; t < A; t += blockDim.x) {
    const int r = r0 + t;
    if (r >= R_cap) break;
    if (t >= total) {
      rt.flags[r] = 0; rt.qinfo[r] = make_int4(0, -1, 0, b); rt.kvinfo[r] = make_int4(0, b, 0, 0);
      next_tok[r] = -1;
      if (qinfo_x) qinfo_x[r] = make_int4(0, -1, 0, b);
      if (t < gen_cap) st.gen_sub[(size_t)b * gen_stride + (L & 7) + t] = 65535;
      continue;
    }
    int i = 0, hi = S - 1;              // the last subsequence that starts at or before t (empty ones only at the end)
    while (i < hi) {
      const int mid = (i + hi + 1) >> 1;
      if (off[mid] <= t && len[mid] > 0) i = mid; else hi = mid - 1;
    }
    const int j = t - off[i];
    const bool more = j + 1 < len[i];
    const int fl = ROW_VALID | (more ? ROW_PRODUCE : 0), c = (i * dt + j) + i, p = L + c;
    rt.req[r] = b; rt.sub[r] = i + 1; rt.tok[r] = tb[(size_t)i * ML + j]; rt.pos[r] = p;
    rt.slot[r] = L + t; rt.lim[r] = L; rt.flags[r] = fl;
    rt.qinfo[r] = make_int4(fl, i + 1, L, b);
    rt.kvinfo[r] = make_int4(fl, b, L + t, p);
    st.gen_sub[(size_t)b * gen_stride + (L & 7) + t] = (uint16_t)(i + 1);
    gen_coord[(size_t)b * gen_stride + (L & 7) + t] = (uint16_t)c;
    next_tok[r] = more ? tb[(size_t)i * ML + j + 1] : -1;
    if (qinfo_x) qinfo_x[r] = make_int4(fl, 0, Lx, b);     // encoder-decoder form: all Lx encoder states
  }
  if (blockIdx.x != gridDim.x - 1) return;
  for (int r = r0 + A + threadIdx.x; r < R_cap; r += blockDim.x) {
    rt.flags[r] = 0; rt.qinfo[r] = make_int4(0, -1, 0, b); rt.kvinfo[r] = make_int4(0, b, 0, 0);
    next_tok[r] = -1;
    if (qinfo_x) qinfo_x[r] = make_int4(0, -1, 0, b);
  }
}

int launch_teacher_rows(pd_ctx *c, const int32_t *tgt_dev, int b, int nreq, int A, int ML, hipStream_t s) {
  hipLaunchKernelGGL(k_teacher_rows, dim3(nreq), dim3(1024), 0, s, c->rows, c->sch, c->gen_coord, c->row_argmax, tgt_dev,
                     b, c->S, ML, A, c->dt, c->L, c->gen_cap, c->gen_stride, c->R_cap, c->qinfo_x, c->Lx);
  PD_CHECK_HIP(hipGetLastError());
  return PD_OK;
}

// Eq. 6, one row per block: nll[r] = log sum_v exp(logits[r][v]) - logits[r][next_tok[r]], 0 for rows
// without a successor.  One pass over the row: every thread keeps a running maximum and the sum around it over 8
// requests in flight at a time, the threads' pairs are merged at the end (398 rows of 50265: 24 us; two passes of 256
// threads one value at a time took 110 for 172 rows).
__global__ __launch_bounds__(1024) void k_row_nll(float *nll, const float *logits, size_t ld, int V, int A, int cap,
                                                  const int32_t *next_tok) {
  constexpr int U = 8;
  __shared__ float sh_m[16], sh_e[16];
  const int r = blockIdx.x, t = next_tok[r];
  if (t < 0) { if (threadIdx.x == 0) nll[r] = 0.f; return; }      // the same for the whole block
  const float *row = logits + ((size_t)(r / A) * cap + r % A) * ld;
  float m = -INFINITY, e = 0.f;
  for (int v0 = threadIdx.x; v0 < V; v0 += 1024 * U) {
    float x[U], mx = m;
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = row[min(v0 + 1024 * u, V - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (v0 + 1024 * u >= V) x[u] = -INFINITY;
      mx = fmaxf(mx, x[u]);
    }
    if (mx == -INFINITY) continue;
    e *= expf(m - mx);                  // (m = -inf, e = 0 at first)
#pragma unroll
    for (int u = 0; u < U; ++u) e += expf(x[u] - mx);
    m = mx;
  }
  auto merge = [&](float om, float oe) {
    const float mx = fmaxf(m, om);
    e = (m == -INFINITY ? 0.f : e * expf(m - mx)) + (om == -INFINITY ? 0.f : oe * expf(om - mx));
    m = mx;
  };
  auto merge_halves = [&](Halves<float> om, Halves<float> oe) { m = om.lo; e = oe.lo; merge(om.hi, oe.hi); };
  merge_halves(halves32(m), halves32(e));
  merge_halves(halves16(m), halves16(e));
  merge(rotate16<8>(m), rotate16<8>(e)); merge(rotate16<4>(m), rotate16<4>(e));
  merge(rotate16<2>(m), rotate16<2>(e)); merge(rotate16<1>(m), rotate16<1>(e));
  if ((threadIdx.x & 63) == 0) { sh_m[threadIdx.x >> 6] = m; sh_e[threadIdx.x >> 6] = e; }
  __syncthreads();
  if (threadIdx.x >= 64) return;
  m = threadIdx.x < 16 ? sh_m[threadIdx.x] : -INFINITY;
  e = threadIdx.x < 16 ? sh_e[threadIdx.x] : 0.f;
  merge(rotate16<8>(m), rotate16<8>(e)); merge(rotate16<4>(m), rotate16<4>(e));
  merge(rotate16<2>(m), rotate16<2>(e)); merge(rotate16<1>(m), rotate16<1>(e));
  if (threadIdx.x == 0) nll[r] = m + logf(e) - row[t];
}

// loss of a request: its rows' terms added in row order, in double precision (deterministic); one wave per request
__global__ __launch_bounds__(64) void k_loss_sum(double *loss, const float *nll, int A) {
  const int lane = threadIdx.x;
  double acc = 0.0;
  for (int t = 0; t < A; t += 64) {
    const float v = t + lane < A ? nll[(size_t)blockIdx.x * A + t + lane] : 0.f;
    for (int l = 0; l < 64; ++l) acc += (double)__uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), l));
  }
  if (lane == 0) loss[blockIdx.x] = acc;
}

// rows r of the last pass: request r / A, whose logits start at row (r / A) cap
int launch_row_nll(pd_ctx *c, const float *logits, int nreq, int A, int cap, double *loss_dev, hipStream_t s) {
  hipLaunchKernelGGL(k_row_nll, dim3(nreq * A), dim3(1024), 0, s, c->nll, logits, (size_t)c->cfg.vocab, c->cfg.vocab,
                     A, cap, c->row_argmax);
  hipLaunchKernelGGL(k_loss_sum, dim3(nreq), dim3(64), 0, s, loss_dev, c->nll, A);
  PD_CHECK_HIP(hipGetLastError());
  return PD_OK;
}

// ---------------------------------------------------------------------------
// embedding: x[r] = E_tok[tok] (+ E_pos[pos]); rows without a token are zeroed
// ---------------------------------------------------------------------------
template <typename WT>
__global__ void k_embed(float *x, const WT *tok_emb, const WT *pos_emb, RowTables rt, int d) {
  int r = blockIdx.x;
  int fl = rt.flags[r], tok = rt.tok[r], pos = rt.pos[r];     // independent loads, one round trip
  bool valid = fl & ROW_VALID;
  size_t tb = valid ? (size_t)tok * d : 0, pb = valid ? (size_t)pos * d : 0;
  for (int c = threadIdx.x; c < d; c += blockDim.x) {
    float v = 0.f;
    if (valid) {
      v = ld_f32(tok_emb, tb + c);
      if (pos_emb) v += ld_f32(pos_emb, pb + c);
    }
    x[(size_t)r * d + c] = v;
  }
}

int launch_embed(pd_ctx *c, int R, hipStream_t s) {
  int d = c->cfg.d_model;
  if (c->cfg.dtype == 0)
    hipLaunchKernelGGL(k_embed<float>, dim3(R), dim3(256), 0, s, c->x, (const float *)c->tok_emb,
                       (const float *)c->pos_emb, c->rows, d);
  else
    hipLaunchKernelGGL(k_embed<bf16_t>, dim3(R), dim3(256), 0, s, c->x, (const bf16_t *)c->tok_emb,
                       (const bf16_t *)c->pos_emb, c->rows, d);
  PD_CHECK_HIP(hipGetLastError());
  return PD_OK;
}

// ---------------------------------------------------------------------------
// The turn from one time-step to the next, one block of 16 waves per request, in any of its parts:
//   COMMIT  the end of step t: Algorithm 1 lines 9-13
//   TICK    the start of step t + 1: lines 5-7 and the row list of the step.  A subsequence has a row when it holds a token that
//           was not fed yet: its newest token (coordinate tau = t).  A subsequence that finished in the step before is fed
//           once more so that its last token enters the KV cache; that row selects no token.  Rows in subsequence order,
//           the first min(A, free slots) of them.
//   NGW > 0 the first norm of step t + 1: x = E_tok[token] (+ E_pos[position]) of every row and its norm, a wave per row (at
//           most 512 NGW values, TURN_ROWS rows per request)
// In the middle of a run all three are one launch: a chain of dependent reads through one compute unit, where each launch of
// its own cost its boundary and its way from and to memory again (width 768, 8 rows, 50265 words: commit, tick and norm
// 7.0 + 3.8 + 4.6 us, together 10.0; width 2048, commit and tick 6.3 + 4.1, together 7.4).  Bound by that chain, of which the reads
// that do not depend on each other now go out together and without conditions (state, gain and bias, table rows each waited for
// before the next: 10.9 us with it, 9.4 without, both with the norm; 7.5 and 6.2 alone).
// Encoder-decoder form (qinfo_x != NULL): L is 0 (the decoder's own cache holds generated tokens only);
// every row also gets an entry of a second table for the attention over the Lx encoder states, and
// every new key slot its grid coordinate (t - 1) + (i - 1), whose difference between a query and a
// visible key is their Manhattan distance (Section 4.3).
// ---------------------------------------------------------------------------
constexpr int TURN_ROWS = 32;

struct TurnArgs {
  SchedState st; RowTables rt;
  int dt, M, L, time_max, bos, eos, V, gen_cap, gen_stride, Lx;
  uint16_t *gen_coord; int4 *qinfo_x;
  const int32_t *force;      // tokens that replace the selected ones where >= 0 (device or mapped host memory), or NULL
  int32_t *out_tok, *out_done;   // mapped host memory for the tokens appended and the requests that have ended, or NULL
  const bf16_t *tok_emb, *pos_emb; const float *g, *b;
  int d, kind, row_end; float eps;   // row_end: rows the layout of the activations has room for
  float *x; bf16_t *xn, *xn_lo;
};

template <bool COMMIT, bool TICK, int NGW>
__global__ __launch_bounds__(1024) void k_turn(const float *part_val, const int32_t *part_idx, const int32_t *row_of,
                                               const int32_t *n_tok, const int32_t *fin_of, const int32_t *n_fed,
                                               int n_win, uint32_t sa, TurnArgs a) {
  const SchedState &st = a.st;
  const RowTables &rt = a.rt;
  const int S = sa >> 16, A = sa & 0xffff;
  __shared__ int s_arg[COMMIT ? 1024 : 1];            // s_arg[a]: argmax of row a of this request (a < A <= 1024)
  __shared__ float s_best[16];
  __shared__ int s_idx[16], s_cnt[16];
  __shared__ int s_tok[NGW ? TURN_ROWS : 1], s_pos[NGW ? TURN_ROWS : 1];
  const int b = blockIdx.x, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  // Asked for ahead of their use and without conditions (a read under one is waited for where it ends), first by the arguments
  // that arrive in registers: what the threads' subsequences hold, the first winners of the vocabulary's groups of columns,
  // whether or not their row selects a token; then the request's state.
  const int i0 = threadIdx.x;           // subsequence of this thread in the first pass
  const int ic = b * S + min(i0, S - 1);
  int r0 = COMMIT ? row_of[ic] : -1, fin0 = fin_of[ic], nt0 = n_tok[ic], fed0 = TICK ? n_fed[ic] : 0;
  // second stage of the argmax, `share` waves per row; lowest index wins ties (Eq. 4).  One wave takes 512
  // winners in one batch of requests; beyond that all 16 waves work also when there are few rows
  // (shares of a power of two: divisions by a variable are chains of 30 instructions)
  const int lg = n_win <= 512 || A > 8 ? 0 : A > 4 ? 1 : A > 2 ? 2 : A > 1 ? 3 : 4, share = 1 << lg;
  const int span = (n_win + share - 1) >> lg, t_lo = (wave & (share - 1)) * span, t_hi = min(t_lo + span, n_win);
  float wv[8]; int wx[8];
  auto ask_winners = [&](int q, int t0) {
    const size_t at = (size_t)(b * A + min(q, A - 1)) * n_win;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int tt = min(t0 + 64 * u, t_hi - 1);        // clamped: a repeated candidate changes nothing
      wv[u] = part_val[at + tt];
      wx[u] = part_idx[at + tt];
    }
  };
  if (COMMIT) ask_winners(wave >> lg, t_lo + lane);
  int zero = 0;                         // (as lanes' reads: four scalar ones are waited for one by one)
  asm volatile("" : "+v"(zero));
  const int done_v = st.done[b + zero], k_v = st.k_open[b + zero], t_v = st.step[b + zero], ng_v = TICK ? st.n_gen[b + zero] : 0;
  int f0 = -1;
  if (COMMIT && a.force) f0 = a.force[ic];
  __builtin_amdgcn_sched_barrier(0);
  int new_tok = 0;                      // token this thread's subsequence was given in this step
  bool given = false;
  float4 gv[NGW ? NGW : 1][2], bv[NGW ? NGW : 1][2];         // of the first norm: asked for when the winners' registers are free
  if (COMMIT) {
    // stage 1
    for (int q = wave >> lg; q < A; q += 16 >> lg) {
      int bi = 0x7fffffff;
      float best = -INFINITY;
      for (int t0 = t_lo + lane; t0 < t_hi; t0 += 64 * 8) {
        if (q != wave >> lg || t0 != t_lo + lane) ask_winners(q, t0);
#pragma unroll
        for (int u = 0; u < 8; ++u) keep_best(best, bi, wv[u], wx[u]);
      }
      best_wave(best, bi);
      if (lane == 0) {
        if (share == 1) s_arg[q] = bi;
        else { s_best[wave] = best; s_idx[wave] = bi; }
      }
    }
  }
  int done = __builtin_amdgcn_readfirstlane(done_v), k = __builtin_amdgcn_readfirstlane(k_v);
  const int t = __builtin_amdgcn_readfirstlane(t_v), ng = __builtin_amdgcn_readfirstlane(ng_v);
  if constexpr (NGW > 0) {
#pragma unroll
    for (int n = 0; n < NGW; ++n) {
      const int c = min((lane + 64 * n) * 8, a.d - 8);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        gv[n][h] = *(const float4 *)(a.g + c + 4 * h);
        bv[n][h] = *(const float4 *)((a.kind == 0 && a.b ? a.b : a.g) + c + 4 * h);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  if (COMMIT) {
    __syncthreads();
    if (share > 1) {                    // the same for the whole block: one row per group of waves
      const int q = threadIdx.x;
      if (q < A) {
        float best = s_best[q << lg];
        int bi = s_idx[q << lg];
        for (int i = 1; i < share; ++i) keep_best(best, bi, s_best[(q << lg) + i], s_idx[(q << lg) + i]);
        s_arg[q] = bi;
      }
      __syncthreads();
    }
    // stage 2: Algorithm 1 lines 9-13, thread i for subsequence i.  A subsequence selects a token
    // when it has a row and was unfinished when the rows were laid out.
    int open_unfinished = 0;
    for (int i = i0; i < S; i += 1024) {
      int r = r0, fin = fin0, f = f0, nt = nt0, tok = -1;
      if (i != i0) {
        r = row_of[b * S + i]; fin = fin_of[b * S + i]; nt = n_tok[b * S + i];
        f = a.force ? a.force[b * S + i] : -1;
      }
      if (i < k && !done) {
        if (r >= 0 && fin == 0) {
          tok = f >= 0 ? f : s_arg[r - b * A];
          // non-finite logits leave the argmax without a winner: keep the id inside the vocabulary so
          // that the next embedding gather stays in bounds
          if (tok < 0 || tok >= a.V) tok = 0;
          st.grid[(size_t)(b * S + i) * (a.M + 1) + nt] = tok;
          st.n_tok[b * S + i] = nt + 1;
          if (!TICK) st.step_tok[b * S + i] = tok;
          if (a.eos >= 0 && tok == a.eos) fin = 1;
          else if (nt >= a.M) fin = 2;                   // nt generated tokens now held
          st.fin[b * S + i] = fin;
          if (i == i0) { nt0 = nt + 1; fin0 = fin; new_tok = tok; given = true; }
        }
        if (fin == 0) open_unfinished = 1;
      }
      if (a.force == st.force) st.force[b * S + i] = -1;
      if (a.out_tok) a.out_tok[b * S + i] = tok;
    }
    const int any_unfinished = __syncthreads_or(open_unfinished);
    if (!done && ((k > 0 && !any_unfinished) || t >= a.time_max)) {
      done = 1;                         // the same for every thread of the block
      if (threadIdx.x == 0) {
        st.done[b] = 1; st.steps[b] = t;
        atomicAdd(st.all_done, 1);
      }
    }
    if (a.out_done && threadIdx.x == 0) a.out_done[b] = done;
  }
  if (!TICK) return;

  const int tn = t + 1;                 // the step that begins
  if (!done && tn > a.time_max) {       // only reachable with time_max == 0
    done = 1;
    if (threadIdx.x == 0) { st.done[b] = 1; atomicAdd(st.all_done, 1); }
  }
  const bool opens = !done && (tn - 1) % a.dt == 0 && k < S;      // Algorithm 1, lines 5-7: open subsequence k + 1
  if (opens) ++k;
  int a_base = 0;                       // rows of the subsequences before this pass
  for (int i1 = 0; i1 < S; i1 += 1024) {
    const int i = i1 + i0;
    int nt = nt0, fin = fin0, fed = fed0;
    if (i1 > 0 && i < S) { nt = n_tok[b * S + i]; fin = fin_of[b * S + i]; fed = n_fed[b * S + i]; }
    int tok = new_tok;
    bool have_tok = i1 == 0 && given;
    if (opens && i == k - 1) {
      nt = 1; fin = 0; fed = 0; tok = a.bos; have_tok = true;
      st.grid[(size_t)(b * S + i) * (a.M + 1)] = a.bos;
      st.n_tok[b * S + i] = 1; st.fin[b * S + i] = 0; st.n_fed[b * S + i] = 0;
    }
    const bool has = !done && i < k && nt > fed;
    const unsigned long long m = __ballot(has);
    if (i1 > 0) __syncthreads();        // the counts of the pass before have been read
    if (lane == 0) s_cnt[wave] = __popcll(m);
    __syncthreads();
    int q = a_base + __popcll(m & ((1ull << lane) - 1));
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      if (w < wave) q += s_cnt[w];
      a_base += s_cnt[w];
    }
    if (i >= S) continue;
    int r = -1;
    if (has && q < A && ng + q < a.gen_cap) {
      r = b * A + q;
      const int fl = ROW_VALID | (fin ? 0 : ROW_PRODUCE), pos = a.L + (tn - 1) + i, slot = a.L + ng + q;
      if (!have_tok) tok = st.grid[(size_t)(b * S + i) * (a.M + 1) + nt - 1];
      rt.req[r] = b; rt.sub[r] = i + 1; rt.tok[r] = tok; rt.pos[r] = pos; rt.slot[r] = slot; rt.lim[r] = a.L;
      rt.flags[r] = fl;
      rt.qinfo[r] = make_int4(fl, i + 1, a.L, b);
      rt.kvinfo[r] = make_int4(fl, b, slot, pos);
      st.gen_sub[(size_t)b * a.gen_stride + (a.L & 7) + ng + q] = (uint16_t)(i + 1);
      if (a.qinfo_x) {
        a.qinfo_x[r] = make_int4(fl, 0, a.Lx, b);
        a.gen_coord[(size_t)b * a.gen_stride + ng + q] = (uint16_t)((tn - 1) + i);
      }
      st.n_fed[b * S + i] = nt;
      if (NGW) { s_tok[q] = tok; s_pos[q] = pos; }
    }
    st.row_of[b * S + i] = r;
    st.step_tok[b * S + i] = -1;
  }
  const int rows = min(a_base, min(A, max(a.gen_cap - ng, 0)));
  for (int q = rows + i0; q < A; q += 1024) {
    rt.flags[b * A + q] = 0;
    rt.qinfo[b * A + q] = make_int4(0, -1, 0, b);
    rt.kvinfo[b * A + q] = make_int4(0, b, 0, 0);
    if (a.qinfo_x) a.qinfo_x[b * A + q] = make_int4(0, -1, 0, b);
  }
  if (threadIdx.x == 0) {
    st.n_rows[b] = rows;
    if (!done) {
      st.step[b] = tn; st.k_open[b] = k;
      st.n_gen[b] = ng + rows; st.kv_len[b] = a.L + ng + rows;
    }
  }
  if constexpr (NGW > 0) {
    // A wave per row; rows without a token are zero; what lies behind the last request's rows is never stored by any projection
    const int d = a.d;
    __syncthreads();                    // tokens and positions of the rows
    for (int q = wave; q < A; q += 16) {
      const int r = b * A + q;
      if (r >= a.row_end) break;
      const bool has = q < rows;        // the same for the whole wave
      const bf16_t *te = a.tok_emb + (has ? (size_t)s_tok[q] * d : 0);
      const bf16_t *pe = a.pos_emb ? a.pos_emb + (has ? (size_t)s_pos[q] * d : 0) : te;      // (no positions: read again, not added)
      Frag et[NGW], ep[NGW];
#pragma unroll
      for (int n = 0; n < NGW; ++n) {
        const int c = min((lane + 64 * n) * 8, d - 8);
        et[n].u = *(const uint4 *)(te + c);
        ep[n].u = *(const uint4 *)(pe + c);
      }
      __builtin_amdgcn_sched_barrier(0);
      float v[NGW][8], s1 = 0.f, s2 = 0.f;
#pragma unroll
      for (int n = 0; n < NGW; ++n) {
        const bool in = has && (lane + 64 * n) * 8 < d;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          v[n][e] = in ? bf16_to_f32(et[n].h[e]) + (a.pos_emb ? bf16_to_f32(ep[n].h[e]) : 0.f) : 0.f;
          s1 += v[n][e]; s2 += v[n][e] * v[n][e];
        }
      }
      s1 = fold_wave(s1, Add());
      s2 = fold_wave(s2, Add());
      const float mean = a.kind == 0 ? s1 / d : 0.f;
      const float rstd = rsqrtf(fmaxf(s2 / d - mean * mean, 0.f) + a.eps);
#pragma unroll
      for (int n = 0; n < NGW; ++n) {
        const int c = (lane + 64 * n) * 8;
        if (c >= d) continue;
        float y[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float ge = ((const float *)gv[n])[e], be = a.kind == 0 && a.b ? ((const float *)bv[n])[e] : 0.f;
          y[e] = has ? (v[n][e] - mean) * rstd * ge + be : 0.f;
        }
        *(float4 *)(a.x + (size_t)r * d + c) = make_float4(v[n][0], v[n][1], v[n][2], v[n][3]);
        *(float4 *)(a.x + (size_t)r * d + c + 4) = make_float4(v[n][4], v[n][5], v[n][6], v[n][7]);
        store8_split(a.xn, a.xn_lo, act_off(r, c, d), y);
      }
    }
  }
}

// Whether a step's tick also gathers and normalises its rows: one compute unit does that for all rows of a request, and a
// lane holds at most 16 values of a row (32 do not fit the registers of 16 waves: width 2048, 8 rows 17.8 us, commit and tick
// 7.4 with the norm kernel's 4.0 behind them; two waves per row are no faster than one, width 768 11.0 against 10.0; all figures before the reads went out together).
bool turn_embeds(const pd_ctx *c) { return c->impl == 1 && c->cfg.d_model <= 1024 && c->A <= TURN_ROWS; }

int launch_turn(pd_ctx *c, bool commit, bool tick, bool packed, const int32_t *force, int32_t *out_tok, int32_t *out_done,
                hipStream_t s) {
  const pd_config &g = c->cfg;
  const bool embed = tick && turn_embeds(c);
  PD_REQUIRE(c->S < 65536 && c->A <= 1024 && !(commit && tick && c->S > 1024), PD_EINVAL, "%d subsequences, %d rows", c->S, c->A);
  TurnArgs a;
  memset(&a, 0, sizeof(a));
  a.st = c->sch; a.rt = c->rows; a.dt = c->dt; a.M = c->M; a.L = c->L; a.time_max = c->time_max; a.bos = g.bos_id; a.eos = g.eos_id;
  a.V = g.vocab; a.gen_cap = c->gen_cap; a.gen_stride = c->gen_stride; a.Lx = c->Lx; a.gen_coord = c->gen_coord;
  a.qinfo_x = c->qinfo_x; a.force = force; a.out_tok = out_tok; a.out_done = out_done;
  int ngw = 0;
  if (embed) {
    const bool was = c->packed;
    c->packed = packed;                 // (the step that begins decides on the layout)
    a.xn_lo = mfma_lo(c, c->xn, g.d_model);
    c->packed = was;
    a.tok_emb = (const bf16_t *)c->tok_emb; a.pos_emb = (const bf16_t *)c->pos_emb; a.g = c->layers[0].n1g; a.b = c->layers[0].n1b;
    a.d = g.d_model; a.kind = g.norm_kind; a.eps = g.norm_eps; a.x = c->x; a.xn = (bf16_t *)c->xn;
    a.row_end = packed ? 8 : c->R_pad;  // (packed: behind them lie the low parts)
    ngw = a.d <= 512 ? 1 : 2;
  }
#define PD_TURN(C, T, N)                                                                                              \
  hipLaunchKernelGGL((k_turn<C, T, N>), dim3(c->B), dim3(1024), 0, s, c->lm_part_val, c->lm_part_idx, c->sch.row_of,   \
                     c->sch.n_tok, c->sch.fin, c->sch.n_fed, c->lm_win, (uint32_t)c->S << 16 | (uint32_t)c->A, a)
#define PD_TURN_N(C)                                                                                                  \
  if (ngw == 0) PD_TURN(C, true, 0);                                                                                  \
  else if (ngw == 1) PD_TURN(C, true, 1);                                                                             \
  else PD_TURN(C, true, 2);
  if (!tick) PD_TURN(true, false, 0);
  else if (commit) { PD_TURN_N(true) }
  else { PD_TURN_N(false) }
#undef PD_TURN_N
#undef PD_TURN
  PD_CHECK_HIP(hipGetLastError());
  return PD_OK;
}

// ---------------------------------------------------------------------------
// rotary table: cs[p][j] = (cos, sin)(p * base^(-2j/hd)), evaluated in fp64
// ---------------------------------------------------------------------------
__global__ void k_rope_table(float *cs, int rows, int half, double base) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= rows * half) return;
  int p = i / half, j = i % half;
  double ang = (double)p * pow(base, -(double)j / (double)half);
  cs[2 * (size_t)i] = (float)cos(ang);
  cs[2 * (size_t)i + 1] = (float)sin(ang);
}

int launch_rope_table(pd_ctx *c, hipStream_t s) {
  int half = c->cfg.head_dim / 2, n = c->rope_rows * half;
  hipLaunchKernelGGL(k_rope_table, dim3((n + 255) / 256), dim3(256), 0, s, c->rope_cs,
                     c->rope_rows, half, (double)c->cfg.rope_base);
  PD_CHECK_HIP(hipGetLastError());
  return PD_OK;
}
