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
// tick: Algorithm 1 lines 5-7 plus the row list of this time-step.
// One wave per request: lane i looks after subsequences i, i + 64, ...; rows are numbered in
// subsequence order with a ballot and a population count.
// A subsequence has a row when it holds a token that was not fed yet: its newest
// token (coordinate tau = t).  A subsequence that finished in the previous step is
// fed once more so that its last token enters the KV cache; that row selects no token.
// ---------------------------------------------------------------------------
// Encoder-decoder form (qinfo_x != NULL): L is 0 (the decoder's own cache holds generated tokens only);
// every row also gets an entry of a second table for the attention over the Lx encoder states, and
// every new key slot its grid coordinate (t - 1) + (i - 1), whose difference between a query and a
// visible key is their Manhattan distance (Section 4.3).
__global__ __launch_bounds__(64) void k_tick(SchedState st, RowTables rt, int S, int dt, int M, int L, int A,
                                             int time_max, int bos, int gen_cap, int gen_stride,
                                             uint16_t *gen_coord, int4 *qinfo_x, int Lx) {
  // one wave per request: lane i looks after subsequences i, i + 64, ...
  __shared__ int s_k, s_t;
  const int b = blockIdx.x, lane = threadIdx.x;
  for (int a = lane; a < A; a += 64) {
    rt.flags[b * A + a] = 0;
    rt.qinfo[b * A + a] = make_int4(0, -1, 0, b);
    rt.kvinfo[b * A + a] = make_int4(0, b, 0, 0);
    if (qinfo_x) qinfo_x[b * A + a] = make_int4(0, -1, 0, b);
  }
  for (int i = lane; i < S; i += 64) { st.row_of[b * S + i] = -1; st.step_tok[b * S + i] = -1; }
  if (lane == 0) {
    st.n_rows[b] = 0;
    int k = -1, t = 0;
    if (!st.done[b]) {
      t = st.step[b] + 1;
      if (t > time_max) {          // only reachable with time_max == 0
        st.done[b] = 1;
        atomicAdd(st.all_done, 1);
      } else {
        st.step[b] = t;
        k = st.k_open[b];
        if ((t - 1) % dt == 0 && k < S) {      // Algorithm 1, lines 5-7: open subsequence k + 1
          st.grid[(size_t)(b * S + k) * (M + 1)] = bos;
          st.n_tok[b * S + k] = 1; st.n_fed[b * S + k] = 0; st.fin[b * S + k] = 0;
          ++k;
          st.k_open[b] = k;
        }
      }
    }
    s_k = k; s_t = t;
  }
  __syncthreads();
  const int k = s_k, t = s_t;
  if (k < 0) return;
  // rows in subsequence order: the first min(A, free slots) subsequences that hold an unfed token
  const int ng = st.n_gen[b];
  int a_base = 0;
  for (int i0 = 0; i0 < k; i0 += 64) {
    int i = i0 + lane;
    int nt = 0, fin = 0;
    bool has = false;
    if (i < k) {
      nt = st.n_tok[b * S + i];
      fin = st.fin[b * S + i];
      has = nt > st.n_fed[b * S + i];
    }
    unsigned long long m = __ballot(has);
    int a = a_base + __popcll(m & ((1ull << lane) - 1));
    if (has && a < A && ng + a < gen_cap) {
      int r = b * A + a, fl = ROW_VALID | (fin ? 0 : ROW_PRODUCE);
      rt.req[r] = b; rt.sub[r] = i + 1;
      rt.tok[r] = st.grid[(size_t)(b * S + i) * (M + 1) + nt - 1];
      rt.pos[r] = L + (t - 1) + i;
      rt.slot[r] = L + ng + a;
      rt.lim[r] = L;
      rt.flags[r] = fl;
      rt.qinfo[r] = make_int4(fl, i + 1, L, b);
      rt.kvinfo[r] = make_int4(fl, b, L + ng + a, L + (t - 1) + i);
      st.gen_sub[(size_t)b * gen_stride + (L & 7) + ng + a] = (uint16_t)(i + 1);
      if (qinfo_x) {
        qinfo_x[r] = make_int4(fl, 0, Lx, b);
        gen_coord[(size_t)b * gen_stride + ng + a] = (uint16_t)((t - 1) + i);
      }
      st.n_fed[b * S + i] = nt;
      st.row_of[b * S + i] = r;
    }
    a_base += __popcll(m);
  }
  if (lane == 0) {
    int a = min(a_base, min(A, max(gen_cap - ng, 0)));
    st.n_gen[b] = ng + a; st.kv_len[b] = L + ng + a; st.n_rows[b] = a;
  }
}

int launch_tick(pd_ctx *c, hipStream_t s) {
  hipLaunchKernelGGL(k_tick, dim3(c->B), dim3(64), 0, s, c->sch, c->rows, c->S, c->dt, c->M, c->L,
                     c->A, c->time_max, c->cfg.bos_id, c->gen_cap, c->gen_stride, c->gen_coord, c->qinfo_x, c->Lx);
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
// commit: Algorithm 1 lines 9-13 for one request per block.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void k_commit(SchedState st, const float *part_val, const int32_t *part_idx,
                                                 int n_tiles, int S, int M, int A, int time_max, int eos, int V) {
  // Everything the block needs is requested at once, before the first use, so that the kernel costs
  // about one memory round trip: the schedule state of the request, and the winners of the vocabulary
  // tiles of every row, whether or not the row selects a token.
  __shared__ int s_arg[1024];           // s_arg[a]: argmax of row a of this request (a < A <= 1024)
  __shared__ float s_best[16];
  __shared__ int s_idx[16];
  const int b = blockIdx.x, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nwave = blockDim.x >> 6;
  const int done = st.done[b], t = st.step[b], k = st.k_open[b];
  const int i0 = threadIdx.x;           // subsequence of this thread in the first pass
  int r0 = -1, fin0 = 0, f0 = -1, nt0 = 0;
  if (i0 < S) {
    r0 = st.row_of[b * S + i0]; fin0 = st.fin[b * S + i0]; f0 = st.force[b * S + i0];
    nt0 = st.n_tok[b * S + i0];
  }
  // stage 1: second stage of the argmax, `share` waves per row; lowest index wins ties (Eq. 4).  One wave takes the
  // 512 tiles of a vocabulary of 8192 in one batch of requests; beyond that all 16 waves work also when there are few
  // rows (8 rows, 50265 words 8.0 -> 6.9 us; 1000 words: 3.5 us with a wave per row, 4.2 shared)
  const int share = n_tiles > 512 ? max(1, nwave / A) : 1, part = wave % share, span = (n_tiles + share - 1) / share;
  const int t_lo = part * span, t_hi = min(t_lo + span, n_tiles);
  for (int a = wave / share; a < A; a += max(1, nwave / share)) {
    if (wave >= share * (nwave / share)) break;        // (waves left over when A does not divide their number)
    int r = b * A + a;
    int bi = 0x7fffffff;
    const float *pv = part_val + (size_t)r * n_tiles;
    const int32_t *pi = part_idx + (size_t)r * n_tiles;
    float best = -INFINITY;
    for (int t0 = t_lo + lane; t0 < t_hi; t0 += 64 * 8) {
      float v[8]; int ix[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        int tt = min(t0 + 64 * u, t_hi - 1);           // clamped: a repeated candidate changes nothing
        v[u] = pv[tt];
        ix[u] = pi[tt];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (v[u] > best || (v[u] == best && ix[u] < bi)) { best = v[u]; bi = ix[u]; }
    }
    best_wave(best, bi);
    if (lane == 0) {
      if (share == 1) s_arg[a] = bi;
      else { s_best[wave] = best; s_idx[wave] = bi; }
    }
  }
  __syncthreads();
  if (share > 1) {                      // the same for the whole block: one row per group of waves
    const int a = threadIdx.x;
    if (a < A) {
      float best = s_best[a * share];
      int bi = s_idx[a * share];
      for (int i = 1; i < share; ++i) {
        const float ov = s_best[a * share + i];
        const int oi = s_idx[a * share + i];
        if (ov > best || (ov == best && oi < bi)) { best = ov; bi = oi; }
      }
      s_arg[a] = bi;
    }
    __syncthreads();
  }
  if (done) return;                     // the same for every thread of the block
  // stage 2: Algorithm 1 lines 9-13, thread i for subsequence i.  A subsequence selects a token
  // when it has a row and was unfinished when the rows were laid out.
  int open_unfinished = 0;
  for (int i = i0; i < S; i += blockDim.x) {
    int r = r0, fin = fin0, f = f0, nt = nt0;
    if (i != i0) {
      r = st.row_of[b * S + i]; fin = st.fin[b * S + i]; f = st.force[b * S + i]; nt = st.n_tok[b * S + i];
    }
    if (i < k) {
      if (r >= 0 && fin == 0) {
        int tok = f >= 0 ? f : s_arg[r - b * A];
        // non-finite logits leave the argmax without a winner: keep the id inside the vocabulary so
        // that the next embedding gather stays in bounds
        if (tok < 0 || tok >= V) tok = 0;
        st.grid[(size_t)(b * S + i) * (M + 1) + nt] = tok;
        st.n_tok[b * S + i] = nt + 1;
        st.step_tok[b * S + i] = tok;
        if (eos >= 0 && tok == eos) fin = 1;
        else if (nt >= M) fin = 2;                     // nt generated tokens now held
        st.fin[b * S + i] = fin;
      }
      if (fin == 0) open_unfinished = 1;
    }
    st.force[b * S + i] = -1;
  }
  int any_unfinished = __syncthreads_or(open_unfinished);
  if (threadIdx.x == 0 && ((k > 0 && !any_unfinished) || t >= time_max)) {
    st.done[b] = 1; st.steps[b] = t;
    atomicAdd(st.all_done, 1);
  }
}

int launch_commit(pd_ctx *c, hipStream_t s) {
  hipLaunchKernelGGL(k_commit, dim3(c->B), dim3(1024), 0, s, c->sch, c->lm_part_val, c->lm_part_idx, c->vocab_pad / 16,
                     c->S, c->M, c->A, c->time_max, c->cfg.eos_id, c->cfg.vocab);
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
