"""Contexts whose buffers pass 2^31 values, whose matrices pass 2^16 k-tiles or whose requests pass 2^16 rows: what a pass reads
lies where numbers of 16 or 32 bits would not find it.  Little of such a context is used (one request of its capacity), so that the
CPU oracle can say what the logits are: 2e-2 with bf16 weights."""

import numpy as np
import pytest
import torch

import pd_inputs as pi
from oracle import primitives as P
from pd_inputs.configs import WorkloadConfig, DTYPE_BF16
from pd_inputs.generate import bits_to_f32
from parity_util import oracle_run, make_decoder, compare_teacher_forced

pytestmark = pytest.mark.gpu


def W(name, **kw):
    base = dict(name=name, seed=57, dtype=DTYPE_BF16, n_layer=1, d_model=2048, n_head=16, head_dim=128, d_ff=1024, vocab=131,
                batch=1, ctx_len=15, n_sub=7, delta_t=1, sub_tokens=6, norm_init="random", qkv_std=0.05)
    base.update(kw)
    return WorkloadConfig(**base)


def parity(cfg, gigabytes, **capacity):
    if torch.cuda.mem_get_info()[0] < (gigabytes + 10) * 1e9:
        torch.cuda.empty_cache()
        if torch.cuda.mem_get_info()[0] < (gigabytes + 10) * 1e9:
            pytest.skip(f"needs {gigabytes} GB of device memory")
    w, ctx = pi.make_weights(cfg, threads=4), pi.make_context(cfg)
    outs = oracle_run(cfg, w, ctx)
    dec = make_decoder(cfg, w, **capacity)
    try:
        assert dec.workspace_bytes < gigabytes * 1e9
        compare_teacher_forced(cfg, w, ctx, dec, outs, log=lambda m: print(m, flush=True))
    finally:
        dec.close()
        del dec
        torch.cuda.empty_cache()


def test_row_buffers_beyond_32_bits():
    """1050000 rows of 2048 values: the K slices that the last norm adds lie 2^31 values apart."""
    parity(W("rows"), 180, max_batch=150000)


def test_inner_width_of_65536_k_tiles():
    """An FFN of 2^21 inner values: the second projection runs over 65536 k-tiles, in steps and in the context pass."""
    parity(W("inner", n_layer=2, d_model=32, n_head=1, head_dim=32, d_ff=1 << 21, ctx_len=20, n_sub=3, sub_tokens=3), 10)


def test_caches_more_than_64_gib_long():
    """Values lie 68.7 GB behind their keys (64 requests of 262150 context tokens, one of them in use)."""
    parity(W("keys", ctx_len=40, n_sub=3, sub_tokens=4), 150, max_batch=64, max_ctx=262150)


def test_training_target_of_more_rows_than_16_bits_hold():
    """One request's target of 66500 tokens (700 subsequences of 95) in one pass; one layer, so that single rows can be
    computed in 64 bits from the keys and values of all."""
    cfg = W("target", d_model=32, n_head=1, head_dim=32, d_ff=64, vocab=64, ctx_len=8, n_sub=700, sub_tokens=94, qkv_std=0.3)
    w, ctx = pi.make_weights(cfg, threads=4), pi.make_context(cfg)
    rng = np.random.default_rng(3)
    target = rng.integers(0, cfg.vocab, (cfg.n_sub, 95))
    dec = make_decoder(cfg, w, max_batch=710)
    dec.prefill_context(ctx, cfg.n_sub, cfg.delta_t, cfg.sub_tokens, cfg.time_steps)
    logits = dec.teacher_forced([[[int(t) for t in s] for s in target]])[0][0].cpu().numpy()
    dec.close()
    f = lambda a: bits_to_f32(a).astype(np.float64) if a.dtype == np.uint16 else a.astype(np.float64)
    norm = lambda x, name, at: P.layer_norm(x, f(at[name + "_g"]), f(at[name + "_b"]), cfg.norm_eps)
    lw, d, L, n = w["layers"][0], cfg.d_model, cfg.ctx_len, target.size
    sub, j = np.divmod(np.arange(n), 95)
    tau = sub * cfg.delta_t + 1 + j
    x = f(w["tok_emb"])[np.concatenate([ctx[0], target.ravel()])] + f(w["pos_emb"])[np.concatenate([np.arange(L), L + tau - 1 + sub])]
    y = norm(x, "norm1", lw) @ f(lw["wqkv"]).T
    q, k, v = y[:, :d], y[:, d:2 * d], y[:, 2 * d:]
    for r in [0, 94, 95, 65519, *range(65534, 65539), 65552, 65599, *rng.integers(0, n, 20), n - 1]:
        seen = np.concatenate([np.ones(L, bool), (sub <= sub[r]) & (tau <= tau[r])])
        h = x[L + r] + f(lw["wo"]) @ (P.softmax(k[seen] @ q[L + r] / np.sqrt(cfg.head_dim)) @ v[seen])
        h = h + f(lw["w2"]) @ P.gelu(f(lw["w1"]) @ norm(h, "norm2", lw))
        want = f(w["lm_head"]) @ norm(h, "final_norm", w)
        assert np.abs(logits[r] - want).max() < 2e-2, r
