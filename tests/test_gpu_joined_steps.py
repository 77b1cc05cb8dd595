"""Steps enqueued together, where one launch ends a step and begins the next, against the same steps one call each: the same
tokens and, bit for bit, the same logits of the last step (the launches differ in nothing but where they are cut).  Sizes on
both sides of every rule of that launch: rows per request that a wave each normalises (16, 32), widths with and without the
norm, waves that share a row's winners (1, 3 and 8 rows, more than 512 groups of columns), more than 1024 subsequences (steps
stay apart), requests that end at <eos>, at their length or at time_max, several requests, all three kernel families."""

import numpy as np
import pytest
import torch

import pd_inputs as pi
from pd_inputs.configs import WorkloadConfig, DTYPE_BF16, DTYPE_F32, FFN_SWIGLU, NORM_RMSNORM, POS_ROPE
from parity_util import make_decoder

pytestmark = pytest.mark.gpu


def W(name, steps, **kw):
    base = dict(name=name, seed=83, dtype=DTYPE_BF16, n_layer=2, d_model=128, n_head=2, head_dim=64, d_ff=256, vocab=803,
                batch=1, ctx_len=37, n_sub=5, delta_t=1, sub_tokens=6, norm_init="random", qkv_std=0.08)
    base.update(kw)
    return pytest.param(WorkloadConfig(**base), steps, id=name)


CASES = [
    W("packed-to-the-end", 14), W("one-step", 1), W("9-rows", 9, n_sub=9, sub_tokens=12),
    W("17-rows", 12, n_sub=17, sub_tokens=17), W("32-rows", 20, n_sub=32, sub_tokens=32),
    W("33-rows", 20, n_sub=33, sub_tokens=33), W("width-512", 6, d_model=512, n_head=8),
    W("width-1024-gated", 6, d_model=1024, n_head=16, ffn_kind=FFN_SWIGLU, norm_kind=NORM_RMSNORM, pos_kind=POS_ROPE),
    W("width-1056", 6, d_model=1056, n_head=11, head_dim=96), W("3-requests", 13, batch=3),
    W("2-requests-packed", 8, batch=2, n_sub=4, delta_t=2, sub_tokens=5),
    W("eos", 12, eos_id=1, vocab=3, lm_std=0.5, batch=4), W("time-max", 5), W("delay", 15, delta_t=3),
    W("1-row-many-words", 4, n_sub=1, vocab=17000), W("3-rows-many-words", 6, n_sub=3, vocab=17000),
    W("8-rows-many-words", 10, n_sub=8, sub_tokens=9, vocab=17000),
    W("1030-subsequences", 1029, n_sub=1030, sub_tokens=1, ctx_len=3, n_layer=1),
    W("fp32", 14, dtype=DTYPE_F32), W("fp32-tail", 9, dtype=DTYPE_F32, batch=2, d_model=72, n_head=3, head_dim=24),
]


@pytest.mark.parametrize("cfg,steps", CASES)
def test_joined_steps_equal_single_ones(cfg, steps):
    w, ctx = pi.make_weights(cfg, threads=4), pi.make_context(cfg)
    dec = make_decoder(cfg, w)
    time_max = cfg.time_steps if cfg.name != "time-max" else steps - 1
    dec.prefill_context(ctx, cfg.n_sub, cfg.delta_t, cfg.sub_tokens, time_max)
    single = [dec.decode_step(want_logits=(t == steps - 1)) for t in range(steps)]
    dec.reset_decode()
    dec.decode_steps(steps // 2)
    dec.decode_steps(steps - 1 - steps // 2)
    tokens, logits, done = dec.decode_step(want_logits=True)
    assert np.array_equal(tokens, single[-1][0])
    assert done == single[-1][2]
    same = (logits == single[-1][1]) | (torch.isnan(logits) & torch.isnan(single[-1][1]))
    assert bool(same.all())
    # and the whole run, which is enqueued in bursts
    toks, lens, _ = dec.generate(ctx, cfg.n_sub, cfg.delta_t, cfg.sub_tokens, time_max)
    seen = np.stack([s[0] for s in single])                        # [steps][B][S], -1: none
    for b in range(cfg.batch):
        for i in range(cfg.n_sub):
            got = [int(x) for x in seen[:, b, i] if x >= 0 and x != cfg.eos_id]
            n = min(len(got), int(lens[b, i]))
            assert got[:n] == [int(x) for x in toks[b, i, :n]]
            assert steps < cfg.time_steps or len(got) == int(lens[b, i])
    dec.close()
