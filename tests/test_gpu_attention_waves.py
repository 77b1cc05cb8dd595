"""The attention kernel's launch shapes: one work-group of 4 or of 8 waves per request, head and 16 queries, and splits with
the merge kernel, at key counts around the edges of the rule (8 and 96 blocks of 32 keys in the middle of the run, 256
units) and with fewer key blocks than waves; every head size, with and without low parts; the encoder with its position
bias.  Against the CPU oracle, tolerance 2e-2 (bf16), and with low parts less than a third of the difference without
them (measured: a seventh or less): a product that left them out would add half of it or more."""

import numpy as np
import pytest

import pd_inputs as pi
from pd_inputs.configs import WorkloadConfig, DTYPE_BF16
from parity_util import oracle_run, make_decoder, compare_teacher_forced

pytestmark = pytest.mark.gpu


def W(name, heads, hd, ctx, **kw):
    base = dict(name=name, seed=161, dtype=DTYPE_BF16, n_layer=1, d_model=heads * hd, n_head=heads, head_dim=hd, d_ff=128,
                vocab=203, batch=1, ctx_len=ctx, n_sub=3, delta_t=1, sub_tokens=4, norm_init="random", qkv_std=0.08)
    base.update(kw)
    return WorkloadConfig(**base)


CASES = [
    W("one-block-hd64", 2, 64, 5),                      # one key block, 4 waves
    W("hd64-4-blocks", 2, 64, 105),                     # 4 waves
    W("hd64-7-blocks", 2, 64, 200),                     # 4 waves, fewer blocks than 8
    W("hd64-8-blocks", 2, 64, 230),                     # 8 waves from here on
    W("hd32-9-blocks", 2, 32, 262),
    W("hd64-5-to-12-blocks", 2, 64, 140, sub_tokens=80), # 8 waves, at first three of them without a key
    W("hd32-31-blocks", 3, 32, 977),                    # 8 waves
    W("hd64-33-blocks", 2, 64, 1020),                   # 8 waves
    W("hd96-64-blocks", 2, 96, 2033),                   # splits and merge
    W("hd128-96-blocks", 1, 128, 3050),                 # splits and merge
    W("hd64-97-blocks", 1, 64, 3085),                   # splits and merge
    W("hd128-pairs", 2, 128, 300, qkv_std=0.03),        # (pair layers keep 4 waves)
    W("hd32-many-units", 13, 32, 40, batch=20),         # 260 units, 2 blocks: 4 waves
    W("hd32-260-units", 13, 32, 250, batch=20),         # 260 units, 9 blocks: 4 waves
    W("hd32-252-units", 14, 32, 250, batch=18),         # 252 units, 9 blocks: 8 waves
]
WORST = {}              # largest logit difference by case and form


@pytest.mark.parametrize("split_act", [1, 0])
@pytest.mark.parametrize("cfg", CASES, ids=[c.name for c in CASES])
def test_launch_shapes(cfg, split_act):
    from paper_2506_23431_amd import binding
    print(f"[attn-waves] {cfg}", flush=True)
    w, ctx = pi.make_weights(cfg, threads=4), pi.make_context(cfg)
    outs = oracle_run(cfg, w, ctx)
    dec = make_decoder(cfg, w, kv_pair_layers=1 if cfg.name == "hd128-pairs" else -1)
    dec.set_option(binding.PD_OPT_SPLIT_ACT, split_act)
    stats = compare_teacher_forced(cfg, w, ctx, dec, outs, log=lambda m: print(m, flush=True))
    assert stats["rows"] == cfg.batch * (cfg.n_sub * (cfg.sub_tokens + 1) - 1)
    dec.close()
    WORST[cfg.name, split_act] = stats["worst"]
    if (cfg.name, 1 - split_act) in WORST:
        assert 3 * WORST[cfg.name, 1] < WORST[cfg.name, 0]


@pytest.mark.parametrize("hd", [96, 128])
def test_eight_waves_of_wide_heads(hd):
    """Heads of 96 and 128 take 8 waves where 128 units meet 40 key blocks that no cache holds: 64 requests over two
    different contexts."""
    from paper_2506_23431_amd import binding
    cfg = W(f"hd{hd}-128-units", 2, hd, 1260, batch=64, qkv_std=0.05)
    print(f"[attn-waves] {cfg}", flush=True)
    w = pi.make_weights(cfg, threads=4)
    ctx = np.tile(pi.make_context(cfg)[:2], (32, 1))
    outs = oracle_run(cfg.scaled(batch=2), w, ctx[:2]) * 32
    dec = make_decoder(cfg, w)
    dec.set_option(binding.PD_OPT_STREAM_LOADS, 1)
    stats = compare_teacher_forced(cfg, w, ctx, dec, outs, tol=1e-3, log=lambda m: print(m, flush=True))
    assert stats["rows"] == cfg.batch * (cfg.n_sub * (cfg.sub_tokens + 1) - 1)
    dec.close()


def test_eight_waves_with_a_position_bias():
    """Encoder of 300 tokens and 4 heads: 76 units of 10 key blocks, 8 waves with the relative-position table; decoder over
    as many encoder states."""
    from test_gpu_encdec import E, make, oracle_run as encdec_oracle
    cfg = E("encdec-8-waves", 67, d_model=256, n_head=4, d_ff=352, ctx_len=300, n_sub=3, sub_tokens=6)
    print(f"[attn-waves] {cfg}", flush=True)
    rounded, ctx, dec = make(cfg)
    outs = encdec_oracle(cfg, rounded, ctx)
    stats = compare_teacher_forced(cfg, None, ctx, dec, outs, tol=2.5e-3, log=lambda m: print(m, flush=True))
    assert stats["rows"] == cfg.batch * (cfg.n_sub * (cfg.sub_tokens + 1) - 1)
    dec.close()
