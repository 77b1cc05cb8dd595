"""The first norm of a layer handed over from the second FFN projection of the layer before (decode steps of at most 16
rows): inner widths around the number of k-tiles a wave asks for at once (4, 5, 6, 7, 8 and 9 per wave of 16; beyond
d_ff = 4096 the norm kernel runs), packed rows, general rows and rows without low parts, learned and rotary positions.
And the commit kernel's shares of waves per row: 1, 3, 5, 8, 9 and 16 rows per request.  Against the CPU oracle, 2e-2."""

import pytest

import pd_inputs as pi
from pd_inputs.configs import WorkloadConfig, DTYPE_BF16, FFN_SWIGLU, NORM_RMSNORM, POS_ROPE
from parity_util import oracle_run, make_decoder, compare_teacher_forced

pytestmark = pytest.mark.gpu

LLAMA = dict(ffn_kind=FFN_SWIGLU, norm_kind=NORM_RMSNORM, pos_kind=POS_ROPE)


def W(name, ff, **kw):
    base = dict(name=name, seed=171, dtype=DTYPE_BF16, n_layer=3, d_model=128, n_head=2, head_dim=64, d_ff=ff, vocab=1203,
                batch=1, ctx_len=40, n_sub=5, delta_t=1, sub_tokens=6, norm_init="random", qkv_std=0.08)
    base.update(kw)
    return WorkloadConfig(**base)


CASES = [
    W("4-per-wave", 2048), W("5-per-wave", 2560), W("6-per-wave", 3072), W("7-per-wave", 3200), W("8-per-wave", 4096),
    W("norm-kernel", 4128),
    W("6-per-wave-15-rows", 3072, batch=3), W("8-per-wave-15-rows", 4096, batch=3),
    W("6-per-wave-llama", 3072, **LLAMA), W("7-per-wave-llama-10-rows", 3424, batch=2, **LLAMA),
    W("1-row", 256, n_sub=1), W("3-rows", 256, n_sub=3), W("8-rows", 256, n_sub=8, sub_tokens=9),
    W("9-rows", 256, n_sub=9, sub_tokens=9), W("16-rows", 256, n_sub=16, sub_tokens=17),
    W("17-rows", 256, n_sub=17, sub_tokens=18),
    W("1-row-513-tiles", 256, n_sub=1, vocab=8195), W("3-rows-513-tiles", 256, n_sub=3, vocab=8195),
    W("5-rows-513-tiles", 256, vocab=8195), W("8-rows-600-tiles", 256, n_sub=8, sub_tokens=9, vocab=9590),
    W("9-rows-513-tiles", 256, n_sub=9, sub_tokens=9, vocab=8195),
]


@pytest.mark.parametrize("split_act", [1, 0])
@pytest.mark.parametrize("cfg", CASES, ids=[c.name for c in CASES])
def test_norm_handover_and_commit(cfg, split_act):
    from paper_2506_23431_amd import binding
    print(f"[handover] {cfg}", flush=True)
    w, ctx = pi.make_weights(cfg, threads=4), pi.make_context(cfg)
    outs = oracle_run(cfg, w, ctx)
    dec = make_decoder(cfg, w)
    dec.set_option(binding.PD_OPT_SPLIT_ACT, split_act)
    stats = compare_teacher_forced(cfg, w, ctx, dec, outs, log=lambda m: print(m, flush=True))
    assert stats["rows"] == cfg.batch * (cfg.n_sub * (cfg.sub_tokens + 1) - 1)
    dec.close()
