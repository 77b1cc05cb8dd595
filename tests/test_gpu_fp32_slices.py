"""Second FFN projection of the fp32 kernels cut along K over blocks (d_ff from 1024 on, at most 32 rows, where that saves more
than the readers of the slices pay): inner widths on both sides of the rule and of the steps of a slice (16 values) and of a
wave, widths that are no multiple of 4 (scalar loads), one layer (only the head adds the slices) and several, 1 to 33 rows (33:
uncut), heads of so many words that the last layer alone is uncut, gated and not, bf16 weights that only these kernels take.
Logits against the CPU oracle: 1e-4 (fp32), 2e-2 (bf16)."""

import pytest

import pd_inputs as pi
from pd_inputs.configs import WorkloadConfig, DTYPE_BF16, DTYPE_F32, FFN_SWIGLU, NORM_RMSNORM, POS_ROPE
from parity_util import oracle_run, make_decoder, compare_teacher_forced

pytestmark = pytest.mark.gpu


def W(name, ff, **kw):
    base = dict(name=name, seed=19, dtype=DTYPE_F32, n_layer=3, d_model=64, n_head=2, head_dim=32, d_ff=ff, vocab=301, batch=1,
                ctx_len=21, n_sub=4, delta_t=1, sub_tokens=5, norm_init="random", qkv_std=0.1)
    base.update(kw)
    return pytest.param(WorkloadConfig(**base), id=name)


CASES = [
    W("uncut", 1020), W("1024", 1024), W("1036", 1036), W("1100", 1100), W("2050", 2050), W("4096-one-layer", 4096, n_layer=1),
    W("1-row", 1024, n_sub=1), W("16-rows", 1040, batch=4), W("32-rows", 1024, batch=8), W("33-rows", 1024, batch=11, n_sub=3),
    W("odd-width", 1025, d_model=42, n_head=3, head_dim=14),
    W("gated-rotary", 1072, ffn_kind=FFN_SWIGLU, norm_kind=NORM_RMSNORM, pos_kind=POS_ROPE),
    W("wide", 1200, d_model=1024, n_head=16, head_dim=64, n_layer=2),
    W("bf16-weights", 1040, dtype=DTYPE_BF16, d_model=48, n_head=2, head_dim=24),
    # uncut before a head of many words, cut in front of it; cut before the head too; uncut at 1024 from width 512 on
    W("many-words", 1100, d_model=512, n_head=8, head_dim=64, vocab=16640), W("fewer-words", 2048, d_model=512, n_head=8, head_dim=64, vocab=8001),
    W("wide-1024", 1024, d_model=768, n_head=12, head_dim=64, n_layer=2),
]


@pytest.mark.parametrize("cfg", CASES)
def test_slices_parity(cfg):
    w, ctx = pi.make_weights(cfg, threads=4), pi.make_context(cfg)
    dec = make_decoder(cfg, w)
    compare_teacher_forced(cfg, w, ctx, dec, oracle_run(cfg, w, ctx))
    dec.close()
