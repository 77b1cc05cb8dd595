"""Attention launches of two blocks per (request, head, 16 queries), each with half of the dims of the values: every head size with
4 and with 8 waves, 127 to 130 units (beyond 128 one block per unit), 17 rows per request (two query groups), without low
parts.  Against the CPU oracle, 2e-2; with activations rounded to single bf16 values (2^-9 of each) twice that: the rounding alone is
2.14e-2 at width 1024, with one block per unit as with two."""

import pytest

import pd_inputs as pi
from pd_inputs.configs import WorkloadConfig, DTYPE_BF16
from parity_util import oracle_run, make_decoder, compare_teacher_forced

pytestmark = pytest.mark.gpu


def W(heads, hd, ctx, **kw):
    base = dict(name=f"{heads}x{hd}-{ctx}", seed=29, dtype=DTYPE_BF16, n_layer=1, d_model=heads * hd, n_head=heads, head_dim=hd,
                d_ff=128, vocab=203, batch=1, ctx_len=ctx, n_sub=3, delta_t=1, sub_tokens=3, norm_init="random", qkv_std=0.08)
    base.update(kw)
    return WorkloadConfig(**base)


CASES = [W(2, hd, ctx) for hd in (32, 64, 96, 128) for ctx in (33, 290)] + \
        [W(16, 64, 270, batch=8), W(13, 32, 270, batch=10), W(43, 32, 40, batch=3), W(2, 64, 300, n_sub=17, sub_tokens=17)]


@pytest.mark.parametrize("split_act", [1, 0])
@pytest.mark.parametrize("cfg", CASES, ids=[c.name for c in CASES])
def test_halves_parity(cfg, split_act):
    from paper_2506_23431_amd import binding
    w, ctx = pi.make_weights(cfg, threads=4), pi.make_context(cfg)
    dec = make_decoder(cfg, w)
    dec.set_option(binding.PD_OPT_SPLIT_ACT, split_act)
    compare_teacher_forced(cfg, w, ctx, dec, oracle_run(cfg, w, ctx), tol=2e-2 if split_act else 4e-2)
    dec.close()
