"""Encoder-decoder decode steps whose attention over the encoder states projects its queries itself: heads of 32 and 64, 1 to 16 rows
per request (8 and 9: rows packed or not), widths of 2 to 33 k-tiles (8 waves take two rounds of two beyond 16 and 32),
inputs of 1 to 300 tokens; and the edges from which the projection is a launch of its own: 17 rows, 128 and 130 units,
heads of 96, width 1056, no low parts, a separate norm kernel.  Against the CPU oracle, 2e-2."""

import pytest

from paper_2506_23431_amd import binding
from parity_util import compare_teacher_forced
from test_gpu_encdec import E, make, oracle_run

pytestmark = pytest.mark.gpu


def C(name, options=(), **kw):
    base = dict(n_enc_layer=1, n_dec_layer=2, vocab=403, ctx_len=90, batch=1, n_sub=4, delta_t=1, sub_tokens=5)
    base.update(kw)
    return pytest.param(E(name, 71, **base), options, id=name)


NO_LOW, OWN_NORM = ((binding.PD_OPT_SPLIT_ACT, 0),), ((binding.PD_OPT_FUSE_NORM, 0),)
CASES = [
    C("1-row", n_sub=1), C("8-rows", n_sub=8, sub_tokens=9), C("9-rows", n_sub=9, sub_tokens=10),
    C("16-rows", n_sub=16, sub_tokens=16), C("17-rows", n_sub=17, sub_tokens=17), C("one-token-input", ctx_len=1),
    C("300-tokens-3-requests", ctx_len=300, batch=3), C("hd32-2-k-tiles", d_model=64, head_dim=32),
    C("hd32-17-k-tiles", d_model=544, n_head=17, head_dim=32, d_ff=128), C("hd64-24-k-tiles", d_model=768, n_head=12, d_ff=128),
    C("hd64-32-k-tiles", d_model=1024, n_head=16, d_ff=128, batch=2), C("hd32-33-k-tiles", d_model=1056, n_head=33, head_dim=32, d_ff=128),
    C("128-units", batch=64), C("130-units", batch=65), C("hd96", d_model=192, head_dim=96),
    C("no-low-parts", NO_LOW), C("norm-kernel", OWN_NORM), C("norm-kernel-9-rows", OWN_NORM, n_sub=9, sub_tokens=10),
]


@pytest.mark.parametrize("cfg,options", CASES)
def test_query_projection_parity(cfg, options):
    rounded, ctx, dec = make(cfg)
    for key, value in options:
        dec.set_option(key, value)
    compare_teacher_forced(cfg, None, ctx, dec, oracle_run(cfg, rounded, ctx), tol=2e-2, log=lambda m: print(m, flush=True))
    dec.close()
