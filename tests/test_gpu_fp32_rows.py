"""Where the rows of an fp32 step's projections come from is a part of the kernel's type (the row buffer, the buffer and the slices
it lacks, the embedding tables with and without positions).  Each source with each width of loads: output rows that are no
multiple of 4 behind inner rows that are, and the other way round, 1 to 32 rows, one layer (gathered rows and slices meet in
the residual and the head) and several, heads of whole quads and of broken ones.  Against the CPU oracle, 1e-4."""

import pytest

import pd_inputs as pi
from pd_inputs.configs import WorkloadConfig, DTYPE_F32, FFN_SWIGLU, NORM_RMSNORM, POS_ROPE
from parity_util import oracle_run, make_decoder, compare_teacher_forced

pytestmark = pytest.mark.gpu

LLAMA = dict(ffn_kind=FFN_SWIGLU, norm_kind=NORM_RMSNORM, pos_kind=POS_ROPE)


def W(name, heads, hd, ff, **kw):
    base = dict(name=name, seed=229, dtype=DTYPE_F32, n_layer=2, d_model=heads * hd, n_head=heads, head_dim=hd, d_ff=ff, vocab=131,
                batch=1, ctx_len=19, n_sub=3, delta_t=1, sub_tokens=4, norm_init="random", qkv_std=0.1)
    base.update(kw)
    return pytest.param(WorkloadConfig(**base), id=name)


CASES = [
    W("narrow-out-wide-in", 3, 14, 512), W("wide-out-narrow-in", 3, 16, 130), W("narrow-out-slices", 3, 14, 1100),
    W("one-layer-slices", 4, 20, 1028, n_layer=1), W("one-layer-slices-rotary", 4, 20, 1028, n_layer=1, **LLAMA),
    W("32-rows-slices", 5, 12, 1100, batch=8, n_sub=4), W("1-row-rotary", 3, 6, 40, n_sub=1, **LLAMA),
    W("two-waves-of-rows", 9, 32, 1200, batch=4, n_sub=4), W("four-quads-a-lane", 10, 64, 1056, batch=2),
]


@pytest.mark.parametrize("cfg", CASES)
def test_row_sources(cfg):
    print(f"[fp32-rows] {cfg}", flush=True)
    w, ctx = pi.make_weights(cfg, threads=4), pi.make_context(cfg)
    dec = make_decoder(cfg, w)
    compare_teacher_forced(cfg, w, ctx, dec, oracle_run(cfg, w, ctx), log=lambda m: print(m, flush=True))
    dec.close()
