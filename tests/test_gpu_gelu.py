"""GELU of the first FFN projection over its whole range: first-layer weights scaled so that the values under it are a few
hundredths, of order one, around the end of the fitted range (8) and far beyond it, where it is 0 or the value itself.  A
decode step and a context pass (few and many rows) against the CPU oracle's erf; the second projection is scaled back, so
that the logits keep their size and the tolerance of the bf16 path (2e-2) its meaning."""

import pytest

import numpy as np

import pd_inputs as pi
from pd_inputs.configs import WorkloadConfig, DTYPE_BF16
from parity_util import oracle_run, make_decoder, compare_teacher_forced

pytestmark = pytest.mark.gpu


def scaled(bits, f):
    """bf16 bit patterns times a power of two."""
    v = (bits.astype(np.uint32) << 16).view(np.float32) * np.float32(f)
    return (v.view(np.uint32) >> 16).astype(np.uint16)


@pytest.mark.parametrize("scale", [1 / 64, 1.0, 8.0, 512.0])
@pytest.mark.parametrize("ctx_len", [20, 140])
def test_gelu_over_its_range(ctx_len, scale):
    cfg = WorkloadConfig(name="gelu", seed=227, dtype=DTYPE_BF16, n_layer=2, d_model=128, n_head=2, head_dim=64, d_ff=512,
                         vocab=517, batch=1, ctx_len=ctx_len, n_sub=3, delta_t=1, sub_tokens=3, norm_init="random", qkv_std=0.08)
    print(f"[gelu] {cfg} scale {scale}", flush=True)
    w, ctx = pi.make_weights(cfg, threads=4), pi.make_context(cfg)
    for lw in w["layers"]:
        lw["w1"], lw["w2"] = scaled(lw["w1"], scale), scaled(lw["w2"], 1 / scale)
    outs = oracle_run(cfg, w, ctx)
    dec = make_decoder(cfg, w)
    compare_teacher_forced(cfg, w, ctx, dec, outs, log=lambda m: print(m, flush=True))
    dec.close()
