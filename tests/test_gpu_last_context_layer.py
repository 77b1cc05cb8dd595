"""The last layer of a context pass projects keys and values only, from the second third of its weights.  Models of one
layer, whose every key and value comes from that launch, in each form of it: fp32 kernels with learned and rotary
positions (whole tiles, ragged ones, widths without wide loads, bf16 weights), matrix-core kernels with both, few and many
rows, pairs of halves.  Against the CPU oracle, 1e-4 with fp32 weights and 2e-2 with bf16."""

import pytest

import pd_inputs as pi
from pd_inputs.configs import (WorkloadConfig, DTYPE_BF16, DTYPE_F32, FFN_SWIGLU, NORM_RMSNORM, POS_ROPE)
from parity_util import oracle_run, make_decoder, compare_teacher_forced

pytestmark = pytest.mark.gpu

LLAMA = dict(ffn_kind=FFN_SWIGLU, norm_kind=NORM_RMSNORM, pos_kind=POS_ROPE)


def W(name, dtype, d, heads, ctx, **kw):
    base = dict(name=name, seed=223, dtype=dtype, n_layer=1, d_model=d, n_head=heads, head_dim=d // heads, d_ff=128, vocab=259,
                batch=2, ctx_len=ctx, n_sub=3, delta_t=1, sub_tokens=3, norm_init="random", qkv_std=0.08)
    base.update(kw)
    return WorkloadConfig(**base)


CASES = [
    W("f32", DTYPE_F32, 64, 4, 13), W("f32-rope", DTYPE_F32, 64, 4, 13, **LLAMA),
    W("f32-ragged", DTYPE_F32, 60, 3, 70), W("f32-narrow-loads-rope", DTYPE_F32, 54, 3, 70, **LLAMA),
    W("f32-kernels-bf16", DTYPE_BF16, 80, 5, 37), W("f32-kernels-bf16-rope", DTYPE_BF16, 80, 5, 37, **LLAMA),
    W("bf16-few", DTYPE_BF16, 96, 3, 5), W("bf16-few-rope", DTYPE_BF16, 96, 3, 5, **LLAMA),
    W("bf16", DTYPE_BF16, 128, 2, 131), W("bf16-rope", DTYPE_BF16, 128, 2, 131, **LLAMA),
    W("bf16-many", DTYPE_BF16, 256, 4, 1030), W("bf16-many-rope", DTYPE_BF16, 256, 2, 1030, **LLAMA),
]


@pytest.mark.parametrize("pairs", [0, 1])
@pytest.mark.parametrize("cfg", CASES, ids=[c.name for c in CASES])
def test_one_layer(cfg, pairs):
    if pairs and cfg.dtype == DTYPE_F32:
        pytest.skip("fp32 caches have no low halves")
    print(f"[last-layer] {cfg}", flush=True)
    w, ctx = pi.make_weights(cfg, threads=4), pi.make_context(cfg)
    outs = oracle_run(cfg, w, ctx)
    dec = make_decoder(cfg, w, kv_pair_layers=pairs)
    compare_teacher_forced(cfg, w, ctx, dec, outs, log=lambda m: print(m, flush=True))
    dec.close()
