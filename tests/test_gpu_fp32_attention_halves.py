"""fp32 attention with two blocks per request and head, each with half of the dims of the values: head sizes on both sides of
where it starts (32) and of its 16-dim blocks (whole, broken, an odd number of them), keys and units on both sides of the rule
(160 keys, 128 units), scalar loads, caches of pairs of halves.  Against the CPU oracle, 1e-4 (fp32) and 2e-2 (bf16 weights)."""

import pytest

import pd_inputs as pi
from pd_inputs.configs import WorkloadConfig, DTYPE_BF16, DTYPE_F32
from parity_util import oracle_run, make_decoder, compare_teacher_forced

pytestmark = pytest.mark.gpu


def W(name, heads, hd, ctx, **kw):
    base = dict(name=name, seed=241, dtype=DTYPE_F32, n_layer=2, d_model=heads * hd, n_head=heads, head_dim=hd, d_ff=64, vocab=131,
                batch=1, ctx_len=ctx, n_sub=3, delta_t=1, sub_tokens=3, norm_init="random", qkv_std=0.5 * (heads * hd) ** -0.5)
    base.update(kw)
    return pytest.param(WorkloadConfig(**base), id=name)


CASES = [
    W("32-whole", 2, 32, 300), W("34", 3, 34, 200), W("36", 2, 36, 200), W("48", 2, 48, 333), W("50-scalar", 2, 50, 200),
    W("64-few-keys", 2, 64, 150), W("64", 2, 64, 155), W("64-long", 1, 64, 700), W("66-scalar", 1, 66, 200), W("80", 3, 80, 200),
    W("96-batch", 4, 96, 170, batch=3), W("128", 2, 128, 400), W("130", 1, 130, 200), W("256", 1, 256, 170),
    W("128-units", 16, 40, 160, batch=8), W("129-units-whole", 43, 36, 160, batch=3),
    W("bf16-80", 2, 80, 200, dtype=DTYPE_BF16), W("bf16-48-16-rows", 2, 48, 200, dtype=DTYPE_BF16, batch=2, n_sub=8, sub_tokens=8),
    W("bf16-50-scalar", 2, 50, 200, dtype=DTYPE_BF16), W("bf16-66-scalar", 2, 66, 333, dtype=DTYPE_BF16),
    W("bf16-130-scalar", 1, 130, 170, dtype=DTYPE_BF16), W("bf16-50-scalar-129-units-whole", 43, 50, 160, batch=3, dtype=DTYPE_BF16),
]


@pytest.mark.parametrize("cfg", CASES)
def test_halves(cfg):
    print(f"[f32-halves] {cfg}", flush=True)
    w, ctx = pi.make_weights(cfg, threads=4), pi.make_context(cfg)
    outs = oracle_run(cfg, w, ctx)
    for pairs in ([0, 1] if cfg.dtype == DTYPE_BF16 else [-1]):
        dec = make_decoder(cfg, w, kv_pair_layers=pairs)
        compare_teacher_forced(cfg, w, ctx, dec, outs, log=lambda m: print(m, flush=True))
        dec.close()
