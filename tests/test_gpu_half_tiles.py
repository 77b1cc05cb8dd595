"""The second FFN projection in halves of column tiles, which hands the next layer's first norm over with row sums per 8 columns:
widths on both sides of where it starts and ends (1024, 2048), inner widths of 2 k-tiles to 12 per wave of 16, shares of a wave
in every combination of its batches, odd numbers of k-tiles (whole tiles or the norm kernel), packed and general rows, 1 to 16
rows (17: the norm kernel), learned and rotary positions.  Logits against the CPU oracle (2e-2), and no further from it than
with the norm kernels, up to rounding order."""

import pytest

import pd_inputs as pi
from pd_inputs.configs import WorkloadConfig, DTYPE_BF16, FFN_SWIGLU, NORM_RMSNORM, POS_ROPE
from parity_util import oracle_run, make_decoder, compare_teacher_forced

pytestmark = pytest.mark.gpu

LLAMA = dict(ffn_kind=FFN_SWIGLU, norm_kind=NORM_RMSNORM, pos_kind=POS_ROPE)


def W(name, d, ff, **kw):
    base = dict(name=name, seed=239, dtype=DTYPE_BF16, n_layer=3, d_model=d, n_head=d // 32, head_dim=32, d_ff=ff, vocab=259, batch=1,
                ctx_len=17, n_sub=4, delta_t=1, sub_tokens=4, norm_init="random", qkv_std=0.5 * d ** -0.5)
    base.update(kw)
    return pytest.param(WorkloadConfig(**base), id=name)


CASES = [
    W("1024-whole", 1024, 512), W("1056-64", 1056, 64), W("1056-odd", 1056, 96), W("1056-640", 1056, 640),
    W("1088-2112", 1088, 2112), W("1056-4096-llama", 1056, 4096, n_layer=2, **LLAMA), W("1056-5120", 1056, 5120, n_layer=2),
    W("1056-6144", 1056, 6144, n_layer=2), W("1056-6208-kernel", 1056, 6208, n_layer=2), W("2048-512", 2048, 512, n_layer=2),
    W("2080-512-kernel", 2080, 512, n_layer=2), W("1-row", 1056, 576, n_sub=1), W("8-rows", 1056, 576, n_sub=8, sub_tokens=9),
    W("9-rows", 1056, 1600, batch=3, n_sub=3), W("16-rows", 1056, 2112, batch=4), W("16-rows-llama", 1056, 6144, n_layer=2, batch=4, **LLAMA),
    W("17-rows-kernel", 1056, 512, n_sub=17, sub_tokens=18),
]


@pytest.mark.parametrize("cfg", CASES)
def test_half_tiles(cfg):
    from paper_2506_23431_amd import binding
    print(f"[halves] {cfg}", flush=True)
    w, ctx = pi.make_weights(cfg, threads=4), pi.make_context(cfg)
    outs = oracle_run(cfg, w, ctx)
    worst = {}
    for fuse in (1, 0):
        dec = make_decoder(cfg, w)
        dec.set_option(binding.PD_OPT_FUSE_NORM, fuse)
        worst[fuse] = compare_teacher_forced(cfg, w, ctx, dec, outs, log=lambda m: print(m, flush=True))["worst"]
        dec.close()
    assert worst[1] < 1.5 * worst[0] + 1e-4
