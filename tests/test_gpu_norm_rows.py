"""Norm kernels at the edges of their granules: a wave per row (launches of more than 128 rows, here a context) takes 512
values a granule, with 1, 2, 4, 8 or 16 granules; a block per row 2048.  Widths below, at and beyond each edge, with the K
slices that the projections of that width leave, through a context pass and the decode steps behind it, against the CPU
oracle (2e-2, the tolerance of the bf16 path; with low parts less than a third of the difference without them)."""

import pytest

import pd_inputs as pi
from pd_inputs.configs import WorkloadConfig, DTYPE_BF16, NORM_RMSNORM
from parity_util import oracle_run, make_decoder, compare_teacher_forced

pytestmark = pytest.mark.gpu

WIDTHS = [480, 512, 544, 1024, 1056, 2048, 2080, 4128]


@pytest.mark.parametrize("rms", [False, True], ids=["layernorm", "rmsnorm"])
@pytest.mark.parametrize("d", WIDTHS)
def test_norms_of_a_context_and_of_steps(d, rms):
    from paper_2506_23431_amd import binding
    cfg = WorkloadConfig(name=f"norm-{d}", seed=211, dtype=DTYPE_BF16, n_layer=2, d_model=d, n_head=d // 32, head_dim=32,
                         d_ff=512 if d < 2000 else 256, vocab=259, batch=1, ctx_len=150 if d < 4000 else 131, n_sub=2, delta_t=1,
                         sub_tokens=2, norm_init="random", qkv_std=0.5 * d ** -0.5, **({"norm_kind": NORM_RMSNORM} if rms else {}))
    print(f"[norm-rows] {cfg}", flush=True)
    w, ctx = pi.make_weights(cfg, threads=4), pi.make_context(cfg)
    outs = oracle_run(cfg, w, ctx)
    worst = {}
    for split in (1, 0):
        dec = make_decoder(cfg, w)
        dec.set_option(binding.PD_OPT_SPLIT_ACT, split)
        worst[split] = compare_teacher_forced(cfg, w, ctx, dec, outs, log=lambda m: print(m, flush=True))["worst"]
        dec.close()
    assert 3 * worst[1] < worst[0]
