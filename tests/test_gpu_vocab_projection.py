"""The vocabulary projection of steps of 33-128 rows: shared row tiles of 4, 5 and 8, one and two column tiles per wave, on both
sides of the line between the two kernels (1500 tiles of 16 words; 1025 with 8 row tiles), vocabularies that end inside a
tile, weights with and without the non-temporal hint.  Every logit row against the CPU oracle, 2e-2."""

import pytest

import pd_inputs as pi
from pd_inputs.configs import WorkloadConfig, DTYPE_BF16
from parity_util import oracle_run, make_decoder, compare_teacher_forced

pytestmark = pytest.mark.gpu


def W(name, batch, n_sub, vocab, d=128):
    return WorkloadConfig(name=name, seed=173, dtype=DTYPE_BF16, n_layer=1, d_model=d, n_head=d // 64, head_dim=64, d_ff=2 * d,
                          vocab=vocab, batch=batch, ctx_len=20, n_sub=n_sub, delta_t=1, sub_tokens=n_sub, norm_init="random",
                          qkv_std=0.08)


CASES = [
    W("33-rows-4x1", 3, 11, 24001), W("33-rows-K-cut", 3, 11, 23983), W("64-rows-4x2", 8, 8, 65553),
    W("65-rows-5x1", 5, 13, 24001), W("80-rows-5x2", 8, 10, 65553),
    W("81-rows-8x1", 9, 9, 16399), W("128-rows-K-cut", 8, 16, 16384), W("128-rows-8x2", 8, 16, 32770, d=640),
]


@pytest.mark.parametrize("stream", [0, 1])
@pytest.mark.parametrize("cfg", CASES, ids=[c.name for c in CASES])
def test_vocabulary_projection_of_many_rows(cfg, stream):
    from paper_2506_23431_amd import binding
    print(f"[vocab] {cfg}", flush=True)
    w, ctx = pi.make_weights(cfg, threads=4), pi.make_context(cfg)
    outs = oracle_run(cfg, w, ctx)
    dec = make_decoder(cfg, w)
    dec.set_option(binding.PD_OPT_STREAM_LOADS, stream)
    stats = compare_teacher_forced(cfg, w, ctx, dec, outs, log=lambda m: print(m, flush=True))
    assert stats["rows"] == cfg.batch * (cfg.n_sub * (cfg.sub_tokens + 1) - 1)
    if stream == 0:     # without low parts (the kernel that cuts K): an order of magnitude further off
        dec.set_option(binding.PD_OPT_SPLIT_ACT, 0)
        single = compare_teacher_forced(cfg, w, ctx, dec, outs, tol=0.1, log=lambda m: print(m, flush=True))
        assert 3 * stats["worst"] < single["worst"]
    dec.close()
