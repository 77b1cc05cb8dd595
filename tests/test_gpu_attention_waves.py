"""The attention kernel's launch shapes in decode steps: one work-group of 8 waves per request and head (short key sets),
of 4 waves (more units than compute units), and splits with the merge kernel, at key counts around the edges of the
rule (32 and 96 blocks of 32 keys over the capacity of the run) and with fewer key blocks than waves; every head size,
with and without low parts, decoder-only and encoder-decoder.  Against the CPU oracle, tolerance 2e-2 (bf16)."""

import pytest

import pd_inputs as pi
from pd_inputs.configs import WorkloadConfig, DTYPE_BF16
from parity_util import oracle_run, make_decoder, compare_teacher_forced

pytestmark = pytest.mark.gpu


def W(name, heads, hd, ctx, **kw):
    base = dict(name=name, seed=161, dtype=DTYPE_BF16, n_layer=1, d_model=heads * hd, n_head=heads, head_dim=hd, d_ff=128,
                vocab=203, batch=1, ctx_len=ctx, n_sub=3, delta_t=1, sub_tokens=4, norm_init="random", qkv_std=0.08)
    base.update(kw)
    return WorkloadConfig(**base)


CASES = [
    W("one-block-hd64", 2, 64, 5),                      # one key block, 8 waves
    W("hd32-31-blocks", 3, 32, 977),                    # 32 blocks of capacity: at the first edge
    W("hd64-33-blocks", 2, 64, 1020),                   # just beyond it
    W("hd96-64-blocks", 2, 96, 2033),
    W("hd128-96-blocks", 1, 128, 3050),                 # at the second edge
    W("hd64-97-blocks", 1, 64, 3085),                   # splits and merge
    W("hd128-pairs", 2, 128, 300, qkv_std=0.03),        # (pair layers keep 4 waves)
    W("hd32-many-units", 13, 32, 40, batch=20),         # 260 units: 4 waves
]


@pytest.mark.parametrize("split_act", [1, 0])
@pytest.mark.parametrize("cfg", CASES, ids=[c.name for c in CASES])
def test_launch_shapes(cfg, split_act):
    from paper_2506_23431_amd import binding
    print(f"[attn-waves] {cfg}", flush=True)
    w, ctx = pi.make_weights(cfg, threads=4), pi.make_context(cfg)
    outs = oracle_run(cfg, w, ctx)
    dec = make_decoder(cfg, w, kv_pair_layers=1 if cfg.name == "hd128-pairs" else -1)
    dec.set_option(binding.PD_OPT_SPLIT_ACT, split_act)
    stats = compare_teacher_forced(cfg, w, ctx, dec, outs, log=lambda m: print(m, flush=True))
    assert stats["rows"] == cfg.batch * (cfg.n_sub * (cfg.sub_tokens + 1) - 1)
    dec.close()
