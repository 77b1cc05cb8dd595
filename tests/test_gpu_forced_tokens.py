"""Forced tokens on their two ways into a step: through mapped host memory (single steps) and through the device copy that a
replayed step looks at (PD_OPT_USE_GRAPH).  Steps that force tokens with and without a look at the outputs, steps that force
none and steps with logits (never replayed) follow each other; tokens and logits are those of the same steps without replay,
bit for bit (more than 8 rows: the layout of the activations is the same on both sides)."""

import numpy as np
import pytest
import torch

import pd_inputs as pi
from pd_inputs.configs import WorkloadConfig, DTYPE_BF16, DTYPE_F32
from paper_2506_23431_amd import binding
from parity_util import make_decoder

pytestmark = pytest.mark.gpu


def run(cfg, w, ctx, force, graph):
    """What twelve steps return: tokens and logits, in the order of the steps."""
    dec = make_decoder(cfg, w)
    dec.set_option(binding.PD_OPT_USE_GRAPH, graph)
    dec.prefill_context(ctx, cfg.n_sub, cfg.delta_t, cfg.sub_tokens, cfg.time_steps)
    out = []
    for t in range(12):
        print(f"[forced] graph {graph} step {t}", flush=True)
        if t % 4 == 0:                  # forced, nothing read: the call returns before the step has run
            dec.decode_step(force=force[t], want_tokens=False, want_done=False)
        elif t % 4 == 1:                # forced, tokens read
            out.append(dec.decode_step(force=force[t])[0])
        elif t % 4 == 2:                # the library's own tokens
            out.append(dec.decode_step()[0])
        else:                           # forced, with logits
            tokens, logits, _ = dec.decode_step(force=force[t], want_logits=True)
            out += [tokens, logits.cpu().numpy()]
    dec.close()
    return out


@pytest.mark.parametrize("dtype", [DTYPE_F32, DTYPE_BF16])
def test_forced_tokens_of_replayed_steps(dtype):
    cfg = WorkloadConfig(name="forced", seed=61, dtype=dtype, n_layer=2, d_model=128, n_head=2, head_dim=64, d_ff=256, vocab=211,
                         batch=3, ctx_len=19, n_sub=5, delta_t=1, sub_tokens=12, norm_init="random", qkv_std=0.08)
    w, ctx = pi.make_weights(cfg, threads=4), pi.make_context(cfg)
    rng = np.random.default_rng(5)
    force = rng.integers(0, cfg.vocab, (12, cfg.batch, cfg.n_sub), dtype=np.int32)
    force[rng.random(force.shape) < 0.4] = -1
    seen = []
    for graph in (0, 1):
        with torch.cuda.stream(torch.cuda.Stream()):          # (the default stream cannot be captured)
            seen.append(run(cfg, w, ctx, force, graph))
    for a, b in zip(*seen):
        assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f")
    forced = [force[t] for t in (1, 3, 5, 7, 9, 11)]
    got = [seen[0][i] for i in (0, 2, 4, 6, 8, 10)]
    for f, g in zip(forced, got):
        assert np.array_equal(g[(f >= 0) & (g >= 0)], f[(f >= 0) & (g >= 0)])
