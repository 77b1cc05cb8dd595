"""A model whose step reads more than the last-level cache holds: the matrices that start within the first 110 MB of its
packed weights are loaded without the non-temporal hint, the others with it.  Here those are the first layer's four (101 MB) and one
of the second's (25 MB); logits and tokens are the same bits as with the hint on every weight and on none, for packed, general and many rows."""

import numpy as np
import pytest
import torch

import pd_inputs as pi
from pd_inputs.configs import WorkloadConfig, DTYPE_BF16
from parity_util import make_decoder

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,n_sub", [(1, 4), (2, 6), (5, 8)])
def test_same_bits_wherever_the_hint_is(batch, n_sub):
    from paper_2506_23431_amd import binding
    cfg = WorkloadConfig(name="kept", seed=233, dtype=DTYPE_BF16, n_layer=2, d_model=2048, n_head=16, head_dim=128, d_ff=8192,
                         vocab=32000, batch=batch, ctx_len=33, n_sub=n_sub, delta_t=1, sub_tokens=9, norm_init="random", qkv_std=0.02)
    print(f"[kept] {cfg}", flush=True)
    w, ctx = pi.make_weights(cfg, threads=8), pi.make_context(cfg)
    out = {}
    for stream in (None, 1, 2, 0):
        dec = make_decoder(cfg, w)
        assert dec.get_info(binding.PD_INFO_STREAM_LOADS) == 1
        if stream is not None:
            dec.set_option(binding.PD_OPT_STREAM_LOADS, stream)
        assert dec.get_info(binding.PD_INFO_KEPT_BYTES) == (2 * 15 * 2048 ** 2 if stream in (None, 1) else 0)
        dec.prefill_context(ctx, n_sub, 1, 9, n_sub + 9)
        steps = [dec.decode_step(want_logits=True) for _ in range(n_sub + 1)]
        out[stream] = [(np.array(s[0]), s[1].clone()) for s in steps]
        dec.close()
    for stream in (1, 2, 0):
        for (t0, l0), (t1, l1) in zip(out[None], out[stream]):
            assert np.array_equal(t0, t1) and torch.equal(torch.nan_to_num(l0), torch.nan_to_num(l1))


@pytest.mark.parametrize("d_ff,chosen,kept", [(8192, 1, 2 * 15 * 2048 ** 2), (512, 0, 0)])
def test_the_choice_of_the_creation_comes_back(d_ff, chosen, kept):
    """Every value that the option takes can be set again as it was read, and 1 brings back what creation kept."""
    from paper_2506_23431_amd import binding
    cfg = WorkloadConfig(name="kept", seed=233, dtype=DTYPE_BF16, n_layer=2, d_model=2048, n_head=16, head_dim=128, d_ff=d_ff,
                         vocab=32000, batch=1, ctx_len=9, n_sub=2, delta_t=1, sub_tokens=3, norm_init="random", qkv_std=0.02)
    dec = make_decoder(cfg, pi.make_weights(cfg, threads=8))

    def state():
        return dec.get_info(binding.PD_INFO_STREAM_LOADS), dec.get_info(binding.PD_INFO_KEPT_BYTES)
    assert state() == (chosen, kept)
    for value, then in ((chosen, kept), (0, 0), (1, kept), (2, 0), (2, 0), (chosen, kept)):
        dec.set_option(binding.PD_OPT_STREAM_LOADS, value)
        assert state() == (value, then)
    dec.close()
