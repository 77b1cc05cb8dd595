"""Contexts whose buffers pass 2^31 values or whose matrices pass 2^16 k-tiles: what a step reads lies where a 32-bit
product of sizes would not find it.  Little of such a context is used (one request of its capacity), so that the CPU oracle
can say what the logits are: 2e-2 with bf16 weights."""

import pytest
import torch

import pd_inputs as pi
from pd_inputs.configs import WorkloadConfig, DTYPE_BF16
from parity_util import oracle_run, make_decoder, compare_teacher_forced

pytestmark = pytest.mark.gpu


def W(name, **kw):
    base = dict(name=name, seed=57, dtype=DTYPE_BF16, n_layer=1, d_model=2048, n_head=16, head_dim=128, d_ff=1024, vocab=131,
                batch=1, ctx_len=15, n_sub=7, delta_t=1, sub_tokens=6, norm_init="random", qkv_std=0.05)
    base.update(kw)
    return WorkloadConfig(**base)


def parity(cfg, gigabytes, **capacity):
    if torch.cuda.mem_get_info()[0] < (gigabytes + 10) * 1e9:
        torch.cuda.empty_cache()
        if torch.cuda.mem_get_info()[0] < (gigabytes + 10) * 1e9:
            pytest.skip(f"needs {gigabytes} GB of device memory")
    w, ctx = pi.make_weights(cfg, threads=4), pi.make_context(cfg)
    outs = oracle_run(cfg, w, ctx)
    dec = make_decoder(cfg, w, **capacity)
    try:
        assert dec.workspace_bytes < gigabytes * 1e9
        compare_teacher_forced(cfg, w, ctx, dec, outs, log=lambda m: print(m, flush=True))
    finally:
        dec.close()
        del dec
        torch.cuda.empty_cache()


def test_row_buffers_beyond_32_bits():
    """1050000 rows of 2048 values: the K slices that the last norm adds lie 2^31 values apart."""
    parity(W("rows"), 180, max_batch=150000)


def test_inner_width_of_65536_k_tiles():
    """An FFN of 2^21 inner values: the second projection runs over 65536 k-tiles, in steps and in the context pass."""
    parity(W("inner", n_layer=2, d_model=32, n_head=1, head_dim=32, d_ff=1 << 21, ctx_len=20, n_sub=3, sub_tokens=3), 10)


def test_caches_more_than_64_gib_long():
    """Values lie 68.7 GB behind their keys (64 requests of 262150 context tokens, one of them in use)."""
    parity(W("keys", ctx_len=40, n_sub=3, sub_tokens=4), 150, max_batch=64, max_ctx=262150)
