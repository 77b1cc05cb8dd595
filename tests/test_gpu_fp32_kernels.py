"""The fp32-activation kernels at the edges of their tiles: row counts beside 16, 32 and 64, widths that are and are not
multiples of the 16-value steps or of 4 (scalar loads), head sizes of every instantiation (16-dim blocks 1, 2, 4, 8, 16
and sizes in between), key counts beside the 16-key tiles, norms inside the projections (at most 32 rows of up to 1024
values) and outside, rows embedded by the first projection or by a kernel.  Against the CPU oracle: 1e-4 in fp32, 2e-2
with bf16 weights and the half cache (tests/parity_util.py)."""

import numpy as np
import pytest
import torch

import pd_inputs as pi
from pd_inputs.configs import WorkloadConfig, DTYPE_BF16, DTYPE_F32, FFN_GELU, FFN_SWIGLU, NORM_RMSNORM, POS_ROPE
from parity_util import oracle_run, make_decoder, compare_teacher_forced

pytestmark = pytest.mark.gpu

LLAMA = dict(ffn_kind=FFN_SWIGLU, norm_kind=NORM_RMSNORM, pos_kind=POS_ROPE)


def W(name, heads, hd, ff, ctx, **kw):
    base = dict(name=name, seed=141, dtype=DTYPE_F32, n_layer=2, d_model=heads * hd, n_head=heads, head_dim=hd, d_ff=ff,
                vocab=131, batch=1, ctx_len=ctx, n_sub=3, delta_t=1, sub_tokens=3, norm_init="random", qkv_std=0.05)
    base.update(kw)
    return WorkloadConfig(**base)


CASES = [
    W("hd2", 3, 2, 7, 15, qkv_std=0.5),                        # K = 6 and 7: scalar loads, fewer than 16 values
    W("hd10", 5, 10, 33, 17, qkv_std=0.3),                     # K = 50, 33
    W("hd16", 4, 16, 100, 33, batch=3),                        # K = 64, 100; rows of three requests
    W("hd24-llama", 2, 24, 65, 31, **LLAMA),
    W("hd32", 9, 32, 257, 129, batch=2),                       # K = 288 (8 waves); context of 128 + 1 rows
    W("hd50", 2, 50, 300, 65),                                 # scalar keys
    W("hd64-16rows", 2, 64, 256, 40, n_sub=8, sub_tokens=9, batch=2),    # 16 rows
    W("hd64-33rows", 1, 64, 256, 64, n_sub=11, sub_tokens=11, batch=3),  # 33 rows: norm and embedding kernels
    W("hd80", 7, 80, 1100, 50),                                # K = 560 (16 waves), 1100
    W("hd96-llama", 11, 96, 1056, 47, **LLAMA),                # d = 1056: norms outside the projections
    W("hd130", 2, 130, 96, 70),
    W("hd256", 2, 256, 2100, 81),                              # K = 512, 2100
    W("bf16-hd48", 3, 48, 200, 90, dtype=DTYPE_BF16, batch=2),
    W("bf16-hd80-llama", 2, 80, 199, 33, dtype=DTYPE_BF16, **LLAMA),
]


@pytest.mark.parametrize("cfg", CASES, ids=[c.name for c in CASES])
def test_fp32_kernels(cfg):
    print(f"[fp32] {cfg}", flush=True)
    w, ctx = pi.make_weights(cfg, threads=4), pi.make_context(cfg)
    outs = oracle_run(cfg, w, ctx)
    for pair_layers in ([-1, 1] if cfg.dtype == DTYPE_BF16 else [-1]):
        dec = make_decoder(cfg, w, kv_pair_layers=pair_layers)
        stats = compare_teacher_forced(cfg, w, ctx, dec, outs, log=lambda m: print(m, flush=True))
        assert stats["rows"] == cfg.batch * (cfg.n_sub * (cfg.sub_tokens + 1) - 1)
        dec.close()


def test_more_requests_than_a_grid_dimension_holds():
    """65600 requests in one batch (the second and third grid dimension end at 65535), their contexts 16 different
    tokens over and over: every request's logits are those of its token in a batch of 16."""
    cfg = W("many-requests", 2, 2, 8, 1, n_layer=1, n_sub=1, sub_tokens=1, batch=16, qkv_std=0.5)
    w = pi.make_weights(cfg, threads=4)
    logits = {}
    for batch in (16, 65600):
        dec = make_decoder(cfg, w, max_batch=batch)
        dec.prefill_context(np.arange(batch, dtype=np.int32)[:, None] % 16, 1, 1, 1, 1)
        logits[batch] = dec.decode_step(want_logits=True)[1].cpu().numpy()
        dec.close()
    want = np.tile(logits[16], (65600 // 16, 1, 1))
    assert np.abs(logits[65600] - want).max() < 1e-4


@pytest.mark.parametrize("scale", [1e5, 1e6, 1e7])
@pytest.mark.parametrize("heads,hd,ctx", [(4, 16, 70), (2, 64, 300)])
def test_scores_far_apart(heads, hd, ctx, scale):
    """Query and key rows scaled so that a row's scores differ by 1e6 to 1e14: one key takes the whole weight, every other
    exponential is 0 (its argument is beyond what a 32-bit product can be reduced from), in the tiles of a wave, between
    them and where the waves are merged."""
    cfg = W(f"scores-{scale:g}", heads, hd, 100, ctx)
    w, tokens = pi.make_weights(cfg, threads=4), pi.make_context(cfg)
    for layer in w["layers"]:
        layer["wqkv"][:2 * cfg.d_model] *= np.float32(scale)
    dec = make_decoder(cfg, w)
    compare_teacher_forced(cfg, w, tokens, dec, oracle_run(cfg, w, tokens), log=lambda m: print(m, flush=True))
    dec.close()


def test_more_heads_than_16_bits_hold(monkeypatch):
    """65600 heads of 2 values (bf16 weights, fp32 kernels).  Queries and keys are 0, so every key has the same weight; values
    and output projection use one value of one head beyond 2^16, and what it adds to the rows is known: v = u[5] of the
    normalised row, x[7] += the mean of v over the keys so far."""
    from paper_2506_23431_amd import binding
    H, d, V = 65600, 131200, 64
    if torch.cuda.mem_get_info()[0] < 160e9:
        torch.cuda.empty_cache()
        if torch.cuda.mem_get_info()[0] < 160e9:
            pytest.skip("needs 150 GB of device memory")
    shape = WorkloadConfig(name="heads", seed=1, dtype=DTYPE_BF16, n_layer=1, d_model=d, n_head=H, head_dim=2, d_ff=16, vocab=V,
                           ffn_kind=FFN_GELU, norm_kind=NORM_RMSNORM, ctx_len=3, n_sub=1, sub_tokens=2)
    bf = dict(dtype=torch.bfloat16, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(3)
    emb, head = torch.randn((V, d), generator=g, device="cuda").bfloat16(), torch.randn((V, d), generator=g, device="cuda").mul_(0.01).bfloat16()
    channel = 2 * (H - 3) + 1
    mats = {"wqkv": torch.zeros((3 * d, d), **bf), "wo": torch.zeros((d, d), **bf), "w1": torch.zeros((16, d), **bf),
            "w2": torch.zeros((d, 16), **bf)}
    mats["wqkv"][2 * d + channel, 5] = 1.0
    mats["wo"][7, channel] = 300.0
    ones, pos = torch.ones(d, device="cuda"), torch.zeros((16, d), **bf)

    def upload(torch_, device, shape_, weights):
        w = binding.PdWeights()
        w.tok_emb, w.pos_emb, w.lm_head, w.final_norm_g = emb.data_ptr(), pos.data_ptr(), head.data_ptr(), ones.data_ptr()
        arrays = []
        for name, t in {**mats, "norm1_g": ones, "norm2_g": ones}.items():
            arrays.append((binding.C.c_void_p * 1)(t.data_ptr()))
            setattr(w, name, binding.C.cast(arrays[-1], binding.C.POINTER(binding.C.c_void_p)))
        return w, [], arrays

    monkeypatch.setattr(binding, "_upload_weights", upload)
    dec = binding.PipelinedDecoder(shape, {}, max_batch=1, max_ctx=3, max_sub=1, max_sub_tokens=2, max_pos=16)
    dec.prefill_context(np.array([[9, 21, 40]], dtype=np.int32), 1, 1, 2, 2)
    logits = dec.decode_step(want_logits=True)[1][0, 0].double()
    dec.close()
    mats.clear()
    torch.cuda.empty_cache()
    x = emb[[9, 21, 40, 0]].double()                       # the context and <bos>
    u = x * torch.rsqrt(x.square().mean(1, keepdim=True) + shape.norm_eps)
    y = x[3].clone()
    y[7] += 300.0 * u[:, 5].mean()
    want = head.double() @ (y * torch.rsqrt(y.square().mean() + shape.norm_eps))
    without = head.double() @ (x[3] * torch.rsqrt(x[3].square().mean() + shape.norm_eps))
    assert float((want - without).abs().max()) > 0.1       # (the head's share is visible)
    assert float((logits - want).abs().max()) < 2e-2


@pytest.mark.parametrize("ctx", [96, 113, 128])
def test_row_tiles_per_block(ctx):
    """Context passes whose first FFN projection (2048 x 512) takes two row tiles per block (96 rows) and four, the last group
    whole and not; the other projections take one."""
    cfg = W(f"rows-{ctx}", 8, 64, 2048, ctx)
    w, tokens = pi.make_weights(cfg, threads=4), pi.make_context(cfg)
    dec = make_decoder(cfg, w)
    compare_teacher_forced(cfg, w, tokens, dec, oracle_run(cfg, w, tokens), log=lambda m: print(m, flush=True))
    dec.close()
