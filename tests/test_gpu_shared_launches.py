"""Requests that share launches: contexts in one context pass (as many as fit a chunk, the rest in another), training
targets of different lengths in one teacher-forced pass (rows padded to the longest), against the CPU oracle request by
request.  The chunk option splits the same requests into other groups; the bf16 tolerance is 2e-2, fp32 1e-4."""

import ctypes as C

import numpy as np
import pytest

import pd_inputs as pi
from oracle import training
from oracle.model import OracleModel
from pd_inputs.configs import WorkloadConfig, DTYPE_BF16, DTYPE_F32, FFN_SWIGLU, NORM_RMSNORM, POS_ROPE
from parity_util import oracle_run, make_decoder, compare_teacher_forced
from test_library import config_struct

pytestmark = pytest.mark.gpu

LLAMA = dict(ffn_kind=FFN_SWIGLU, norm_kind=NORM_RMSNORM, pos_kind=POS_ROPE)


def W(name, **kw):
    base = dict(name=name, seed=151, dtype=DTYPE_BF16, n_layer=2, d_model=128, n_head=2, head_dim=64, d_ff=256, vocab=517,
                batch=5, ctx_len=45, n_sub=3, delta_t=2, sub_tokens=5, norm_init="random", qkv_std=0.1)
    base.update(kw)
    return WorkloadConfig(**base)


CASES = [
    W("hd64"),                                                         # rows of a request not a multiple of 16
    W("hd128-llama", d_model=256, n_head=2, head_dim=128, d_ff=352, ctx_len=64, qkv_std=0.05, **LLAMA),
    W("hd32-one-token", d_model=96, n_head=3, head_dim=32, d_ff=160, ctx_len=1, batch=7),
    W("f32", dtype=DTYPE_F32, ctx_len=77),
    W("f32-llama", dtype=DTYPE_F32, d_model=60, n_head=5, head_dim=12, ctx_len=33, **LLAMA),
]
TARGETS = [W("long-targets", n_sub=4, delta_t=1, sub_tokens=30)]


@pytest.mark.parametrize("chunk", [0, 112], ids=["all", "two-at-a-time"])
@pytest.mark.parametrize("cfg", CASES, ids=[c.name for c in CASES])
def test_contexts_share_a_launch(cfg, chunk):
    from paper_2506_23431_amd import binding
    print(f"[shared] {cfg} chunk {chunk}", flush=True)
    w, ctx = pi.make_weights(cfg, threads=4), pi.make_context(cfg)
    outs = oracle_run(cfg, w, ctx)
    dec = make_decoder(cfg, w)
    dec.set_option(binding.PD_OPT_PREFILL_CHUNK, chunk)
    stats = compare_teacher_forced(cfg, w, ctx, dec, outs, log=lambda m: print(m, flush=True))
    assert stats["rows"] == cfg.batch * (cfg.n_sub * (cfg.sub_tokens + 1) - 1)
    dec.close()


def test_workspace_without_room_for_shared_contexts(monkeypatch):
    """A workspace that holds the rows of one context per launch (what the library asked for before contexts shared
    launches) is taken, the contexts then have launches of their own; a smaller one is refused."""
    from paper_2506_23431_amd import binding
    cfg = W("one-context-per-launch", d_model=768, n_head=12, d_ff=3072, vocab=2003, batch=24, ctx_len=200, delta_t=1,
            sub_tokens=4, qkv_std=0.05)
    one_context = 86428928
    lib = binding.load()
    assert lib.pd_workspace_bytes(C.byref(config_struct(cfg))) > one_context
    w, ctx = pi.make_weights(cfg, threads=4), pi.make_context(cfg)
    outs = oracle_run(cfg, w, ctx)
    monkeypatch.setattr(lib, "pd_workspace_bytes", lambda c: one_context)
    dec = make_decoder(cfg, w)
    stats = compare_teacher_forced(cfg, w, ctx, dec, outs, log=lambda m: print(m, flush=True))
    assert stats["rows"] == cfg.batch * (cfg.n_sub * (cfg.sub_tokens + 1) - 1)
    dec.close()
    monkeypatch.setattr(lib, "pd_workspace_bytes", lambda c: one_context // 2)
    with pytest.raises(binding.PdError, match="workspace too small"):
        make_decoder(cfg, w)


@pytest.mark.parametrize("name,lens", [
    ("hd64", [[5, 3, 2], [2], [6, 5, 6], [1, 1], [6]]),          # 10, 2, 17, 2 and 6 rows, padded to 17
    ("hd128-llama", [[6, 6, 6], [3, 6], [6], [2, 2, 2], [6, 4, 5]]),
    # 124, 1, 90, 124 and 31 rows where a pass holds 256: groups that begin behind request 0
    ("long-targets", [[31, 31, 31, 31], [1], [30, 30, 30], [31, 31, 31, 31], [31]]),
])
def test_targets_share_a_pass(name, lens):
    """Every request's logits, terms and loss, request by request; without low parts the logits are several times further
    off, so that a product that left them out would show."""
    cfg = next(c for c in CASES + TARGETS if c.name == name)
    print(f"[shared] {cfg} targets {lens}", flush=True)
    w, ctx = pi.make_weights(cfg, threads=4), pi.make_context(cfg)
    rng = np.random.default_rng(3)
    targets = [[[0] + [int(t) for t in rng.integers(1, cfg.vocab, n - 1)] for n in t] for t in lens]
    from paper_2506_23431_amd import binding
    model = OracleModel(cfg, w)
    dec = make_decoder(cfg, w)
    dec.prefill_context(ctx, cfg.n_sub, cfg.delta_t, cfg.sub_tokens, cfg.time_steps)
    for _ in range(2):                # the second pass meets the tags and caches of the first
        logits, nll, loss = dec.teacher_forced(targets)
        for b, target in enumerate(targets):
            want, terms, total = training.teacher_forced(model, ctx[b], target, cfg.delta_t)
            assert np.abs(logits[b].cpu().numpy() - want).max() < 2e-2
            assert np.abs(nll[b] - terms).max() < 4e-2 and abs(loss[b] - total) < 4e-2 * max(1, len(terms))
        targets = [t[::-1] if i % 2 else t for i, t in enumerate(targets)]
    off = {}
    for split_act in (0, 1):
        dec.set_option(binding.PD_OPT_SPLIT_ACT, split_act)
        logits, _, _ = dec.teacher_forced(targets)
        off[split_act] = max(np.abs(logits[b].cpu().numpy() - training.teacher_forced(model, ctx[b], t, cfg.delta_t)[0]).max()
                             for b, t in enumerate(targets))
    print(f"[shared] {name}: {off}", flush=True)
    assert 3 * off[1] < off[0]
    dec.close()


def test_nothing_is_written_behind_a_target():
    """A pass pads every request's rows to the longest of its group: the caller's logits and terms keep what they held from
    a request's last row on."""
    import torch
    from paper_2506_23431_amd import binding
    cfg = CASES[0]
    w, ctx = pi.make_weights(cfg, threads=4), pi.make_context(cfg)
    lens, cap, mark = [[5, 3, 2], [2], [6, 5, 6], [1, 1], [6]], 20, 12345.0
    target = np.full((cfg.batch, cfg.n_sub, 6), -1, dtype=np.int32)
    for b, t in enumerate(lens):
        for i, n in enumerate(t):
            target[b, i, :n] = np.arange(n) + 2 + b
    dec = make_decoder(cfg, w)
    dec.prefill_context(ctx, cfg.n_sub, cfg.delta_t, cfg.sub_tokens, cfg.time_steps)
    logits = torch.full((cfg.batch, cap, cfg.vocab), mark, device="cuda:0")
    nll = np.full((cfg.batch, cap), mark, dtype=np.float32)
    loss, rows = np.zeros(cfg.batch), np.zeros(cfg.batch, dtype=np.int32)
    i32p = C.POINTER(C.c_int32)
    assert dec.lib.pd_teacher_forced(dec.ctx, target.ctypes.data_as(i32p), 6, C.c_void_p(logits.data_ptr()), cap,
                                     nll.ctypes.data_as(C.POINTER(C.c_float)), loss.ctypes.data_as(C.POINTER(C.c_double)),
                                     rows.ctypes.data_as(i32p), dec._stream()) == 0
    logits = logits.cpu().numpy()
    assert rows.tolist() == [sum(t) for t in lens]
    for b, n in enumerate(rows):
        assert (logits[b, n:] == mark).all() and (nll[b, n:] == mark).all()
        assert (logits[b, :n] != mark).all() and (nll[b, :n] != mark).all()
    dec.close()
