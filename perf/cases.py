"""The workloads whose speed counts, through the public entry points of paper_2506_23431_amd.

Every case is a model (random weights at the scales of a trained one, made from the seed), a batch of contexts and a
schedule of Algorithm 1, and one of these uses of them:

  decode   contexts are encoded already; `steps` time-steps from t = 1 in one go, the logits of the last one
           (a server that lets the library pick the tokens)
  client   the same, one step per call with forced tokens going in and tokens and logits coming out of each
           (a program that samples or ends subsequences itself)
  context  new contexts are encoded, then the first time-step gives logits (time to the first token)
  whole    new contexts are encoded, then `steps` time-steps
  train    new contexts are encoded, then whole training targets are fed in one pass: logits, terms and loss

Greedy tokens are fed back, so a tie that two correct programs break differently would change everything behind it.
The vocabulary projection is therefore the (shifted) embedding table, as in models that tie the two, which gives the
winner the clear margin it has in a trained model; the logits themselves are what is compared.

Sizes are those of pd_inputs (cfg1 ... cfg5, encdec-*), of the tests, or generic.
"""

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2506_23431_amd import PipelinedDecoder
from paper_2506_23431_amd import binding

SHIFT = 37                      # the likeliest successor of token v is v + SHIFT (mod vocabulary)


def _case(name, use, kind, layers, d, heads, ff, vocab, batch, ctx, subs, delay, tokens, steps, gated=False, pairs=True):
    return {"name": name, "use": use, "kind": kind, "layers": layers, "d": d, "heads": heads, "ff": ff, "vocab": vocab,
            "batch": batch, "ctx": ctx, "subs": subs, "delay": delay, "tokens": tokens, "steps": steps,
            "gated": gated, "pairs": pairs}


def listed():
    # kind: "f32" (fp32 weights and cache), "bf16", "encdec" (bf16 encoder-decoder); gated: RMS norm, SwiGLU, rotary
    # positions instead of LayerNorm, GELU, learned positions; pairs: the context pass keeps bf16 pairs (the default)
    return [
        # cfg1 over its whole run: the smallest model, fp32 end to end; launches and latency only
        _case("f32-tiny", "decode", "f32", 1, 64, 4, 256, 512, 1, 128, 4, 2, 16, 22),
        # an ordinary fp32 model (reference-precision runs), context and decoding
        _case("f32-mid", "whole", "f32", 4, 512, 8, 2048, 8192, 2, 257, 6, 2, 16, 12),
        # cfg2, one request: an interactive model that the last-level cache holds, steady state of 8 rows
        _case("small-decode", "decode", "bf16", 6, 768, 12, 3072, 50265, 1, 1024, 8, 4, 64, 36),
        # cfg2's model driven step by step by a program that decides on the tokens itself
        _case("small-client", "client", "bf16", 6, 768, 12, 3072, 50265, 2, 700, 6, 1, 24, 8),
        # cfg3: a batch of 8 requests, steady state of 9 rows each
        _case("batch-decode", "decode", "bf16", 12, 1024, 16, 4096, 50265, 8, 2048, 16, 4, 32, 40),
        # cfg4, the benchmark workload: 24 layers over one context of 8192 tokens, up to 8 rows
        _case("long-decode", "decode", "bf16", 24, 2048, 16, 8192, 32000, 1, 8192, 32, 8, 64, 64),
        # cfg5's width and schedule, 4 of its 32 layers: 4 requests, up to 64 rows, one pair layer
        _case("wide-decode", "decode", "bf16", 4, 4096, 32, 11008, 32000, 4, 4096, 16, 4, 128, 64, gated=True),
        # many short requests at once: 192 rows per step
        _case("many-decode", "decode", "bf16", 6, 768, 12, 3072, 50265, 24, 384, 8, 1, 32, 12),
        # cfg4's context pass (3 of its 24 layers)
        _case("long-context", "context", "bf16", 3, 2048, 16, 8192, 32000, 1, 8192, 4, 1, 8, 1),
        # cfg5's context pass (2 of its 32 layers), two requests of an odd length
        _case("wide-context", "context", "bf16", 2, 4096, 32, 11008, 32000, 2, 2041, 4, 1, 8, 1, gated=True),
        # cfg2's model in training or scoring: ragged targets of 8 subsequences, 2 requests
        _case("small-train", "train", "bf16", 6, 768, 12, 3072, 50265, 2, 1024, 8, 4, 64, 1),
        # the encoder-decoder form at its base shape, one whole example (512 input tokens)
        _case("encdec-base", "whole", "encdec", 12, 768, 12, 3072, 32128, 1, 512, 8, 1, 16, 20),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _estimate(c):
    """Rough seconds of one pass: what a drawn case costs against the largest listed one."""
    w = work(c)
    rate = 2e12 if c["kind"] == "f32" else 5e13
    return w["bytes"] / 1.5e12 + w["flops"] / rate + 1.2e-4 * c["steps"] * c["layers"]


def draw(rng):
    most = 0.8 * max(_estimate(c) for c in listed())
    while True:
        kind = rng.choice(["f32", "bf16", "bf16", "bf16", "bf16", "encdec"])
        use = rng.choice({"f32": ["decode", "client", "whole"], "encdec": ["whole", "whole", "train"],
                          "bf16": ["decode", "decode", "decode", "client", "context", "context", "whole", "train"]}[kind])
        head = rng.choice([16, 32, 64, 80] if kind == "f32" else [32, 64, 64, 96, 128, 128])
        d = head * max(1, _log(rng, 64, 768 if kind == "f32" else 4096 if kind == "bf16" else 1024) // head)
        if d < 128 and kind != "f32":
            continue
        gated = kind != "encdec" and rng.random() < 0.4
        ff = 32 * max(1, int(d * rng.choice([2.6875, 4, 4, 3.1]) / 32))
        vocab = _log(rng, 500, 8192 if kind == "f32" else 50265)
        layers = _log(rng, 1, 4 if kind == "f32" else 12)
        batch = _log(rng, 1, 4 if kind == "f32" or use == "train" else 24)
        ctx = _log(rng, 16, 500 if kind == "f32" else 6000 if kind == "bf16" else 1024)
        subs, delay, tokens = _log(rng, 1, 16), _log(rng, 1, 6), _log(rng, 8, 96)
        if tokens < delay or batch * subs > 256:
            continue
        steps = 1 if use in ("context", "train") else max(1, min(_log(rng, 4, 48), (subs - 1) * delay + tokens))
        if use == "client":
            steps = min(steps, 8)
        c = _case("", use, kind, layers, d, d // head, ff, vocab, batch, ctx, subs, delay, tokens, steps, gated,
                  kind != "bf16" or d >= 4096 or rng.random() < 0.8)
        c.pop("name")
        if use == "train" and sum(len(r) for r in _lens(c)) and max(map(sum, _lens(c))) > min(subs * (tokens + 1), max(128, ctx // 128 * 128)):
            continue
        weights = 2 * layers * (4 * d * d + 3 * d * ff) + 2 * vocab * d
        keys = layers * batch * (ctx + subs * tokens) * d
        if weights > 6e8 or keys > 2e9 or _estimate(c) > most:
            continue
        return c


# ---- the work of a case -----------------------------------------------------------------------------------

def _lens(c):
    """Training targets: tokens (<bos>, Y, <eos>) of every subsequence of every request, the last one empty."""
    return [[3 + (5 * b + 7 * i + i * i) % max(1, c["tokens"] - 2) for i in range(c["subs"] - 1)] + [2]
            for b in range(c["batch"])]


def _rows(c, t):
    """Rows a request feeds at time-step t: subsequence i from the step that opens it to one after its last token."""
    return [i for i in range(c["subs"]) if 0 <= t - 1 - i * c["delay"] <= c["tokens"]]


def work(c):
    d, ff, V, n, B, L = c["d"], c["ff"], c["vocab"], c["layers"], c["batch"], c["ctx"]
    es = 4 if c["kind"] == "f32" else 2
    mats = (3 if c["gated"] else 2) * d * ff
    encdec = c["kind"] == "encdec"
    layer = (6 if encdec else 4) * d * d + mats           # weights of a decoder layer that a step uses
    nbytes = flops = 0.0
    if c["use"] in ("context", "whole", "train"):
        if encdec:
            enc = 4 * d * d + mats
            nbytes += n * es * (enc + 2 * d * d) + B * n * es * 2 * L * d
            flops += B * n * (2.0 * L * (enc + 2 * d * d) + 4.0 * L * L * d)
        else:                                               # the last layer: keys and values only
            nbytes += es * ((n - 1) * layer + 2 * d * d) + B * n * es * 2 * L * d
            flops += B * (2.0 * L * ((n - 1) * layer + 2 * d * d) + (n - 1) * 2.0 * L * L * d)
    if c["use"] == "train":
        rows = [sum(r) for r in _lens(c)]
        nbytes += es * (n * layer + V * d) + sum(es * n * 2 * (L + r) * d + 4.0 * r * V for r in rows)
        flops += sum(2.0 * r * (n * layer + V * d) + 4.0 * n * r * (L + r / 2) * d for r in rows)
        return {"bytes": nbytes, "flops": flops}
    keys = 0
    for t in range(1, c["steps"] + 1):
        r = len(_rows(c, t))
        keys += r
        nbytes += es * (n * layer + V * d) + B * n * es * 2 * (L + keys) * d
        flops += B * (2.0 * r * (n * layer + V * d) + 4.0 * n * r * (L + keys) * d)
        if c["use"] == "client" or t == c["steps"]:
            nbytes += 4.0 * B * r * V
    return {"bytes": nbytes, "flops": flops}


def tolerance(c):
    # four times the largest errors against exact() over the listed and 210 drawn cases: 4.8e-7 with fp32 throughout; 4.3e-4
    # with activations as bf16 pairs (rounding of the half-precision cache, largest for the shortest contexts, where
    # few keys are averaged); 2.7e-3 where the context pass is asked for single bf16 activations
    if c["kind"] == "f32":
        return {"rel": 2e-6}
    return {"rel": 1.7e-3 if c["pairs"] else 1.1e-2}


# ---- inputs ---------------------------------------------------------------------------------------------------

def _weights(c, seed):
    """Row-major [out][in] weights on the GPU: matrices in the type the model keeps them in, vectors float32.

    Projections keep the scale of what they are fed; query and key scales give scores of standard deviation 2 (an
    attention that looks at a few dozen keys); what a layer adds to the residual stream shrinks with the depth."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    d, ff, V, n = c["d"], c["ff"], c["vocab"], c["layers"]
    kind = torch.float32 if c["kind"] == "f32" else torch.bfloat16

    def normal(*shape, std=1.0):
        return torch.randn(shape, generator=g, device="cuda").mul_(std)

    def mat(*shape, std):
        return normal(*shape, std=std).to(kind)

    def gain():
        return 1 + normal(d, std=0.1)

    encdec = c["kind"] == "encdec"
    hd = d // c["heads"]
    sq = math.sqrt(2.0 / d) * (hd ** -0.25 if encdec else 1.0)   # that family has no 1 / sqrt(head_dim) in its scores

    def attn():
        return torch.cat([mat(2 * d, d, std=sq), mat(d, d, std=d ** -0.5)])

    def layer():
        w = {"wqkv": attn(), "wo": mat(d, d, std=2.0 * (d * n) ** -0.5), "w1": mat(ff, d, std=d ** -0.5),
             "w2": mat(d, ff, std=1.2 * (ff * n) ** -0.5), "norm1_g": gain(), "norm2_g": gain()}
        if c["gated"]:
            w["w_up"] = mat(ff, d, std=d ** -0.5)
        elif not encdec:
            w["norm1_b"], w["norm2_b"] = normal(d, std=0.1), normal(d, std=0.1)
        return w

    se = max(1.0, (512 / d) ** 0.5)             # narrow models: the winner's margin grows with std * sqrt(width) only
    emb = mat(V, d, std=se)
    w = {"tok_emb": emb, "lm_head": (torch.roll(emb, SHIFT, 0).float() * (d ** -0.5 / se)).to(kind)}
    if encdec:
        w["enc_rel_bias"], w["dec_rel_bias"] = normal(32, c["heads"], std=0.5), normal(32, c["heads"], std=0.5)
        w["enc_final_g"], w["dec_final_g"] = gain(), gain()
        w["enc_layers"], w["dec_layers"] = [layer() for _ in range(n)], [layer() for _ in range(n)]
        for lw in w["dec_layers"]:
            lw["cq"] = mat(d, d, std=sq)
            lw["ckv"] = torch.cat([mat(d, d, std=sq), mat(d, d, std=d ** -0.5)])
            lw["co"], lw["norm3_g"] = mat(d, d, std=2.0 * (d * n) ** -0.5), gain()
        return w
    w["final_norm_g"] = gain()
    if not c["gated"]:
        w["final_norm_b"] = normal(d, std=0.1)
        w["pos_emb"] = mat(_positions(c), d, std=0.3)
    w["layers"] = [layer() for _ in range(n)]
    return w


def _positions(c):
    return c["ctx"] + (c["subs"] - 1) * (c["delay"] + 1) + c["tokens"] + 2


def _tokens(c, seed):
    """(contexts [B][L], forced tokens [steps][B][S] of a client, training targets or None)."""
    rng = np.random.default_rng([int(seed), 7])
    B, V = c["batch"], c["vocab"]
    ctx = rng.integers(0, V, (B, c["ctx"]), dtype=np.int32)
    force = rng.integers(0, V, (c["steps"], B, c["subs"]), dtype=np.int32) if c["use"] == "client" else None
    target = None
    if c["use"] == "train":
        target = [[[0] + [int(t) for t in rng.integers(2, V, n - 2)] + [1] for n in lens] for lens in _lens(c)]
    return ctx, force, target


def _shape(c):
    return SimpleNamespace(n_layer=c["layers"], n_enc_layer=c["layers"], n_dec_layer=c["layers"], d_model=c["d"],
                           n_head=c["heads"], head_dim=c["d"] // c["heads"], d_ff=c["ff"], vocab=c["vocab"],
                           ffn_kind=int(c["gated"]), norm_kind=int(c["gated"]), pos_kind=int(c["gated"]),
                           rope_base=10000.0, norm_eps=1e-6 if c["kind"] == "encdec" else 1e-5,
                           dtype=0 if c["kind"] == "f32" else 1, bos_id=0, eos_id=-1, rel_buckets=32,
                           rel_max_distance=128)


def _host(v):
    if isinstance(v, dict):
        return {k: _host(x) for k, x in v.items()}
    if isinstance(v, list):
        return [_host(x) for x in v]
    if v.dtype == torch.bfloat16:
        return v.view(torch.int16).cpu().numpy().view(np.uint16)
    return v.cpu().numpy()


def prepare(case, seed):
    c = case
    weights = _host(_weights(c, seed))
    ctx, force, target = _tokens(c, seed)
    room = dict(max_batch=c["batch"], max_ctx=c["ctx"], max_sub=c["subs"], max_sub_tokens=c["tokens"])
    if c["kind"] == "encdec":
        dec = binding.EncDecPipelinedDecoder(_shape(c), weights, **room)
    else:
        dec = PipelinedDecoder(_shape(c), weights, max_pos=_positions(c), **room)
    if not c["pairs"]:
        dec.set_option(binding.PD_OPT_CONTEXT_SPLIT_ACT, 0)
    state = {"case": c, "dec": dec, "ctx": ctx, "force": force, "target": target,
             "plan": (c["subs"], c["delay"], c["tokens"], (c["subs"] - 1) * c["delay"] + c["tokens"])}
    if c["use"] in ("decode", "client"):
        dec.prefill_context(ctx, *state["plan"])
    return state


def run(state):
    c, dec = state["case"], state["dec"]
    if c["use"] in ("decode", "client"):
        dec.reset_decode()
    else:
        dec.prefill_context(state["ctx"], *state["plan"])
    if c["use"] == "train":
        logits, terms, loss = dec.teacher_forced(state["target"])
        return {"logits": logits, "terms": terms, "loss": loss}
    if c["use"] == "client":
        steps = [dec.decode_step(force=f, want_logits=True) for f in state["force"]]
        return {"tokens": np.stack([s[0] for s in steps]), "logits": [s[1] for s in steps]}
    dec.decode_steps(c["steps"] - 1)
    tokens, logits, _ = dec.decode_step(want_logits=True)
    return {"tokens": tokens, "logits": logits}


# ---- the same in 64 bits ----------------------------------------------------------------------------------------

class _Exact:
    """The model in float64 with library operations: one pass over a request's context and generated tokens."""

    def __init__(self, c, w):
        self.c, self.w, self.s = c, w, _shape(c)

    def norm(self, x, g, b=None):
        x = x.double()
        if self.s.norm_kind == 1 or self.c["kind"] == "encdec":
            return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + self.s.norm_eps) * g.double()
        x = x - x.mean(-1, keepdim=True)
        return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + self.s.norm_eps) * g.double() + b.double()

    def heads(self, y):
        return y.view(y.shape[0], self.c["heads"], -1).transpose(0, 1).contiguous()

    def attend(self, q, k, v, scale, mask, bias=None):
        """q [H][n][hd] over k, v [H][m][hd]; mask(lo, hi) and bias(lo, hi): [hi - lo][m], [H][hi - lo][m]."""
        kt, out = k.transpose(1, 2).contiguous(), torch.empty_like(q)
        step = max(1, int(1.5e8 / (k.shape[0] * k.shape[1])))
        for lo in range(0, q.shape[1], step):
            hi = min(q.shape[1], lo + step)
            s = torch.matmul(q[:, lo:hi].contiguous(), kt).mul_(scale)
            if bias is not None:
                s += bias(lo, hi)
            m = mask(lo, hi)
            if m is not None:
                s.masked_fill_(~m, -math.inf)
            out[:, lo:hi] = torch.matmul(torch.softmax(s, -1), v)
        return out.transpose(0, 1).reshape(q.shape[1], -1)

    def rotate(self, y, pos):
        half = y.shape[2] // 2
        ang = pos.double()[:, None] * self.s.rope_base ** (-torch.arange(half, device="cuda", dtype=torch.float64) / half)
        c, s = ang.cos(), ang.sin()
        a, b = y[..., :half], y[..., half:]
        return torch.cat([a * c - b * s, b * c + a * s], -1)

    def ffn(self, lw, u):
        y = u @ lw["w1"].double().T
        if self.c["kind"] == "encdec":
            y = y.clamp_(min=0)
        elif self.c["gated"]:
            y = torch.nn.functional.silu(y) * (u @ lw["w_up"].double().T)
        else:
            y = torch.nn.functional.gelu(y)
        return y @ lw["w2"].double().T

    def logits(self, x, g, b=None):
        return self.norm(x, g, b) @ self.w["lm_head"].double().T

    def decoder_only(self, ctx, tok, sub, tau):
        """Logits of the generated-side tokens `tok` of subsequences `sub` (from 0) fed at steps `tau` (from 1)."""
        c, w, d, L = self.c, self.w, self.c["d"], len(ctx)
        tok = torch.cat([torch.as_tensor(ctx, device="cuda").long(), tok])
        pos = torch.cat([torch.arange(L, device="cuda"), L + tau - 1 + sub])
        x = w["tok_emb"][tok].double()
        if not c["gated"]:
            x = x + w["pos_emb"][pos].double()
        n = len(tok)
        at = torch.arange(n, device="cuda")
        vis = (sub[None, :] <= sub[:, None]) & (tau[None, :] <= tau[:, None])
        vis = torch.cat([torch.ones(n - L, L, dtype=torch.bool, device="cuda"), vis], 1)

        def mask(lo, hi):
            m = at[None, :] <= at[lo:hi, None]
            if hi > L:
                m[max(L - lo, 0):] = vis[max(lo - L, 0):hi - L]
            return m
        for lw in w["layers"]:
            y = self.norm(x, lw["norm1_g"], lw.get("norm1_b")) @ lw["wqkv"].double().T
            q, k, v = (self.heads(y[:, i * d:(i + 1) * d]) for i in range(3))
            if c["gated"]:
                q, k = self.rotate(q, pos), self.rotate(k, pos)
            x = x + self.attend(q, k, v, q.shape[2] ** -0.5, mask) @ lw["wo"].double().T
            x = x + self.ffn(lw, self.norm(x, lw["norm2_g"], lw.get("norm2_b")))
        return self.logits(x[L:], w["final_norm_g"], w.get("final_norm_b"))

    def bucket(self, n, buckets):
        half = buckets // 2                              # (whole values of the logarithm must not round down)
        far = torch.log(n.clamp(min=1).double() / half) / math.log(128 / half) * (buckets - half)
        far = half + torch.floor(far + 1e-9).long()
        return torch.where(n < half, n, far.clamp(max=buckets - 1))

    def encdec(self, ctx, tok, sub, tau):
        w, d = self.w, self.c["d"]
        x = w["tok_emb"][torch.as_tensor(ctx, device="cuda").long()].double()
        at = torch.arange(len(ctx), device="cuda")
        rel = at[None, :] - at[:, None]
        enc = w["enc_rel_bias"].double()[torch.where(rel > 0, 16, 0) + self.bucket(rel.abs(), 16)].permute(2, 0, 1)

        def everything(lo, hi):
            return None
        for lw in w["enc_layers"]:
            y = self.norm(x, lw["norm1_g"]) @ lw["wqkv"].double().T
            q, k, v = (self.heads(y[:, i * d:(i + 1) * d]) for i in range(3))
            x = x + self.attend(q, k, v, 1.0, everything, lambda lo, hi: enc[:, lo:hi]) @ lw["wo"].double().T
            x = x + self.ffn(lw, self.norm(x, lw["norm2_g"]))
        states = self.norm(x, w["enc_final_g"])
        x = w["tok_emb"][tok].double()
        vis = (sub[None, :] <= sub[:, None]) & (tau[None, :] <= tau[:, None])
        far = torch.where(vis, (tau[:, None] - tau[None, :]) + (sub[:, None] - sub[None, :]), 0)
        bias = w["dec_rel_bias"].double()[self.bucket(far, 32)].permute(2, 0, 1)
        for lw in w["dec_layers"]:
            y = self.norm(x, lw["norm1_g"]) @ lw["wqkv"].double().T
            q, k, v = (self.heads(y[:, i * d:(i + 1) * d]) for i in range(3))
            x = x + self.attend(q, k, v, 1.0, lambda lo, hi: vis[lo:hi], lambda lo, hi: bias[:, lo:hi]) @ lw["wo"].double().T
            q = self.heads(self.norm(x, lw["norm3_g"]) @ lw["cq"].double().T)
            y = states @ lw["ckv"].double().T
            x = x + self.attend(q, self.heads(y[:, :d]), self.heads(y[:, d:]), 1.0, everything) @ lw["co"].double().T
            x = x + self.ffn(lw, self.norm(x, lw["norm2_g"]))
        return self.logits(x, w["dec_final_g"])

    def __call__(self, *a):
        return self.encdec(*a) if self.c["kind"] == "encdec" else self.decoder_only(*a)


@torch.no_grad()
def exact(case, seed):
    c = case
    ctx, force, target = _tokens(c, seed)
    model = _Exact(c, _weights(c, seed))
    B, S, V, steps = c["batch"], c["subs"], c["vocab"], c["steps"]
    ints = dict(device="cuda", dtype=torch.long)
    if c["use"] == "train":
        logits, terms, loss = [], [], []
        for b in range(B):
            sub = torch.tensor([i for i, s in enumerate(target[b]) for _ in s], **ints)
            tau = torch.tensor([i * c["delay"] + 1 + j for i, s in enumerate(target[b]) for j in range(len(s))], **ints)
            y = model(ctx[b], torch.tensor([t for s in target[b] for t in s], **ints), sub, tau)
            nxt = torch.tensor([t for s in target[b] for t in s[1:] + [-1]], **ints)
            nll = torch.where(nxt >= 0, torch.logsumexp(y, -1) - y.gather(1, nxt.clamp(min=0)[:, None])[:, 0], 0)
            logits.append(y)
            terms.append(nll.cpu().numpy())
            loss.append(float(nll.sum()))
        return {"logits": logits, "terms": terms, "loss": np.array(loss)}
    grid = [(i, t) for t in range(1, steps + 1) for i in _rows(c, t)]      # subsequence, step
    sub, tau = (torch.tensor([g[k] for g in grid], **ints) for k in (0, 1))
    at = {g: n for n, g in enumerate(grid)}
    tokens = np.full((steps, B, S), -1, dtype=np.int32)
    logits = [torch.full((B, S, V), math.nan, dtype=torch.float64, device="cuda") if c["use"] == "client" or t == steps else None
              for t in range(1, steps + 1)]
    for b in range(B):
        # what is fed: the forced tokens, or the most likely successors, which the pass then has to confirm
        fed = np.array([0 if t - 1 == i * c["delay"] else force[t - 2, b, i] if force is not None
                        else SHIFT * (t - 1 - i * c["delay"]) % V for i, t in grid])
        for _ in range(steps + 1):
            y = model(ctx[b], torch.as_tensor(fed, **ints), sub, tau)
            best = y.argmax(-1).cpu().numpy()
            if force is not None:
                break
            then = np.array([fed[n] if (i, t - 1) not in at else best[at[i, t - 1]] for n, (i, t) in enumerate(grid)])
            if np.array_equal(fed, then):
                break
            fed = then
        for n, (i, t) in enumerate(grid):
            if t - 1 - i * c["delay"] < c["tokens"]:
                tokens[t - 1, b, i] = force[t - 1, b, i] if force is not None else best[n]
            if logits[t - 1] is not None:
                logits[t - 1][b, i] = y[n]
    return {"tokens": tokens, "logits": logits} if c["use"] == "client" else {"tokens": tokens[-1], "logits": logits[-1]}
