"""The workloads whose speed this framework is judged by, through its public entry points.

A case is a dict of plain values.  Its ``kind`` names the call a user's program makes:

* ``step``      one ``wino_step``: the forward over prompt, response and shadow
                block, the LM head's statistics and the draft / verify update
* ``decode``    a whole ``wino_decode`` from an all-mask response, then
                ``wino_row_losses`` of the decoded ids under the all-mask state
                (how a trajectory is scored)
* ``layers``    the first ``sublayers`` sublayers of the backbone
                (``wino_debug_forward``): an attention layer, or attention and MLP
* ``losses``    ``wino_row_losses`` of partly revealed training states
* ``epilogue``  the standalone decision from given bf16 logits

Weights are random with the distributions of the repository's presets: N(0, 0.02)
matrices, RMSNorm gains around one, an LM head of std 0.5/sqrt(d) and a Zipf bias,
on which a masked position's best id leads by a wide margin.
"""
from __future__ import annotations

import math

import torch

import paper_2605_16941_amd as P

DEV = "cuda"
TINY = dict(n_layers=2, d=256, hd=64, ff=704, vocab=4096, theta=10000.0)
LLADA = dict(d=4096, hd=128, ff=12288, vocab=126464, theta=500000.0)
MMADA = dict(LLADA, vocab=134656)  # the text vocabulary extended by 8192 image-code ids


def _case(name, kind, batch, prompt, gen, block, **kw):
    return dict(name=name, kind=kind, batch=batch, prompt=prompt, gen=gen, block=block, **kw)


def listed():
    return [
        # the smallest call: one step of the tiny model, bounded by launches and latency
        _case("tiny_step", "step", 1, 32, 64, 16, **TINY),
        # a whole decode of the tiny model: the host loop, its read-backs, every kernel at its smallest
        _case("tiny_decode", "decode", 4, 32, 64, 16, **TINY),
        # one decoder layer of the 8B model for a single user: 544 rows, weights streamed from memory
        _case("layer_bs1", "layers", 1, 256, 256, 32, sublayers=2, n_layers=1, **LLADA),
        # the same layer in a serving batch of 16: 8704 rows, bounded by the matrix cores
        _case("layer_bs16", "layers", 16, 256, 256, 32, sublayers=2, n_layers=1, **LLADA),
        # the attention half of a layer over the long image-and-text sequences: 4 x 2112 rows
        _case("attention_long", "layers", 4, 1024, 1024, 64, sublayers=1, n_layers=1, **MMADA),
        # fp16 activations, a ragged length: 4 x 361 rows
        _case("layer_fp16_ragged", "layers", 4, 201, 128, 32, sublayers=2, n_layers=1, fp16=True, **LLADA),
        # a model of about a billion parameters with 64-wide heads, odd prompt, short blocks
        _case("step_1b", "step", 3, 77, 120, 24, n_layers=4, d=2048, hd=64, ff=5632, vocab=32000, theta=10000.0),
        # the end of a step in a batch: a layer, the last layer's block rows, the LM head of 128 rows, the decision
        _case("step_bs4", "step", 4, 256, 256, 32, n_layers=2, **LLADA),
        # the whole 8B model for a single user, mid-block
        _case("step_8b_bs1", "step", 1, 256, 256, 32, n_layers=32, **LLADA),
        # training states of the trajectory-consistency objective: LM head over 1024 response rows
        _case("losses", "losses", 4, 128, 256, 32, n_layers=1, **LLADA),
        # the standalone decision on the logits of another engine
        _case("epilogue_b8", "epilogue", 8, 0, 32, 32, vocab=126464),
        # ... for one sequence with short blocks and a small vocabulary
        _case("epilogue_b1", "epilogue", 1, 0, 16, 16, vocab=32000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "layers", "layers", "layers", "losses", "decode", "epilogue"])
    if kind == "epilogue":
        block = rng.choice([8, 16, 24, 32, 48, 64])
        vocab = 8 * _log_int(rng, 500, 16900)
        batch = max(1, min(_log_int(rng, 1, 17), int(512 * 126464 / (2 * block * vocab))))
        return dict(kind=kind, batch=batch, prompt=0, gen=block, block=block, vocab=vocab)
    block = rng.choice([8, 12, 16, 24, 32, 48, 64])
    hd = rng.choice([64, 128])
    d = 256 * _log_int(rng, 1, 16)
    ff = 64 * max(4, int(round(d * rng.uniform(2.5, 3.2) / 64)))
    vocab = 256 * _log_int(rng, 16, 526 if d >= 2048 else 200)
    if kind == "decode":  # (small enough that a pass stays a few milliseconds)
        d, ff, vocab = min(d, 1024), min(ff, 3072), min(vocab, 32768)
    n_layers = 1 if kind in ("layers", "losses") else rng.choice([1, 2, 3])
    gen = block * rng.choice([2, 4, 6, 8])
    prompt = _log_int(rng, 16, 1024)
    rows = prompt + gen + block
    batch = max(1, min(_log_int(rng, 1, 17), 8704 // rows))
    if kind == "decode":
        gen, batch = block * 4, min(batch, 4)
    # no more than the largest listed case: 8704 rows of a 4096-wide layer
    while batch > 1 and n_layers * batch * rows * (4 * d * d + 3 * d * ff) > 8704 * 218e6:
        batch -= 1
    c = dict(kind=kind, batch=batch, prompt=prompt, gen=gen, block=block, n_layers=n_layers, d=d, hd=hd, ff=ff,
             vocab=vocab, theta=rng.choice([10000.0, 500000.0]))
    if kind == "layers":
        c["sublayers"] = rng.choice([1, 2, 2])
    if rng.random() < 0.25:
        c["fp16"] = True
    return c


class _Config:
    """Backbone fields as the package's model config takes them."""

    def __init__(self, c):
        self.n_layers, self.d_model, self.head_dim, self.d_ff = c["n_layers"], c["d"], c["hd"], c["ff"]
        self.n_heads, self.vocab = c["d"] // c["hd"], c["vocab"]
        self.rope_theta, self.rms_eps = c["theta"], 1e-5


def _mask_id(c):
    # the text vocabulary's last id
    return (LLADA["vocab"] if c["vocab"] > LLADA["vocab"] else c["vocab"]) - 1


def _weights(c, g):
    d, ff, v = c["d"], c["ff"], c["vocab"]

    def mat(*shape, std=0.02):
        return torch.randn(shape, dtype=torch.bfloat16, device=DEV, generator=g).mul_(std)

    def gain():
        return torch.randn(d, device=DEV, generator=g).mul_(0.1).add_(1.0).to(torch.bfloat16)

    rank = torch.empty(v, device=DEV, dtype=torch.float64)
    rank[torch.randperm(v, device=DEV, generator=g)] = torch.arange(1, v + 1, device=DEV, dtype=torch.float64)
    norm = torch.log(torch.sum(rank ** -1.1))
    return {
        "tok_emb": mat(v, d),
        "layers": [{"attn_norm": gain(), "w_qkv": mat(3 * d, d), "w_o": mat(d, d), "ffn_norm": gain(),
                    "w_gate_up": mat(2 * ff, d), "w_down": mat(d, ff)} for _ in range(c["n_layers"])],
        "final_norm": gain(),
        "lm_head": mat(v, d, std=0.5 / math.sqrt(d)),
        "lm_bias": (4.0 * (-1.1 * torch.log(rank) - norm)).float(),
    }


def _ids(c, g, shape):
    """Ids other than the mask."""
    x = torch.randint(0, c["vocab"] - 1, shape, device=DEV, generator=g)
    return (x + (x >= _mask_id(c))).to(torch.int32)


def prepare(case, seed):
    c = case
    g = torch.Generator(device=DEV).manual_seed(int(seed))
    s = {"kind": c["kind"], "case": c}
    b, lb, gen, prompt, mask = c["batch"], c["block"], c["gen"], c["prompt"], _mask_id(c)
    s["prm"] = P.make_params(b, prompt, gen, lb, mask, 0.7, 0.9)
    if c["kind"] == "epilogue":
        v = c["vocab"]
        logits = torch.randn(b, 2 * lb, v, dtype=torch.bfloat16, device=DEV, generator=g)
        peak = _ids(c, g, (b, 2 * lb, 1)).long()
        high = torch.rand(b, 2 * lb, 1, device=DEV, generator=g).mul_(6.0).add_(10.0)
        logits.scatter_(2, peak, high.to(torch.bfloat16))
        u = torch.rand(b, lb, device=DEV, generator=g)
        cur = torch.where(u < 0.75, peak[:, lb:, 0].to(torch.int32), _ids(c, g, (b, lb)))
        s.update(logits=logits, start=torch.where(u < 0.5, torch.full_like(cur, mask), cur))
        s.update(tokens=s["start"].clone(), bitmap=torch.empty(b, lb, dtype=torch.uint8, device=DEV),
                 flags=torch.empty(b, lb, dtype=torch.uint8, device=DEV),
                 stats=torch.empty(b, lb, 6, dtype=torch.int32, device=DEV),
                 ws=torch.empty(P.wino_epilogue_workspace_bytes(b, lb, v), dtype=torch.uint8, device=DEV))
        return s
    s["w"] = _weights(c, g)
    s["model"] = P.WinoModel(_Config(c), s["w"], b, prompt + gen + lb, P.ACT_FP16 if c.get("fp16") else P.ACT_BF16)
    resp = torch.full((b, gen), mask, dtype=torch.int32, device=DEV)
    n_blocks = gen // lb
    starts = [(lb * (i + n_blocks // 2)) % gen for i in range(b)]  # sequences are at different blocks
    if c["kind"] == "losses":
        seen = torch.rand(b, gen, device=DEV, generator=g) < 0.4
        s["targets"] = _ids(c, g, (b, gen))
        resp = torch.where(seen, s["targets"], resp)
    elif c["kind"] != "decode":
        # blocks before the current one are decoded, the current one partly
        at = torch.arange(gen, device=DEV)[None, :]
        st = torch.tensor(starts, device=DEV)[:, None]
        drafted = (at < st) | ((at < st + lb) & (torch.rand(b, gen, device=DEV, generator=g) < 0.4))
        resp = torch.where(drafted, _ids(c, g, (b, gen)), resp)
    s["start"] = torch.cat([_ids(c, g, (b, prompt)), resp], dim=1).contiguous()
    s["tokens"] = s["start"].clone()
    s["block_start"] = torch.tensor(starts, dtype=torch.int32, device=DEV)
    if c["kind"] == "layers":
        s["out"] = torch.empty(b, prompt + gen + lb, c["d"], device=DEV)
    else:
        s["loss"] = torch.empty(b, gen, 4, device=DEV)
        s["flags"] = torch.empty(b, lb, dtype=torch.uint8, device=DEV)
        s["n_masked"] = torch.empty(b, dtype=torch.int32, device=DEV)
        s["stats"] = torch.empty(b, lb, 6, dtype=torch.int32, device=DEV)
        s["final_step"] = torch.zeros(b, gen, dtype=torch.int32, device=DEV)
    return s


def _stats(s):
    f = s["stats"].view(torch.float32)
    return {"m_all": f[..., 0], "sumexp": f[..., 1], "z_best": f[..., 2], "z_target": f[..., 3],
            "argmax": s["stats"][..., 4], "row_kind": s["stats"][..., 5]}


def _losses(s):
    f = s["loss"]
    return {"entropy": f[..., 0], "nll": f[..., 1], "conf": f[..., 2], "argmax": f.view(torch.int32)[..., 3]}


def run(state):
    s = state
    kind = s["kind"]
    if kind == "layers":
        P.wino_debug_forward(s["model"].ctx, s["prm"], s["tokens"], s["block_start"], s["case"]["sublayers"], s["out"])
        return {"residual": s["out"]}
    if kind == "losses":
        P.wino_row_losses(s["model"].ctx, s["prm"], s["tokens"], s["targets"], s["loss"])
        return _losses(s)
    s["tokens"].copy_(s["start"])  # the caller's ids go into the buffer the call updates
    if kind == "epilogue":
        P.wino_epilogue(s["prm"], s["case"]["vocab"], s["logits"], s["tokens"], s["bitmap"], s["flags"], s["stats"], s["ws"])
        return dict(_stats(s), tokens=s["tokens"], flags=s["flags"], bitmap=s["bitmap"])
    if kind == "step":
        P.wino_step(s["model"].ctx, s["prm"], s["tokens"], s["block_start"], None, s["flags"], s["n_masked"], s["stats"])
        return dict(_stats(s), tokens=s["tokens"], flags=s["flags"], n_masked=s["n_masked"])
    s["block_start"].zero_()
    _, forwards = P.wino_decode(s["model"].ctx, s["prm"], s["tokens"], s["block_start"], s["final_step"])
    P.wino_row_losses(s["model"].ctx, s["prm"], s["start"], s["tokens"][:, s["case"]["prompt"]:].contiguous(), s["loss"])
    return dict(_losses(s), tokens=s["tokens"], final_step=s["final_step"], forwards=forwards)


def work(case):
    c = case
    b, lb, gen = c["batch"], c["block"], c["gen"]
    if c["kind"] == "epilogue":  # one row per position, the decision's outputs
        n = b * lb
        return {"bytes": n * (2.0 * c["vocab"] + 4 + 4 + 2 + 24), "flops": n * 3.0 * c["vocab"]}
    d, ff, v = c["d"], c["ff"], c["vocab"]

    def forward(shadow, sublayers, rows_out, compact):
        """(weight bytes, flops) of the backbone over every row, and of the LM head over rows_out; with compact the
        last layer computes only keys and values for every row."""
        S = c["prompt"] + gen
        t = S + (lb if shadow else 0)
        wb = fl = 0.0
        for i in range(sublayers):
            few = compact and i >= 2 * (c["n_layers"] - 1)
            m = b * (t - S + lb if few else t)
            if i % 2 == 0:
                pairs = (lb if few else S) * S + (t - S) * (t - 1)
                wb += 2.0 * 4 * d * d
                fl += 2.0 * d * d * (2 * b * t + 2 * m) + 4.0 * d * b * pairs
            else:
                wb += 2.0 * 3 * d * ff
                fl += 2.0 * m * 3 * d * ff
        if rows_out:
            wb += 2.0 * v * d
            fl += 2.0 * rows_out * v * d
        return wb, fl

    S, full = c["prompt"] + gen, 2 * c["n_layers"]
    if c["kind"] == "layers":
        rows = b * (S + lb)
        wb, fl = forward(True, c["sublayers"], 0, False)
        return {"bytes": wb + rows * d * (2.0 + 4.0), "flops": fl}
    if c["kind"] == "losses":
        wb, fl = forward(False, full, b * gen, False)
        return {"bytes": wb + b * S * (2.0 * d + 4) + b * gen * 20.0, "flops": fl}
    if c["kind"] == "step":
        wb, fl = forward(True, full, b * lb, True)
        return {"bytes": wb + b * S * (2.0 * d + 4) + b * lb * 30.0, "flops": fl}
    n = gen // lb  # each block drafts in one step, which has nothing to verify
    wb, fl = forward(False, full, b * lb, True)
    wl, ll = forward(False, full, b * gen, False)
    return {"bytes": n * (wb + b * S * (2.0 * d + 4)) + wl + b * gen * 20.0, "flops": n * fl + ll}


def tolerance(case):
    # epilogue: fp32 sums of exponentials over the vocabulary in another order.
    # The others: against 64 bits the bf16 path is off by 7e-3 on a layer's
    # residual stream and by up to 3e-3 on statistics and losses, the fp16 path
    # by 1e-3; another order or place of rounding moves results by as much.
    if case["kind"] == "epilogue":
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.01}
    if case.get("fp16"):
        return {"rel": 3e-3, "max": 0.05, "differ": 0.01}
    return {"rel": 1e-2, "max": 0.1, "differ": 0.01}


# ---------------------------------------------------------------- 64-bit reference
def _norm(x, gain):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + 1e-5) * gain.double()


def _forward(c, w, ids, pos, allowed, sublayers):
    """Residual stream [T, d] of one extended sequence after the first sublayers."""
    t, h, hd, d, ff = len(ids), c["d"] // c["hd"], c["hd"], c["d"], c["ff"]
    x = w["tok_emb"][ids.long()].double()
    inv = c["theta"] ** (-2.0 * torch.arange(hd // 2, dtype=torch.float64, device=DEV) / hd)
    ang = pos.double()[:, None] * inv
    cos, sin = ang.cos()[:, None], ang.sin()[:, None]

    def rope(a):
        a1, a2 = a[..., :hd // 2], a[..., hd // 2:]
        return torch.cat([a1 * cos - a2 * sin, a2 * cos + a1 * sin], -1)

    for i in range(sublayers):
        lw = w["layers"][i // 2]
        if i % 2 == 0:
            q, k, v = (_norm(x, lw["attn_norm"]) @ lw["w_qkv"].double().T).view(t, 3, h, hd).unbind(1)
            q, k = rope(q).transpose(0, 1).contiguous(), rope(k).permute(1, 2, 0).contiguous()
            z = (q @ k / math.sqrt(hd)).masked_fill_(~allowed, -math.inf).softmax(-1)
            x = x + (z @ v.transpose(0, 1).contiguous()).transpose(0, 1).reshape(t, d) @ lw["w_o"].double().T
        else:
            a = _norm(x, lw["ffn_norm"]) @ lw["w_gate_up"].double().T
            x = x + (torch.nn.functional.silu(a[:, :ff]) * a[:, ff:]) @ lw["w_down"].double().T
    return x


def _extended(c, ids, start):
    """Ids, positions and attention mask of prompt, response and shadow block."""
    S, lb = len(ids), c["block"]
    c0 = c["prompt"] + start
    ext = torch.cat([ids, torch.full((lb,), _mask_id(c), dtype=ids.dtype, device=DEV)])
    pos = torch.cat([torch.arange(S, device=DEV), c0 + torch.arange(lb, device=DEV)])
    allowed = torch.ones(S + lb, S + lb, dtype=torch.bool, device=DEV)
    allowed[:S, S:] = False
    j = torch.arange(lb, device=DEV)
    allowed[S + j, c0 + j] = False
    return ext, pos, allowed


def _logits(w, rows):
    return _norm(rows, w["final_norm"]) @ w["lm_head"].double().T + w["lm_bias"].double()


def exact(case, seed):
    c = case
    s = prepare(case, seed)
    lb, S, mask = c["block"], c["prompt"] + c["gen"], _mask_id(c)
    none = dict(z_target=None, argmax=None, row_kind=None, tokens=None, flags=None)

    def row_stats(z):
        m, best = z.max(-1).values, z.clone()
        best[..., mask] = -math.inf
        return {"m_all": m, "sumexp": (z - m[..., None]).exp().sum(-1), "z_best": best.max(-1).values}

    if c["kind"] == "epilogue":
        n = torch.arange(lb, device=DEV)
        rows = torch.where(s["start"] == mask, n, lb + n).long()
        z = torch.gather(s["logits"], 1, rows[..., None].expand(-1, -1, c["vocab"])).double()
        return dict(none, **row_stats(z), bitmap=None)
    s["model"].close()
    w, full = s["w"], 2 * c["n_layers"]
    starts = s["block_start"].tolist()
    if c["kind"] == "layers":
        return {"residual": torch.stack([_forward(c, w, *_extended(c, ids, st), c["sublayers"])
                                         for ids, st in zip(s["start"], starts)])}
    if c["kind"] == "step":
        got = []
        for ids, st in zip(s["start"], starts):
            x = _forward(c, w, *_extended(c, ids, st), full)
            c0 = c["prompt"] + st
            n = torch.arange(lb, device=DEV)
            got.append(row_stats(_logits(w, x[torch.where(ids[c0:c0 + lb] == mask, c0 + n, S + n)])))
        return dict(none, **{k: torch.stack([r[k] for r in got]) for k in got[0]}, n_masked=None)
    got = []
    for b, ids in enumerate(s["start"]):
        ones = torch.ones(S, S, dtype=torch.bool, device=DEV)
        x = _forward(c, w, ids, torch.arange(S, device=DEV), ones, full)
        lp = _logits(w, x[c["prompt"]:]).log_softmax(-1)
        p = lp.exp()
        r = {"entropy": -(p * lp).sum(-1), "conf": row_stats(lp)["z_best"].exp()}
        if c["kind"] == "losses":
            r["nll"] = -lp.gather(1, s["targets"][b].long()[:, None])[:, 0]
        got.append(r)
    out = {k: torch.stack([r[k] for r in got]) for k in got[0]}
    if c["kind"] == "losses":
        return dict(out, argmax=None)
    return dict(out, nll=None, argmax=None, tokens=None, final_step=None, forwards=None)
