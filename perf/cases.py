"""Performance cases of the linear-cross-entropy (LCE) library: what a training or scoring program has it do.

Each case is one pass through the torch entry points of ``paper_2605_21442_amd``: a loss and its
gradients, as one step of a recipe computes them for its vocabulary head. The widths and
vocabularies are those of the heads in ``workloads.py`` (512 x 4096, 2048 / 4096 / 8192 x 128256,
3584 x 152064); the token counts go from a 256-token step to a long-sequence batch of 32768 tokens,
with the micro-batches between (one to two sequences of 2048, gradient accumulation) and odd counts,
widths and vocabularies among them. Inputs follow the same recipe: H ~ N(0, 1) and W ~ N(0, sigma),
both bf16, Zipf targets, a share of the positions ignored as prompt tokens (spread, or a prefix of
every sequence).

The kinds of pass:

train     loss (mean or sum) and both gradients (full fine-tuning)
score     per-token losses, no gradient (log-probabilities of given text, evaluation)
pertoken  per-token losses and both gradients under a per-token upstream gradient (DPO / GRPO style)
hidden    loss and the gradient of the hidden states, the head frozen (LoRA fine-tuning)
accum     one micro-batch of several: dW added to the running gradient
adamw     loss, dH and an AdamW step on the head inside the backward (fp32 moments and master copy)
shard     one device's part of a vocabulary-parallel head: partials, combine, dH term and dW rows
kd        distillation of a teacher head into a student head: loss and the student's gradients
"""
from __future__ import annotations

import math

import torch

from paper_2605_21442_amd import AdamWState, autograd as A, linear_cross_entropy, linear_kd_loss

IGNORE = -100
SHARDS, SHARD = 8, 3           # the vocabulary-parallel cases: 8 devices, this one holds part 3
TEMPERATURE = 2.0              # distillation
OPT = dict(lr=1e-5, betas=(0.9, 0.95), eps=1e-8, weight_decay=0.1)
OPT_STEPS = 100                # updates the optimizer state has seen


def _case(name, kind, batch, seq, d, v, mask, prefix=False, reduction="mean", bits=64, dt=0):
    c = dict(kind=kind, batch=batch, seq=seq, d=d, v=v, mask=mask, prefix=prefix, reduction=reduction,
             target_bits=bits, dt=dt)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest training step: a small head and one short sequence; launches and latency
        _case("tiny", "train", 1, 256, 512, 4096, 0.10),
        # scoring one reply after its prompt with a 1B-class head: one short odd sequence, no gradient
        _case("score_1seq", "score", 1, 709, 2048, 128256, 0.30, prefix=True, reduction="none"),
        # per-token losses of a few sampled completions and their gradients (policy optimisation)
        _case("pertoken_3584", "pertoken", 4, 487, 3584, 152064, 0.30, prefix=True, reduction="none"),
        # full fine-tuning of a 1B-class model, the usual micro-batch of 2 x 2048
        _case("micro_1b", "train", 2, 2048, 2048, 128256, 0.25),
        # the benchmark batch: an 8B-class head, 8 x 2048 tokens
        _case("batch_8b", "train", 8, 2048, 4096, 128256, 0.25),
        # long sequences with prompt spans masked: the largest step
        _case("long_3584", "train", 4, 8192, 3584, 152064, 0.30, prefix=True),
        # a head whose width and vocabulary fit no tile (a pruned or custom model), summed loss, 32-bit labels
        _case("ragged_1000", "train", 1, 2999, 1000, 32003, 0.15, reduction="sum", bits=32),
        # one micro-batch of an accumulated step of an 8B-class model
        _case("accum_8b", "accum", 1, 2048, 4096, 128256, 0.25),
        # the optimizer step of the head inside the backward pass, a 1B-class micro-batch
        _case("adamw_1b", "adamw", 2, 2048, 2048, 128256, 0.25),
        # one of 8 devices of a vocabulary-parallel 70B-class head
        _case("shard_70b", "shard", 2, 2048, 8192, 128256, 0.20),
        # distilling an 8B-class head into a 1B-class head
        _case("kd_8b_to_1b", "kd", 2, 2048, 2048, 128256, 0.25, dt=4096),
        # LoRA fine-tuning of an 8B-class model: the head is frozen, only dH is wanted
        _case("frozen_8b", "hidden", 2, 2048, 4096, 128256, 0.25),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kinds = ["train", "train", "train", "score", "pertoken", "hidden", "accum", "adamw", "shard", "kd"]
    most = max(work(c)["flops"] for c in listed())
    while True:
        kind = rng.choice(kinds)
        n = int(_log_uniform(rng, 64, 32768))
        batch = rng.choice([1, 1, 2, 4])
        step = rng.choice([64, 64, 64, 8])          # widths: mostly whole 64s, some only multiples of 8
        d = max(256, int(_log_uniform(rng, 256, 8192)) // step * step)
        dt = max(256, int(_log_uniform(rng, 256, 8192)) // 64 * 64) if kind == "kd" else 0
        v = int(_log_uniform(rng, 4096, 152064))
        reduction = "none" if kind in ("score", "pertoken") else rng.choice(["mean", "mean", "sum"])
        c = _case("", kind, batch, max(1, n // batch), d, v, round(rng.uniform(0.0, 0.4), 3), rng.random() < 0.5,
                  reduction, rng.choice([64, 64, 32]), dt)
        if work(c)["flops"] <= 0.8 * most:
            return c


# ---- sizes ------------------------------------------------------------------------------------

def _span(c):
    return int(round(c["mask"] * c["seq"]))


def _valid(c):
    return c["batch"] * (c["seq"] - _span(c))       # both mask forms ignore the same number of positions


def _ids(c):
    """Ids of the vocabulary whose rows of W this device holds: (first, count)."""
    if c["kind"] != "shard":
        return 0, c["v"]
    v0, v1 = c["v"] * SHARD // SHARDS, c["v"] * (SHARD + 1) // SHARDS
    return v0, v1 - v0


def work(case):
    """The contractions of a pass, each over the valid tokens only: the logits (2 Nv D V), the logits again
    for the gradients (they are never held), dH and dW; and every input read and output written once."""
    c = case
    n, nv, d, dt = c["batch"] * c["seq"], _valid(c), c["d"], c["dt"]
    v = _ids(c)[1]
    unit = 2.0 * nv * d * v
    kind = c["kind"]
    h, w, t = 2 * n * d, 2 * v * d, n * c["target_bits"] // 8
    read = h + w + t
    if kind == "score":
        return {"bytes": read + 4 * n, "flops": unit}
    if kind == "hidden":
        return {"bytes": read + h, "flops": 3 * unit}
    if kind == "kd":
        return {"bytes": read + 2 * (n + v) * dt + h + w, "flops": 4 * unit + 2 * 2.0 * nv * dt * v}
    if kind == "accum":
        return {"bytes": read + h + 2 * w, "flops": 4 * unit}
    if kind == "adamw":
        return {"bytes": read + h + w + 24 * v * d, "flops": 4 * unit}   # m, v, master: fp32, read and written
    if kind == "shard":
        return {"bytes": read + 2 * h + w, "flops": 4 * unit}            # the dH term is fp32
    return {"bytes": read + h + w, "flops": 4 * unit}


def tolerance(case):
    # scoring: fp32 sums of exact bf16 products. Gradients: G rounded to bf16 once, sums in fp32, the result
    # in bf16; the measured error against 64 bits is about 2.6e-3, two such results differ by up to 1.4 times that
    if case["kind"] == "score":
        return {"rel": 1e-5}
    if case["kind"] == "adamw":         # the second moment holds the squared gradient: 5.4e-3 from 64 bits
        return {"rel": 2e-2}
    return {"rel": 1e-2}


# ---- inputs -----------------------------------------------------------------------------------

def _gen(seed, stream):
    return torch.Generator(device="cuda").manual_seed(seed * 64 + stream)


def _normal(shape, sigma, seed, stream, dtype=torch.bfloat16):
    x = torch.randn(shape, generator=_gen(seed, stream), device="cuda", dtype=torch.float32)
    return (x if sigma == 1.0 else x.mul_(sigma)).to(dtype)


def _sigma(d):
    return 0.015 if d >= 8192 else 0.02


def _targets(c, seed):
    """[batch, seq] ids by a truncated Zipf law P(k) ~ (k + 1)^-1.1, ignored positions at IGNORE."""
    b, s, v = c["batch"], c["seq"], c["v"]
    cdf = torch.cumsum(torch.arange(1, v + 1, device="cuda", dtype=torch.float64).pow(-1.1), 0)
    u = torch.rand((b, s), generator=_gen(seed, 2), device="cuda", dtype=torch.float64)
    t = torch.searchsorted(cdf, u * cdf[-1]).clamp_(max=v - 1)
    if c["prefix"]:
        t[:, :_span(c)] = IGNORE
    else:
        order = torch.rand((b * s,), generator=_gen(seed, 3), device="cuda").argsort()
        t.view(-1)[order[:b * _span(c)]] = IGNORE
    return t.to(torch.int64 if c["target_bits"] == 64 else torch.int32)


def _inputs(c, seed):
    """Hidden states [batch, seq, D], this device's rows of W, targets."""
    h = _normal((c["batch"], c["seq"], c["d"]), 1.0, seed, 0)
    w = _normal((_ids(c)[1], c["d"]), _sigma(c["d"]), seed, 1)
    return h, w, _targets(c, seed)


def _upstream(c, seed):
    """Upstream gradients of the per-token losses: advantage-like weights over the token count."""
    return _normal((c["batch"], c["seq"]), 1.0 / _valid(c) if _valid(c) else 1.0, seed, 4, torch.float32)


def _other_parts(c, seed):
    """[SHARDS, N] partials as an all-gather brings them: the other devices' log-sum-exps and target logits
    (this device's row is overwritten by each pass)."""
    n = c["batch"] * c["seq"]
    t = _targets(c, seed).reshape(-1)
    sd = _sigma(c["d"]) * math.sqrt(c["d"])
    lse = _normal((SHARDS, n), 0.01, seed, 5, torch.float32) + (math.log(c["v"] / SHARDS) + 0.5 * sd * sd)
    own = torch.arange(SHARDS, device="cuda").view(-1, 1) == torch.div(t.clamp(min=0) * SHARDS, c["v"], rounding_mode="floor")
    tgt = torch.where(own & (t >= 0), _normal((SHARDS, n), sd, seed, 6, torch.float32), 0.0)
    return torch.where(t >= 0, lse, 0.0).contiguous(), tgt.contiguous()


def _moments(c, seed):
    shape = (c["v"], c["d"])
    m = _normal(shape, 1e-5, seed, 7, torch.float32)
    v = torch.rand(shape, generator=_gen(seed, 8), device="cuda").add_(0.5).mul_(1e-10)
    off = _normal(shape, 1e-5, seed, 9, torch.float32)     # the master copy's offset from its rounding
    return m, v, off


def prepare(case, seed):
    c = case
    h, w, t = _inputs(c, seed)
    s = {"c": c, "h": h, "w": w, "t": t}
    kind = c["kind"]
    if kind in ("train", "pertoken", "hidden", "adamw", "kd"):
        h.requires_grad_(True)
    if kind in ("train", "pertoken", "kd"):
        w.requires_grad_(True)
    if kind == "pertoken":
        s["g"] = _upstream(c, seed)
    elif kind == "accum":
        s["g"] = torch.full((1,), 0.125, dtype=torch.float32, device="cuda")     # one of 8 micro-batches
        s["dw"] = _normal(tuple(w.shape), 1e-4, seed, 10)
    elif kind == "adamw":
        s["opt"] = AdamWState(w, master_weights=True, **OPT)
        m, v, off = _moments(c, seed)
        s["opt"].load_state_dict(dict(step=OPT_STEPS, exp_avg=m, exp_avg_sq=v, master=w.float() + off))
    elif kind == "shard":
        s["lse_parts"], s["tgt_parts"] = _other_parts(c, seed)
        s["g"] = torch.ones(1, dtype=torch.float32, device="cuda")
    elif kind == "kd":
        s["ht"] = _normal((c["batch"], c["seq"], c["dt"]), 1.0, seed, 11)
        s["wt"] = _normal((c["v"], c["dt"]), _sigma(c["dt"]), seed, 12)
    return s


def run(state):
    s, c = state, state["c"]
    h, w, t, kind, red = s["h"], s["w"], s["t"], c["kind"], c["reduction"]
    if kind == "train":
        loss = linear_cross_entropy(h, w, t, IGNORE, red)
        return (loss.detach(), *torch.autograd.grad(loss, (h, w)))
    if kind == "score":
        with torch.no_grad():
            return (linear_cross_entropy(h, w, t, IGNORE, red),)
    if kind == "pertoken":
        loss = linear_cross_entropy(h, w, t, IGNORE, red)
        return (loss.detach(), *torch.autograd.grad(loss, (h, w), s["g"]))
    if kind == "hidden":
        loss = linear_cross_entropy(h, w, t, IGNORE, red)
        return (loss.detach(), *torch.autograd.grad(loss, (h,)))
    if kind == "accum":
        loss, lse, nv, _, ws = A.forward(h, w, t, IGNORE, red, keep_workspace=True)
        dh, dw = A.backward(h, w, t, lse, nv, s["g"], IGNORE, red, accumulate_into=s["dw"], workspace=ws)
        return loss, dh, dw
    if kind == "adamw":
        opt = s["opt"]
        loss = linear_cross_entropy(h, w, t, IGNORE, red, optimizer=opt)
        dh, = torch.autograd.grad(loss, (h,))
        return loss.detach(), dh, w, opt.exp_avg, opt.exp_avg_sq, opt.master
    if kind == "shard":
        v0 = _ids(c)[0]
        lse_part, tgt_part, nv, _ = A.forward_shard(h, w, t, v0, c["v"], IGNORE)
        s["lse_parts"][SHARD].copy_(lse_part)
        s["tgt_parts"][SHARD].copy_(tgt_part)
        loss, lse, nv, _ = A.combine_shards(s["lse_parts"], s["tgt_parts"], t, c["v"], c["d"], IGNORE, red)
        dh, dw = A.backward_shard(h, w, t, lse, nv, s["g"], v0, c["v"], IGNORE, red)
        return lse_part, tgt_part, loss, lse, dh, dw
    loss = linear_kd_loss(h, w, s["ht"], s["wt"], t, TEMPERATURE, IGNORE, red)
    return (loss.detach(), *torch.autograd.grad(loss, (h, w)))


# ---- the same in 64 bits ------------------------------------------------------------------------

CHUNK = 8192                   # ids per block of logits


def _blocks(w):
    for v0 in range(0, w.shape[0], CHUNK):
        yield v0, w[v0:v0 + CHUNK].double()


def _lse(x, w, scale=1.0):
    out = torch.full((x.shape[0],), -math.inf, dtype=torch.float64, device=x.device)
    for _, wb in _blocks(w):
        out = torch.logaddexp(out, torch.logsumexp((x @ wb.T).mul_(scale), 1))
    return out


def _spread(rows, values, n):
    out = torch.zeros((n, *values.shape[1:]), dtype=torch.float64, device=values.device)
    out[rows] = values
    return out


def _reduce(terms, rows, n, red):
    if red == "none":
        return _spread(rows, terms, n)
    return terms.sum() if red == "sum" else terms.mean()


def exact(case, seed):
    c = case
    h3, w, t3 = _inputs(c, seed)
    n, d, kind, red = c["batch"] * c["seq"], c["d"], c["kind"], c["reduction"]
    t = t3.reshape(-1).long()
    rows = torch.nonzero(t != IGNORE).view(-1)
    if not len(rows):
        return None
    x, tv = h3.reshape(n, d)[rows].double(), t[rows]
    v0, v = _ids(c)
    own = (tv >= v0) & (tv < v0 + v)
    local = (tv - v0).clamp(0, v - 1)
    scale = 1.0 / TEMPERATURE if kind == "kd" else 1.0
    lse = _lse(x, w, scale)
    extra = []
    if kind == "kd":
        xt = _normal((c["batch"], c["seq"], c["dt"]), 1.0, seed, 11).reshape(n, -1)[rows].double()
        wt = _normal((c["v"], c["dt"]), _sigma(c["dt"]), seed, 12)
        lse_t = _lse(xt, wt, scale)
        terms = lse.clone()
    else:
        z = torch.where(own, (x * w[local].double()).sum(1), 0.0)
        if kind == "shard":
            lp, tp = (p.double() for p in _other_parts(c, seed))
            lp[SHARD], tp[SHARD] = _spread(rows, lse, n), _spread(rows, z, n)
            extra = [lp[SHARD].clone(), tp[SHARD].clone()]
            lse, z = torch.logsumexp(lp[:, rows], 0), tp[:, rows].sum(0)
        terms = lse - z
    if kind == "score":
        return (_reduce(terms, rows, n, red).view(t3.shape),)
    if kind == "pertoken":
        g = _upstream(c, seed).reshape(-1)[rows].double()
    else:
        g = torch.full((len(rows),), 0.125 if kind == "accum" else 1.0, dtype=torch.float64, device=x.device)
        g = g / len(rows) if red == "mean" else g
    dh = torch.zeros_like(x)
    dw = None if kind == "hidden" else torch.empty((v, d), dtype=torch.float64, device=x.device)
    for b0, wb in _blocks(w):
        zs = (x @ wb.T).mul_(scale)
        if kind == "kd":
            pt = ((xt @ wt[b0:b0 + CHUNK].double().T).mul_(scale) - lse_t[:, None]).exp_()
            terms -= (pt * zs).sum(1)
        zs.sub_(lse[:, None]).exp_()
        if kind == "kd":
            zs.sub_(pt)
        else:
            hit = torch.nonzero(own & (local >= b0) & (local < b0 + wb.shape[0])).view(-1)
            zs[hit, local[hit] - b0] -= 1.0
        zs.mul_((g * scale)[:, None])
        dh += zs @ wb
        if dw is not None:
            dw[b0:b0 + wb.shape[0]] = zs.T @ x
    loss = _reduce(terms, rows, n, red)
    loss = loss.view(t3.shape) if red == "none" else loss
    dh = _spread(rows, dh, n)
    if kind in ("accum", "shard"):
        if kind == "accum":
            dw += _normal((v, d), 1e-4, seed, 10).double()
        return (*extra, loss, *([_spread(rows, lse, n)] if kind == "shard" else []), dh, dw)
    dh = dh.view(h3.shape)
    if kind == "hidden":
        return loss, dh
    if kind != "adamw":
        return loss, dh, dw
    m, v2, off = (y.double() for y in _moments(c, seed))
    p = (w.float() + off.float()).double()
    b1, b2 = OPT["betas"]
    k = OPT_STEPS + 1
    m.mul_(b1).add_(dw, alpha=1 - b1)
    v2.mul_(b2).addcmul_(dw, dw, value=1 - b2)
    p.mul_(1 - OPT["lr"] * OPT["weight_decay"])
    p.addcdiv_(m, (v2 / (1 - b2 ** k)).sqrt_().add_(OPT["eps"]), value=-OPT["lr"] / (1 - b1 ** k))
    return loss, dh, p, m, v2, p
