"""The work whose time is measured: training and forward passes of the GPT,
FAL, FAL+ and parallel decoder stacks, and the AdamW update, each through a
public entry point of ``paper_2510_14614_amd.fal`` over the range of sizes
that the repository's configurations, tests and benchmark use.

A case is a dict of plain values.  ``kind`` names the entry point:

* ``model``   one training step of a whole language model (``model_step``):
              loss and every gradient;
* ``forward`` the forward pass of a whole language model (``model_forward``):
              loss and logits;
* ``block``   forward and backward of one block (``block_fwd``,
              ``block_bwd``), the last one of a two-block context;
* ``stack``   one training step of a block stack (``stack_step``): loss,
              input gradient and every parameter gradient;
* ``adamw``   one clipped AdamW update of a flat parameter buffer
              (``adamw_step_noalloc``).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2510_14614_amd import fal
from paper_2510_14614_amd.config import (ARCH_FAL, ARCH_FALPLUS, ARCH_GPT, ARCH_PARALLEL, SCHED_MERGED, SCHED_SEQ,
                                         SCHED_STREAMS, SCHED_STREAMS_MERGED, Config)

EPS = 1e-5  # LayerNorm epsilon of every case
F32, BF16 = 0, 1
HP = {"lr": 1e-4, "beta1": 0.9, "beta2": 0.999, "eps": 1e-8, "weight_decay": 1e-3, "max_grad_norm": 1.0}
OPT_STEP = 100  # an update in the middle of a run

BLOCK = ("ln1_g", "ln1_b", "w_qkv", "b_qkv", "w_o", "b_o", "ln2_g", "ln2_b", "w_fc", "b_fc", "w_2", "b_2", "lnF_g",
         "lnF_b")
GLOBAL = ("wte", "wpe", "lnf_g", "lnf_b")


def _case(name, kind, **kw):
    base = {"kind": kind, "L": 2, "H": 0, "kv": 0, "hd": 64, "V": 0, "B": 1, "arch": ARCH_FAL, "dtype": BF16,
            "sched": SCHED_STREAMS_MERGED, "tanh": 1, "bidir": 0, "first_block_standard": 0}
    base.update(kw)
    return {"name": name, **base} if name else base


def listed():
    return [
        # The smallest call: the tiny fp32 model that smoke tests and unit
        # tests train; its time is launches and latency.
        _case("tiny-fp32-step", "model", L=2, d=64, H=4, hd=16, f=256, V=256, T=32, B=2, dtype=F32, sched=SCHED_SEQ),
        # A small research model: narrow heads, a few thousand ids, a few
        # thousand tokens a step, the parallel block that FAL is compared to.
        _case("small-hd32-step", "model", L=4, d=256, H=8, hd=32, f=1024, V=8000, T=256, B=16, arch=ARCH_PARALLEL),
        # fp32 training of GPT-2-small-sized blocks on a few thousand tokens,
        # as a run that checks bf16 against fp32 does.
        _case("gpt2-small-fp32-stack", "stack", L=2, d=768, H=12, hd=64, f=3072, T=1024, B=2, dtype=F32),
        # Time to first token: the forward pass over one GPT-2-small prompt.
        _case("gpt2-small-prompt", "forward", L=12, d=768, H=12, hd=64, f=3072, V=50257, T=1024, B=1),
        # The whole GPT-2-small FAL training step at the benchmark's batch.
        _case("gpt2-small-step", "model", L=12, d=768, H=12, hd=64, f=3072, V=50257, T=1024, B=8),
        # FAL+ blocks at the GPT-2-medium shape (a GPT block and two FAL+ ones).
        _case("gpt2-medium-falplus-stack", "stack", L=3, d=1024, H=16, hd=64, f=4096, T=1024, B=8, arch=ARCH_FALPLUS,
              sched=SCHED_SEQ),
        # One FAL block of the ~1.3B shape: most of the flagship step is
        # twenty-three of these.
        _case("fal-block-1.3b", "block", d=2048, H=16, hd=128, f=8192, T=2048, B=4),
        # The baseline block at the same shape.
        _case("gpt-block-1.3b", "block", d=2048, H=16, hd=128, f=8192, T=2048, B=4, arch=ARCH_GPT, sched=SCHED_SEQ),
        # One GPU's tensor-parallel share of a ~7B stack: wide residual, few
        # heads, an FFN width that is no multiple of a tile.
        _case("7b-shard-stack", "stack", L=2, d=4096, H=8, hd=128, f=2752, T=2048, B=2),
        # Encoder blocks of the depth study: many short unmasked sequences,
        # key and value heads shared in two groups.
        _case("encoder-gqa-stack", "stack", L=2, d=1024, H=16, kv=2, hd=64, f=4096, T=128, B=128, bidir=1),
        # Ragged: lengths and widths that fit no tile, erf GELU, few tokens.
        _case("ragged-gpt-block", "block", d=1000, H=10, hd=64, f=2696, T=777, B=3, arch=ARCH_GPT, sched=SCHED_SEQ,
              tanh=0),
        # The optimizer on GPT-2 small's parameters (bf16 weights, fp32 state).
        _case("adamw-gpt2-small", "adamw", n=124439808, d=0, f=0, T=0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost(case):
    """Work on one scale, fp32 weighted by its lower matrix rate."""
    w = work(case)
    return max(w["flops"] * (16 if case["dtype"] == F32 else 1), w["bytes"] * 300)


def draw(rng):
    cap = {F32: _cost(listed()[2]), BF16: _cost(listed()[4])}
    while True:
        kind = rng.choice(("model", "forward", "block", "block", "stack", "stack", "adamw"))
        dtype = F32 if rng.random() < 0.25 else BF16
        if kind == "adamw":
            c = _case(None, kind, n=_log_int(rng, 1e4, 1.2e8), d=0, f=0, T=0, dtype=dtype)
        else:
            hd = rng.choice((16, 32, 64, 64, 128, 128))
            d = max(64, 8 * _log_int(rng, 8, 512))
            heads = max(1, round(d / hd * rng.choice((0.5, 1, 1, 1))))
            if (heads * hd) % 8:
                continue
            groups = [k for k in range(1, heads) if heads % k == 0 and (k * hd) % 8 == 0]
            arch = rng.choice((ARCH_GPT, ARCH_FAL, ARCH_FAL, ARCH_FALPLUS, ARCH_PARALLEL))
            whole = kind in ("model", "forward")
            c = _case(
                None, kind, L=2 if kind == "block" else rng.randint(1, 4), d=d, H=heads, hd=hd,
                kv=rng.choice(groups) if groups and rng.random() < 0.25 else 0,
                f=8 * _log_int(rng, max(4, d / 16), d / 2), V=_log_int(rng, 100, 50257) if whole else 0,
                T=_log_int(rng, 16, 2048), B=_log_int(rng, 1, 32), arch=arch, dtype=dtype,
                sched=rng.choice((SCHED_SEQ, SCHED_STREAMS, SCHED_MERGED, SCHED_STREAMS_MERGED)),
                tanh=1 if rng.random() < 0.75 else 0, bidir=1 if not whole and rng.random() < 0.25 else 0,
                first_block_standard=1 if arch == ARCH_FAL and rng.random() < 0.25 else 0)
            if whole and c["B"] * c["T"] > 16384:
                continue
            if hd * heads > 8192 or c["B"] * c["H"] * c["T"] ** 2 > 2.7e8:
                continue
        if _cost(c) <= cap[dtype]:
            return c


# ------------------------------------------------------------------ inputs --
def _whole(case):
    return case["kind"] in ("model", "forward")


def _config(case):
    return Config(n_layer=case["L"], d_model=case["d"], n_head=case["H"], head_dim=case["hd"], d_ff=case["f"],
                  vocab=case["V"], seq_len=case["T"], batch=case["B"], arch=case["arch"], dtype=case["dtype"],
                  sched=case["sched"], ln_eps=EPS, gelu_tanh=case["tanh"], has_embed_head=int(_whole(case)),
                  fal_block1_mode=case["first_block_standard"], bidirectional=case["bidir"], n_kv_head=case["kv"])


def _shapes(case):
    d, f, dA = case["d"], case["f"], case["H"] * case["hd"]
    qkv = dA + 2 * (case["kv"] or case["H"]) * case["hd"]
    vec = {"b_qkv": (qkv,), "b_fc": (f,)}
    mat = {"w_qkv": (d, qkv), "w_o": (dA, d), "w_fc": (d, f), "w_2": (f, d)}
    block = {k: mat.get(k) or vec.get(k) or (d,) for k in BLOCK}
    whole = {"wte": (case["V"], d), "wpe": (case["T"], d), "lnf_g": (d,), "lnf_b": (d,)} if _whole(case) else {}
    return whole, block


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == BF16 else torch.float32


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal(g, shape, scale, mean=0.0):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).mul_(scale).add_(mean)


def _weights(case, g):
    """Trained-like values in the storage dtype: matrices N(0, 0.02), gains
    around one, small shifts and biases."""
    dt = _dtype(case)
    whole, block = _shapes(case)

    def draw_one(name, shape):
        return (_normal(g, shape, 0.1, 1.0) if name.endswith("_g") else _normal(g, shape, 0.02)).to(dt)

    return ({k: draw_one(k, s) for k, s in whole.items()},
            [{k: draw_one(k, s) for k, s in block.items()} for _ in range(case["L"])])


def _inputs(case, seed):
    g = _gen(seed)
    whole, blocks = _weights(case, g)
    got = {"whole": whole, "blocks": blocks}
    M, d = case["B"] * case["T"], case["d"]
    if _whole(case):
        # Zipf(1.1) ids over the vocabulary, as text has them
        cdf = torch.arange(1, case["V"] + 1, device="cuda", dtype=torch.float64).pow_(-1.1).cumsum(0)
        u = torch.rand((case["B"], case["T"] + 1), generator=g, device="cuda", dtype=torch.float64)
        ids = torch.searchsorted(cdf, u * cdf[-1])
        got["tokens"] = ids.clamp_(max=case["V"] - 1).to(torch.int32).contiguous()
    else:
        got["x"] = _normal(g, (M, d), 1.0)
        # the upstream gradient of a sum over tokens, partly along the input
        # so that the stack's loss, sum(dy * X_L), does not cancel
        got["dy"] = (_normal(g, (M, d), 1.0) + 0.25 * got["x"]) / math.sqrt(M * d)
        if case["kind"] == "block":
            # the first block's attention output after its LayerNorm
            got["first"] = _normal(g, (M, d), 1.0).to(_dtype(case))
    return got


def _adamw_inputs(case, seed):
    g, n = _gen(seed), case["n"]
    w = _normal(g, (n,), 0.02)
    grads = _normal(g, (n,), 3.0 / math.sqrt(n))  # norm 3: the clip is active
    m = _normal(g, (n,), 0.3 / math.sqrt(n))
    v = m.square() + _normal(g, (n,), 1.0 / n).abs_()
    return w, grads, m, v


def prepare(case, seed):
    if case["kind"] == "adamw":
        w, grads, m, v = _adamw_inputs(case, seed)
        params = w.to(torch.bfloat16) if case["dtype"] == BF16 else None
        return {"case": case, "w": w, "params": params, "grads": grads, "m": m, "v": v, "hp": fal.adamw_params(**HP),
                "norm": torch.zeros(1, device="cuda")}
    got = _inputs(case, seed)
    F = fal.Fal(_config(case))
    lay = F.layout
    for k, name in enumerate(GLOBAL):
        if name in got["whole"]:
            a = got["whole"][name].reshape(-1)
            F.params[lay["global"][k]:lay["global"][k] + a.numel()].copy_(a)
    for i, blk in enumerate(got["blocks"]):
        base = lay["block_base"] + i * lay["block_stride"]
        for k, name in enumerate(BLOCK):
            a = blk[name].reshape(-1)
            F.params[base + lay["block"][k]:base + lay["block"][k] + a.numel()].copy_(a)
    st = {"case": case, "F": F, "tokens": got.get("tokens")}
    if case["kind"] == "forward":
        st["logits"] = torch.empty(case["B"] * case["T"], case["V"], device="cuda")
    if not _whole(case):
        st.update(x=got["x"], dy=got["dy"], dx=torch.empty_like(got["x"]), y=torch.empty_like(got["x"]),
                  first=got.get("first"), dfirst=torch.empty_like(got["x"]))
    return st


# -------------------------------------------------------------------- pass --
def _grads(case, F, layers):
    """Views of the flat gradient buffer, one a tensor name (all layers)."""
    lay, (whole, block) = F.layout, _shapes(case)
    out = {}
    for k, name in enumerate(GLOBAL):
        if name in whole:
            n = math.prod(whole[name])
            out[name] = F.grads[lay["global"][k]:lay["global"][k] + n].view(whole[name])
    L, stride = case["L"], lay["block_stride"]
    rows = F.grads[lay["block_base"]:lay["block_base"] + L * stride].view(L, stride)[layers]
    for k, name in enumerate(BLOCK):
        n = math.prod(block[name])
        out[name] = rows[:, lay["block"][k]:lay["block"][k] + n]
    return out


def run(state):
    case = state["case"]
    if case["kind"] == "adamw":
        s = state
        fal.adamw_step_noalloc(s["hp"], OPT_STEP, case["n"], case["dtype"], s["w"], s["params"], s["grads"], s["m"],
                               s["v"], s["norm"])
        return {"master": s["w"], "params": s["params"], "m": s["m"], "v": s["v"], "norm": s["norm"]}
    F = state["F"]
    if case["kind"] == "model":
        loss = F.model_step(state["tokens"])
        return {"loss": loss, **_grads(case, F, slice(None))}
    if case["kind"] == "forward":
        loss = F.model_forward(state["tokens"], state["logits"])
        return {"loss": loss, "logits": state["logits"]}
    if case["kind"] == "stack":
        loss = F.stack_step(state["x"], state["dy"], state["dx"])
        return {"loss": loss, "dx": state["dx"], **_grads(case, F, slice(None))}
    uses_first = case["arch"] in (ARCH_FAL, ARCH_FALPLUS)
    first, dfirst = (state["first"], state["dfirst"]) if uses_first else (None, None)
    F.block_fwd(1, state["x"], state["y"], first)
    F.block_bwd(1, state["x"], first, state["dy"], state["dx"], dfirst)
    return {"y": state["y"], "dx": state["dx"], "dfirst": dfirst, **_grads(case, F, slice(1, 2))}


# -------------------------------------------------------------------- work --
def work(case):
    """Matrix products of the pass (attention over the pairs that the mask
    leaves, a backward pass twice a forward one), each input read once and
    each output written once."""
    es = 2 if case["dtype"] == BF16 else 4
    if case["kind"] == "adamw":
        # gradient, weights and two moments in; weights, moments and the
        # bf16 copy out
        return {"bytes": case["n"] * (28 + (2 if case["dtype"] == BF16 else 0)), "flops": 15.0 * case["n"]}
    d, T, M = case["d"], case["T"], case["B"] * case["T"]
    whole, block = _shapes(case)
    dA = case["H"] * case["hd"]
    layers = 1 if case["kind"] == "block" else case["L"]
    weights = sum(math.prod(s) for k, s in block.items() if k.startswith("w_"))
    keys = T if case["bidir"] else (T + 1) / 2
    fwd = layers * (2.0 * M * weights + 4.0 * M * dA * keys) + 2.0 * M * d * case["V"]
    params = layers * sum(math.prod(s) for s in block.values()) + sum(math.prod(s) for s in whole.values())
    if case["kind"] == "forward":
        return {"bytes": es * params + 4 * M + 4.0 * M * case["V"], "flops": fwd}
    nbytes = (es + 4) * params
    if case["kind"] == "model":
        return {"bytes": nbytes + 4 * M, "flops": 3 * fwd}
    nbytes += 4 * M * d * 3  # x and dy in, dx out
    if case["kind"] == "block":
        nbytes += 4 * M * d  # y
        if case["arch"] in (ARCH_FAL, ARCH_FALPLUS):
            nbytes += (es + 4) * M * d  # the first-attention tensor and its gradient
    return {"bytes": nbytes, "flops": 3 * fwd}


def tolerance(case):
    """About four times the error measured against ``exact`` over the listed
    cases and forty drawn ones: fp32 sums 3.2e-6 (largest 2.2e-4); bf16
    operands and saved activations with fp32 accumulation 9.6e-3 for a stack
    (largest 0.1), 6.7e-3 for a block (0.2), 5.7e-3 for a model's gradients
    (0.1), 4.4e-3 for logits (0.03); the update 3.2e-8 (1.6e-7)."""
    if case["kind"] == "adamw":
        # a bf16 weight may round the other way (2^-8 of it) where the fp32
        # one is within its error of the middle
        return {"rel": 5e-5, "max": 8e-3} if case["dtype"] == BF16 else {"rel": 2e-7, "max": 2e-6}
    if case["dtype"] == F32:
        return {"rel": 1e-5, "max": 1e-3}
    rel, most = {"stack": (0.03, 0.4), "block": (0.025, 0.8), "model": (0.022, 0.4), "forward": (0.017, 0.12)}[case["kind"]]
    return {"rel": rel, "max": most}


# ------------------------------------------------------------------- exact --
def _ln(x, g, b):
    c = x - x.mean(-1, keepdim=True)
    return c / torch.sqrt((c * c).mean(-1, keepdim=True) + EPS) * g + b


def _norm(x):
    c = x - x.mean(-1, keepdim=True)
    return c / torch.sqrt((c * c).mean(-1, keepdim=True) + EPS)


def _mha(case, p, h):
    B, T, H, hd = case["B"], case["T"], case["H"], case["hd"]
    kv = case["kv"] or H
    q, k, v = (h @ p["w_qkv"] + p["b_qkv"]).split((H * hd, kv * hd, kv * hd), -1)
    q = q.view(B, T, H, hd).transpose(1, 2)
    k = k.view(B, T, kv, hd).transpose(1, 2).repeat_interleave(H // kv, 1)
    v = v.view(B, T, kv, hd).transpose(1, 2).repeat_interleave(H // kv, 1)
    rows = []
    for b in range(B):  # a sequence at a time: the score matrices are large
        s = (q[b] @ k[b].transpose(-1, -2)) / math.sqrt(hd)
        if not case["bidir"]:
            s = s.masked_fill(torch.ones(T, T, dtype=torch.bool, device=s.device).triu_(1), -math.inf)
        rows.append((s.softmax(-1) @ v[b]).transpose(0, 1).reshape(T, H * hd))
    return torch.cat(rows) @ p["w_o"] + p["b_o"]


def _mlp(case, p, h):
    u = h @ p["w_fc"] + p["b_fc"]
    if case["tanh"]:
        a = 0.5 * u * (1 + torch.tanh(math.sqrt(2 / math.pi) * (u + 0.044715 * u ** 3)))
    else:
        a = 0.5 * u * (1 + torch.erf(u / math.sqrt(2)))
    return a @ p["w_2"] + p["b_2"]


def _block(case, i, p, x, first):
    """Output of block i and the first-attention tensor (made by block 0)."""
    arch = case["arch"]
    a = _mha(case, p, _ln(x, p["ln1_g"], p["ln1_b"]))
    if arch == ARCH_FAL and i == 0:
        first = _ln(a, p["lnF_g"], p["lnF_b"])
    if arch == ARCH_FALPLUS and i == 0:
        first = _norm(a)
    if arch == ARCH_PARALLEL:
        return x + a + _mlp(case, p, _ln(x, p["ln2_g"], p["ln2_b"])), first
    if arch == ARCH_FAL and not (i == 0 and case["first_block_standard"]):
        return x + a + _mlp(case, p, _ln(x, p["ln2_g"], p["ln2_b"]) + first), first
    h = _ln(x + a, p["ln2_g"], p["ln2_b"])
    if arch == ARCH_FALPLUS and i > 0:
        h = h + first * p["lnF_g"] + p["lnF_b"]
    return x + a + _mlp(case, p, h), first


def _exact_adamw(case, seed):
    w, g, m, v = (t.double() for t in _adamw_inputs(case, seed))
    # the hyper-parameters as the call holds them, in 32 bits
    h = {k: float(np.float32(x)) for k, x in HP.items()}
    norm = g.norm()
    g = g * torch.clamp(h["max_grad_norm"] / (norm + 1e-6), max=1.0)
    m = h["beta1"] * m + (1 - h["beta1"]) * g
    v = h["beta2"] * v + (1 - h["beta2"]) * g * g
    c1, c2 = 1 - h["beta1"] ** OPT_STEP, 1 - h["beta2"] ** OPT_STEP
    w = w * (1 - h["lr"] * h["weight_decay"]) - h["lr"] / c1 * m / ((v / c2).sqrt() + h["eps"])
    return {"master": w, "params": w if case["dtype"] == BF16 else None, "m": m, "v": v, "norm": norm.reshape(1)}


def exact(case, seed):
    if case["kind"] == "adamw":
        return _exact_adamw(case, seed)
    got = _inputs(case, seed)
    train = case["kind"] != "forward"
    leaf = {k: t.double().requires_grad_(train) for k, t in got["whole"].items()}
    blocks = [{k: t.double().requires_grad_(train) for k, t in b.items()} for b in got["blocks"]]

    def grad_of(t):
        return torch.zeros_like(t) if t.grad is None else t.grad

    def grads(which):
        out = {k: grad_of(t) for k, t in leaf.items()}
        out.update({k: torch.stack([grad_of(b[k]).reshape(-1) for b in which]) for k in BLOCK})
        return out

    with torch.set_grad_enabled(train):
        if _whole(case):
            tok = got["tokens"].long()
            ids, targets = tok[:, :-1].reshape(-1), tok[:, 1:].reshape(-1)
            x, first = leaf["wte"][ids] + leaf["wpe"].repeat(case["B"], 1), None
            for i, p in enumerate(blocks):
                x, first = _block(case, i, p, x, first)
            logits = _ln(x, leaf["lnf_g"], leaf["lnf_b"]) @ leaf["wte"].t()
            loss = torch.nn.functional.cross_entropy(logits, targets)
            if not train:
                return {"loss": loss.reshape(1), "logits": logits}
            loss.backward()
            return {"loss": loss.detach().reshape(1), **grads(blocks)}
        x = got["x"].double().requires_grad_()
        dy = got["dy"].double()
        if case["kind"] == "stack":
            y, first = x, None
            for i, p in enumerate(blocks):
                y, first = _block(case, i, p, y, first)
            loss = (dy * y).sum()
            loss.backward()
            return {"loss": loss.detach().reshape(1), "dx": x.grad, **grads(blocks)}
        first = got["first"].double().requires_grad_()
        y, _ = _block(case, 1, blocks[1], x, first)
        (dy * y).sum().backward()
        uses_first = case["arch"] in (ARCH_FAL, ARCH_FALPLUS)
        return {"y": y.detach(), "dx": x.grad, "dfirst": grad_of(first) if uses_first else None, **grads(blocks[1:])}
