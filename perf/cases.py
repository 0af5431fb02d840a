"""The work that a user of this library has it do, as measurable cases.

A case is a dict of plain values; `kind` says which entry points a pass takes:

  step    a layer on its own, token after token: moe_route_step, moe_expert_forward
  stack   tokens through a stack of layers: moe_stack_route_step, moe_expert_forward with pending outputs
  prompt  a batch of prompt tokens through a layer: moe_route_batch, moe_expert_forward_batch
  static  the experts of one token without a context: moe_expert_forward_static
  pack    one expert's weights into the streamed layout (a model being loaded): moe_pack_expert

Routers of trained models have peaked logits; here a token's experts are chosen first and its input carries a
multiple of their rows of the router matrix, far above the noise of the other logits.  Which experts a token takes
(and so whether something misses) is thereby set by the case and not by rounding, and outputs can be compared.
Weights are normal with standard deviation 0.02 or uniform codes of that spread, as in the other synthetic workloads.
"""
import ctypes as C
import math
import random

import numpy as np
import torch

import paper_2412_00099_amd as moe

DEV = "cuda:0"
STD = 0.02
LAMBDA = 0.5
PERTURB = 0.5
WEIGHT_BYTES = {"fp32": 4.0, "bf16": 2.0, "int8": 1.0, "int4": 0.5 + 2.0 / 128}
ACT = {"fp32": torch.float32, "bf16": torch.bfloat16}
MODES = {"prior": moe.MOE_ROUTE_CACHE_PRIOR, "max_rank": moe.MOE_ROUTE_MAX_RANK, "cumsum": moe.MOE_ROUTE_CUMSUM}


# ---- the cases -------------------------------------------------------------------------------------------
def listed():
    return [
        # The smallest step: one token through a small fp32 layer whose decision the caller waits for.  Launches, the
        # wait and the host's part are all there is.
        dict(name="step_fp32_small", kind="step", hidden=256, experts=16, inter=512, shared=0, topk=2, capacity=8,
             weight="fp32", act="fp32", tokens=1, wait=True, cold=0, mode="prior", top_j=0, renorm=False),
        # Decode of the headline workload's layers (Qwen1.5-MoE-shaped, a large shared expert), four tokens.
        dict(name="stack_bf16_shared", kind="stack", layers=3, hidden=2048, experts=60, inter=1408, shared=5632, topk=4,
             capacity=30, weight="bf16", act="bf16", tokens=4, mode="prior", top_j=0, renorm=False),
        # Decode of OLMoE-shaped layers: many small experts, none shared.
        dict(name="stack_bf16_top8", kind="stack", layers=3, hidden=2048, experts=64, inter=1024, shared=0, topk=8,
             capacity=32, weight="bf16", act="bf16", tokens=4, mode="prior", top_j=0, renorm=False),
        # Decode of DeepSeek-V2-Lite-shaped layers with 4-bit weights: little to stream, latency counts.
        dict(name="stack_int4", kind="stack", layers=3, hidden=2048, experts=64, inter=1408, shared=2816, topk=6,
             capacity=32, weight="int4", act="bf16", tokens=4, mode="prior", top_j=0, renorm=False),
        # Decode of one Mixtral-shaped layer with 8-bit weights: the widest hidden size and the largest experts.
        dict(name="step_int8_wide", kind="step", hidden=4096, experts=8, inter=14336, shared=0, topk=2, capacity=4,
             weight="int8", act="bf16", tokens=4, wait=False, cold=0, mode="prior", top_j=0, renorm=True),
        # Decode with plain LRU routing on a small cache: two of a token's eight experts are filled over the host link.
        dict(name="step_bf16_misses", kind="step", hidden=2048, experts=64, inter=1024, shared=0, topk=8, capacity=16,
             weight="bf16", act="bf16", tokens=6, wait=False, cold=2, mode="prior", top_j=0, renorm=False),
        # Prompt phase of the headline layer: a short prompt, and a full batch.
        dict(name="prompt_8", kind="prompt", hidden=2048, experts=60, inter=1408, shared=5632, topk=4, capacity=30,
             weight="bf16", act="bf16", tokens=8, working=8, mode="prior", top_j=0, renorm=False),
        dict(name="prompt_128", kind="prompt", hidden=2048, experts=60, inter=1408, shared=5632, topk=4, capacity=30,
             weight="bf16", act="bf16", tokens=128, working=19, mode="prior", top_j=0, renorm=False),
        # A ragged prompt on the OLMoE-shaped layer: more experts per token, few tokens per expert.
        dict(name="prompt_37_top8", kind="prompt", hidden=2048, experts=64, inter=1024, shared=0, topk=8, capacity=32,
             weight="bf16", act="bf16", tokens=37, working=26, mode="prior", top_j=0, renorm=False),
        # The entry point for graph capture and loops that may not allocate, with 8-bit weights of a ragged size.
        dict(name="static_int8", kind="static", hidden=2048, inter=1000, shared=0, topk=6, slots=12, weight="int8",
             act="bf16"),
        # Loading a model: one expert into the streamed layout, in the plain and the most packed format.
        dict(name="pack_bf16", kind="pack", hidden=2048, inter=1408, weight="bf16"),
        dict(name="pack_int4", kind="pack", hidden=2048, inter=1408, weight="int4"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _expert_bytes(c, inter):
    return 3 * c["hidden"] * inter * WEIGHT_BYTES[c["weight"]]


def draw(rng):
    """One more case of the ranges above: sizes over their logarithm, every weight format, ragged sizes, the routing
    modes and options, bounded by the largest listed cases (0.35 GB of weights per token and layer)."""
    kind = rng.choice(["step", "step", "stack", "stack", "prompt", "prompt", "prompt", "static", "pack"])
    c = dict(kind=kind)
    if kind == "prompt":
        c.update(weight="bf16", act="bf16", hidden=rng.choice([1024, 2048, 2048]))
    else:
        c["weight"] = rng.choice(["fp32", "bf16", "bf16", "int8", "int4"])
        c["hidden"] = rng.choice({"fp32": [256, 512, 1024, 2048], "bf16": [512, 1024, 2048, 4096],
                                  "int8": [1024, 2048, 4096], "int4": [2048, 4096]}[c["weight"]])
    step = {"fp32": 1, "bf16": 1, "int8": 8, "int4": 128}[c["weight"]] if kind != "prompt" else 16

    def inter(lo, hi):
        return max(step, _log_int(rng, lo, hi) // step * step)

    c["inter"] = inter(128, 4096)
    if kind == "pack":
        return c
    if kind != "prompt":
        c["act"] = "fp32" if rng.random() < (0.7 if c["weight"] == "fp32" else 0.2) else "bf16"
    c["topk"] = rng.randint(1, 8)
    c["shared"] = inter(128, 6000) if rng.random() < 0.5 else 0
    if kind == "static":
        c["slots"] = rng.randint(c["topk"], 24)
    else:
        c["experts"] = rng.randint(max(8, c["topk"]), 64)
        c["capacity"] = rng.randint(c["topk"], c["experts"])
        c["mode"] = rng.choice(["prior", "prior", "prior", "max_rank", "cumsum"])
        c["top_j"] = rng.choice([0, 0, min(2, c["topk"])])
        c["renorm"] = rng.random() < 0.3
    if kind == "step":
        c.update(tokens=rng.randint(1, 6), wait=rng.random() < 0.3, cold=0)
    elif kind == "stack":
        c.update(layers=rng.randint(1, 4), tokens=rng.randint(1, 4))
    elif kind == "prompt":
        c["tokens"] = _log_int(rng, 1, 128)
        c["working"] = rng.randint(c["topk"], c["capacity"])
    # no larger than the listed cases: weights per token, a prompt's weights, and the two tiers in memory
    while (c["topk"] * _expert_bytes(c, c["inter"]) + _expert_bytes(c, c["shared"]) > 3.5e8
           or c.get("working", 0) * _expert_bytes(c, c["inter"]) > 3.5e8
           or c.get("layers", 1) * c.get("experts", c.get("slots", 1)) * _expert_bytes(c, c["inter"]) > 3.0e9):
        c["inter"] = max(step, c["inter"] // 2 // step * step)
        c["shared"] = c["shared"] // 2 // step * step
    if kind in ("step", "stack"):
        while c["tokens"] > 1 and work(c)["bytes"] > 1.4e9:
            c["tokens"] -= 1
    return c


# ---- inputs (made from the seed alone) -----------------------------------------------------------------------
def _gen(seed, *ids):
    key = random.Random("/".join(str(v) for v in (seed,) + ids)).getrandbits(62)
    return torch.Generator(device=DEV).manual_seed(key)


def _expert(c, seed, inter, *ids):
    """Canonical weights of one SwiGLU expert: gate, up [inter, d], down [d, inter], quantised as (codes, scales)."""
    g, d, fmt = _gen(seed, "expert", *ids), c["hidden"], c["weight"]

    def matrix(rows, cols):
        if fmt == "fp32":
            return torch.randn(rows, cols, generator=g, device=DEV) * STD
        if fmt == "bf16":
            return (torch.randn(rows, cols, generator=g, device=DEV, dtype=torch.bfloat16) * STD)
        if fmt == "int8":
            q = torch.randint(-127, 128, (rows, cols), generator=g, device=DEV, dtype=torch.int8)
            s = (0.8 + 0.4 * torch.rand(rows, generator=g, device=DEV)) * (STD / 73.3)
            return q, s.half()
        q = torch.randint(1, 16, (rows, cols), generator=g, device=DEV, dtype=torch.uint8)
        s = (0.8 + 0.4 * torch.rand(rows, cols // 128, generator=g, device=DEV)) * (STD / 4.32)
        return q[:, 0::2] | (q[:, 1::2] << 4), s.half()

    return dict(gate=matrix(inter, d), up=matrix(inter, d), down=matrix(d, inter))


def _gate(c, seed, layer):
    w = torch.randn(c["experts"], c["hidden"], generator=_gen(seed, "gate", layer), device=DEV) * STD
    return w.to(ACT[c["act"]])


def _residents(c, seed, layer):
    ids = list(range(c["experts"]))
    random.Random("%d/residents/%d" % (seed, layer)).shuffle(ids)
    return ids


def _wanted(c, seed, layer):
    """Per token the experts it is made to select, the strongest first."""
    r, ids, K = random.Random("%d/wanted/%d" % (seed, layer)), _residents(c, seed, layer), c["topk"]
    if c.get("cold"):  # hot experts that every token takes, the others from a rotation longer than the cache
        hot, rest = ids[:K - c["cold"]], ids[K - c["cold"]:]
        return [hot + [rest[(t * c["cold"] + i) % len(rest)] for i in range(c["cold"])] for t in range(c["tokens"])]
    pool = ids[:c.get("working", c["capacity"])]
    # a few experts are popular, most are not
    weight = [1.0 / (1 + i) ** 0.5 for i in range(len(pool))]
    out = []
    for _ in range(c["tokens"]):
        score = sorted(range(len(pool)), key=lambda i: -math.log(max(r.random(), 1e-12)) / weight[i])
        out.append([pool[i] for i in score[:K]])
    return out


PEAK = 9.0  # wanted logits lie this many standard deviations of the others above them


def _lift(c, gate, wanted, strength):
    """[T, d]: what makes the tokens' logits peak at the wanted experts, by unequal amounts."""
    K = c["topk"]
    rows = torch.nn.functional.normalize(gate.float(), dim=1)[torch.tensor(wanted, device=DEV)]  # [T, K, d]
    scale = torch.tensor([1.0 + 0.2 * (1.0 - k / K) for k in range(K)], device=DEV)
    return strength * (rows * scale[None, :, None]).sum(1)


def _strengths(c):
    """Per layer of a stack: the residual stream grows, and a layer's own part has to stand out of what it carries."""
    out, r2 = [], 1.0
    for l in range(c["layers"]):
        if l > 0:
            r2 += PERTURB * PERTURB + 0.6  # this layer's noise, the previous layer's output
        out.append(PEAK * math.sqrt(r2) / (1.0 if l == 0 else PERTURB))
        r2 *= 1.0 + 1.2 * c["topk"] * PEAK * PEAK / c["hidden"]
    return out


def _inputs(c, seed):
    """step, prompt: x [T, d] in the activation type.  stack: a [T, L, d] fp32."""
    T, d = c["tokens"], c["hidden"]
    if c["kind"] != "stack":
        x = torch.randn(T, d, generator=_gen(seed, "x"), device=DEV)
        x = x + _lift(c, _gate(c, seed, 0), _wanted(c, seed, 0), PEAK)
        return x.to(ACT[c["act"]])
    a = torch.randn(T, c["layers"], d, generator=_gen(seed, "a"), device=DEV)
    for l, strength in enumerate(_strengths(c)):
        a[:, l] += _lift(c, _gate(c, seed, l), _wanted(c, seed, l), strength)
    return a


# ---- the program's side: what is kept between calls ------------------------------------------------------------
def _pack_args(c, w, blob):
    parts, scales = [], []
    for name in ("gate", "up", "down"):
        q, s = w[name] if isinstance(w[name], tuple) else (w[name], None)
        parts.append(q.contiguous())
        scales.append(None if s is None else s.contiguous())
    return dict(parts=parts, scales=scales, blob=blob)


def _pack(c, inter, p):
    ptr = lambda t: None if t is None else C.c_void_p(t.data_ptr())  # noqa: E731
    moe.moe_pack_expert(moe.WEIGHT_FMT[c["weight"]], c["hidden"], inter, *[ptr(t) for t in p["parts"]],
                        *[ptr(t) for t in p["scales"]], ptr(p["blob"]),
                        C.c_void_p(torch.cuda.current_stream().cuda_stream))


def prepare(case, seed):
    c = case
    if c["kind"] in ("pack", "static"):
        n_bytes = moe.moe_blob_bytes(moe.WEIGHT_FMT[c["weight"]], c["hidden"], c["inter"])
    if c["kind"] == "pack":
        blob = torch.zeros(n_bytes, dtype=torch.uint8, device=DEV)
        return dict(case=c, pack=_pack_args(c, _expert(c, seed, c["inter"], 0), blob))
    if c["kind"] == "static":
        pool = torch.zeros(c["slots"], n_bytes, dtype=torch.uint8, device=DEV)
        for s in range(c["slots"]):
            _pack(c, c["inter"], _pack_args(c, _expert(c, seed, c["inter"], s), pool[s]))
        shared = None
        if c["shared"]:
            n = moe.moe_blob_bytes(moe.WEIGHT_FMT[c["weight"]], c["hidden"], c["shared"])
            shared = torch.zeros(n, dtype=torch.uint8, device=DEV)
            _pack(c, c["shared"], _pack_args(c, _expert(c, seed, c["shared"], "shared"), shared))
        slots, weights, x = _static_inputs(c, seed)
        return dict(case=c, pool=pool, shared=shared, slots=slots, weights=weights, x=x, y=torch.zeros_like(x))

    L = c.get("layers", 1)
    store = moe.ExpertStore(n_layers=L, hidden=c["hidden"], n_experts=c["experts"], inter=c["inter"],
                            shared_inter=c["shared"], capacity=c["capacity"], weight_fmt=c["weight"], act_fmt=c["act"],
                            device=DEV)
    for l in range(L):
        store.put_gate(l, _gate(c, seed, l))
        for e in range(c["experts"]):
            store.put_expert(l, e, _expert(c, seed, c["inter"], l, e))
        if c["shared"]:
            store.put_shared(l, _expert(c, seed, c["shared"], l, "shared"))
    cold = c.get("cold", 0)
    n_initial = c["topk"] - cold if cold else c["capacity"]
    dec = moe.MoEDecoder(store, top_k=c["topk"], top_j=c["top_j"], lam=0.0 if cold else LAMBDA, renormalize=c["renorm"],
                         initial=[_residents(c, seed, l)[:n_initial] for l in range(L)], route_mode=MODES[c["mode"]],
                         max_rank=min(2 * c["topk"], c["experts"]), cumsum_p=0.7)
    T, d, act = c["tokens"], c["hidden"], ACT[c["act"]]
    s = dict(case=c, store=store, dec=dec, y=torch.zeros(T, d, dtype=act, device=DEV))
    if c["kind"] == "stack":
        s.update(a=_inputs(c, seed), h=torch.zeros(T, d, device=DEV), x=torch.zeros(d, dtype=act, device=DEV))
    else:
        s["x"] = _inputs(c, seed)
    return s


def _static_inputs(c, seed):
    r = random.Random("%d/static" % seed)
    raw = [r.uniform(0.2, 1.0) for _ in range(c["topk"])]
    x = torch.randn(c["hidden"], generator=_gen(seed, "x"), device=DEV).to(ACT[c["act"]])
    return r.sample(range(c["slots"]), c["topk"]), [float(np.float32(v / sum(raw))) for v in raw], x


# ---- one pass ----------------------------------------------------------------------------------------------------
_K = moe.MOE_MAX_TOPK
_RECORD = np.dtype([("sel_expert", np.int32, _K), ("sel_slot", np.int32, _K), ("sel_weight", np.float32, _K),
                    ("rest", np.uint8, C.sizeof(moe.moe_route_out_t) - 12 * _K)])


def run(state):
    s, c = state, state["case"]
    if c["kind"] == "pack":
        _pack(c, c["inter"], s["pack"])
        return s["pack"]["blob"]
    if c["kind"] == "static":
        ptr = lambda t: None if t is None else C.c_void_p(t.data_ptr())  # noqa: E731
        moe.moe_expert_forward_static(moe.WEIGHT_FMT[c["weight"]], moe.ACT_FMT[c["act"]], c["hidden"], c["inter"],
                                      c["shared"], c["topk"], ptr(s["pool"]), c["slots"], ptr(s["shared"]), s["slots"],
                                      s["weights"], ptr(s["x"]), ptr(s["y"]),
                                      C.c_void_p(torch.cuda.current_stream().cuda_stream))
        return s["y"]
    dec = s["dec"]
    if c["kind"] == "step":
        sel = []
        for t in range(c["tokens"]):
            out = dec.route_step(0, x=s["x"][t], wait=c["wait"])
            dec.expert_forward(0, s["x"][t], s["y"][t])
            if c["wait"]:
                sel.append(out.sel_expert[:c["topk"]])
        return dict(y=s["y"], sel=np.array(sel, np.int32)) if c["wait"] else s["y"]
    if c["kind"] == "stack":
        last = c["layers"] - 1
        for t in range(c["tokens"]):
            for l in range(last + 1):
                dec.stack_route_step(l, s["h"][t], s["a"][t, l], 1.0 if l == 0 else PERTURB, s["x"], carry=l > 0, wait=False)
                dec.expert_forward(l, s["x"], s["y"][t] if l == last else None)
        return dict(y=s["y"], h=s["h"])
    records = dec.route_batch(0, x=s["x"])
    dec.expert_forward_batch(0, s["x"], s["y"])
    rec = np.frombuffer(records[0]._b_base_, _RECORD)
    return dict(y=s["y"], sel=rec["sel_expert"][:, :c["topk"]], weight=rec["sel_weight"][:, :c["topk"]])


# ---- what a pass cannot do without -----------------------------------------------------------------------------
def work(case):
    """Decode steps follow one another, so each reads the weights of its own experts; a batch reads an expert once.
    Filled experts count as written and as read again."""
    c = case
    one, shared = _expert_bytes(c, c["inter"]), _expert_bytes(c, c.get("shared", 0))
    if c["kind"] == "pack":
        return dict(bytes=2 * one, flops=0)
    act = ACT[c["act"]].itemsize
    d, macs = c["hidden"], 3 * c["hidden"]
    if c["kind"] == "static":
        return dict(bytes=c["topk"] * one + shared + 2 * d * act, flops=2 * macs * (c["topk"] * c["inter"] + c["shared"]))
    T, L = c["tokens"], c.get("layers", 1)
    gate = c["experts"] * d * act
    flops = 2 * T * L * (macs * (c["topk"] * c["inter"] + c["shared"]) + c["experts"] * d)
    if c["kind"] == "prompt":
        distinct = len({e for w in _wanted(c, 1, 0) for e in w})
        return dict(bytes=distinct * one + shared + gate + 2 * T * d * act, flops=flops)
    per_layer = c["topk"] * one + shared + gate + c.get("cold", 0) * one
    glue = 3 * L * d * 4 if c["kind"] == "stack" else d * act
    return dict(bytes=T * (L * per_layer + glue + d * act), flops=flops)


def tolerance(case):
    """Weights, sums and probabilities are 32-bit: with 32-bit activations only the order of the sums differs.  bf16
    outputs are rounded once (2^-9 of a value at most); in a stack a rounding that falls the other way in one layer
    travels through the following ones.  About four times the distance to `exact` as measured."""
    c = case
    if c["kind"] == "pack":
        return "exact"
    if c["act"] == "fp32":
        # (the quantised formats multiply by activations rounded to 16-bit floating point)
        return dict(rel=4e-6, max=4e-5) if c["weight"] in ("fp32", "bf16") else dict(rel=1.2e-3, max=1.2e-2)
    if c["kind"] == "stack":
        return dict(rel=1.5e-2, max=0.12)
    return dict(rel=7e-3, max=6e-2, differ=0.005)


# ---- the same in 64 bits -----------------------------------------------------------------------------------------
def _dense(w):
    if not isinstance(w, tuple):
        return w.double()
    q, s = w
    if q.dtype == torch.int8:
        return q.double() * s.double()[:, None]
    n = torch.stack((q & 15, q >> 4), 2).reshape(q.shape[0], -1).double() - 8.0
    return n * s.double().repeat_interleave(128, 1)


def _swiglu(w, x):
    """x [n, d] -> [n, d]"""
    g = x @ _dense(w["gate"]).t()
    u = x @ _dense(w["up"]).t()
    return (torch.nn.functional.silu(g) * u) @ _dense(w["down"]).t()


def _layer(c, seed, layer, x):
    """One layer on x [T, d]: outputs, the experts each token takes (strongest first), their weights."""
    p = torch.softmax(x @ _gate(c, seed, layer).double().t(), 1)
    w, sel = p.topk(c["topk"], 1)
    if c["renorm"]:
        w = w / w.sum(1, keepdim=True)
    y = torch.zeros_like(x)
    for e in sel.unique().tolist():
        t, k = (sel == e).nonzero(as_tuple=True)
        y[t] += w[t, k, None] * _swiglu(_expert(c, seed, c["inter"], layer, e), x[t])
    if c["shared"]:
        y += _swiglu(_expert(c, seed, c["shared"], layer, "shared"), x)
    return y, sel, w


def exact(case, seed):
    c = case
    if c["kind"] == "pack":
        return None
    if c["kind"] == "static":
        slots, weights, x = _static_inputs(c, seed)
        x = x.double()[None]
        y = sum(w * _swiglu(_expert(c, seed, c["inter"], s), x) for s, w in zip(slots, weights))
        if c["shared"]:
            y = y + _swiglu(_expert(c, seed, c["shared"], "shared"), x)
        return y[0]
    if c["kind"] == "stack":
        a = _inputs(c, seed).double()
        h = a[:, 0].clone()
        for l in range(c["layers"]):
            if l > 0:
                h = h + y + PERTURB * a[:, l]
            x = h / torch.sqrt((h * h).mean(1, keepdim=True) + 1e-6)
            y, _, _ = _layer(c, seed, l, x)
        return dict(y=y, h=h)
    y, sel, w = _layer(c, seed, 0, _inputs(c, seed).double())
    if c["kind"] == "prompt":
        # all of a token's experts are resident, so that the prior leaves them in the order of their logits
        return dict(y=y, sel=sel.int(), weight=w)
    return dict(y=y, sel=sel.int()) if c["wait"] else y
