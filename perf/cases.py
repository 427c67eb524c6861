"""Layer calls to time: what a program that serves a mixture-of-experts model asks of this library.

A case is one MoE layer (or a few) of a model, the cache over its experts, and a pass of layer
calls through `MoeCache.layer_forward`: tokens decoded one at a time, verification windows of a
few tokens, or the tokens of a prompt in one call.  The expert store lies in pinned host memory,
the slots hold all of a layer's experts (`slots` = `experts`: every call after the first finds
its experts there) or fewer (the calls then copy what they miss).

Every layer call gets its own input instead of the previous layer's output, so that a change of
rounding shows in the call that makes it and does not travel.
"""
import math

import torch

from paper_2607_09686_amd import HostBuffer, MoeCache

# format: (bytes per block, weights per block); a mix names the formats of gate/up and of down
FORMATS = {"q8_0": (34, 32), "q4_0": (18, 32), "q4_k": (144, 256), "q6_k": (210, 256)}
MIXES = {"q4_k_m": ("q4_k", "q6_k")}
WEIGHT_SIGMA, ROUTER_SIGMA = 0.02, 0.05

DEFAULTS = {
    "kind": "decode",    # "decode": one token per call; "window": `tokens` per call; "prompt": one call
    "qtype": "q8_0", "hidden": 2048, "inter": 768, "experts": 128, "top_k": 8,
    "slots": 128,        # per layer; = experts: everything resident
    "layers": 1,
    "calls": 1,          # decode and window: calls per layer in a pass
    "tokens": 1,         # tokens per call
    "rho": 0.8,          # decode and window: correlation of consecutive tokens; prompt: share of the
                         #   tokens' standard deviation that the whole prompt has in common
    "norm": True,        # pre-norm input and residual output, as in a transformer's stack
    "static": False,     # decode through the entry point that allocates nothing
}


def _case(name, **kw):
    return dict(DEFAULTS, name=name, **kw)


def listed():
    return [
        # the smallest model of the tests, one token, one layer: nothing but launches and latency
        _case("decode_tiny", hidden=256, inter=128, experts=16, top_k=2, slots=4),
        # token generation of the 8-bit A3B-shaped stack with every expert in HBM (a GPU holds it)
        _case("decode_a3b_q8", layers=2, calls=8),
        # the same with the bench's budget of 19 of 128 slots: four misses per call over the host link
        _case("decode_a3b_q8_19slots", slots=19, calls=16),
        # token generation of the wider 4-bit stack, plain layer output without norm and residual
        _case("decode_q4_0", qtype="q4_0", hidden=2816, inter=1408, calls=8, norm=False),
        # token generation of the A3B shape in the 4-bit K-quant mix, from code that must not allocate
        _case("decode_a3b_q4km_static", qtype="q4_k_m", layers=2, calls=8, static=True),
        # speculative decoding's target pass, one token and four drafts: experts resident ...
        _case("window5_a3b_q8", kind="window", tokens=5, calls=4, layers=2),
        # ... and with the bench's 32 slots, the windows' misses over the host link
        _case("window5_a3b_q8_32slots", kind="window", tokens=5, calls=4, slots=32),
        # a short prompt (or a batch of decoding requests): few tokens for each of 128 experts
        _case("prompt_a3b_q8_61", kind="prompt", tokens=61, rho=0.3),
        # an ordinary prompt of an odd length in the wider 4-bit stack, its experts unevenly liked
        _case("prompt_q4_0_777", kind="prompt", qtype="q4_0", hidden=2816, inter=1408, tokens=777, rho=0.5),
        # long prompt chunks, experts resident: the bench's warm prefill, 8-bit and K-quant mix
        _case("prompt_a3b_q8_4096", kind="prompt", tokens=4096, rho=0.0),
        _case("prompt_a3b_q4km_4096", kind="prompt", qtype="q4_k_m", tokens=4096, rho=0.0, norm=False),
        # the bench's cold prefill: 45 slots, each call copies the experts that do not fit
        _case("prompt_a3b_q8_45slots", kind="prompt", tokens=4096, rho=0.0, slots=45),
    ]


def _payload(c):
    gu, dn = MIXES.get(c["qtype"], (c["qtype"], c["qtype"]))
    size = lambda f: c["hidden"] * c["inter"] // FORMATS[f][1] * FORMATS[f][0]
    return 2 * size(gu) + size(dn)


def draw(rng):
    """One more case: any kind, format and shape a model might have, up to the listed ones' cost."""
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    while True:
        kind = rng.choice(["decode", "decode", "window", "prompt", "prompt"])
        qtype = rng.choice(["q8_0", "q8_0", "q4_0", "q4_k_m", "q4_k_m", "q4_k", "q6_k"])
        k_quant = qtype in ("q4_k_m", "q4_k", "q6_k")
        step = 256 if k_quant else rng.choice([64, 128, 128, 256])
        hidden = max(256, log(512, 4096) // step * step)
        inter = max(step, log(256, 1536) // step * step)
        experts = rng.choice([16, 32, 60, 64, 128, 128])
        top_k = rng.choice([2, 4, 6, 8, 8])
        slots = experts if rng.random() < 0.6 else max(top_k, log(max(top_k, experts // 8), experts))
        tokens = {"decode": 1, "window": rng.randint(2, 8), "prompt": log(9, 4096)}[kind]
        c = dict(DEFAULTS, kind=kind, qtype=qtype, hidden=hidden, inter=inter, experts=experts, top_k=top_k,
                 slots=slots, calls={"decode": rng.randint(1, 8), "window": rng.randint(1, 4), "prompt": 1}[kind],
                 tokens=tokens, rho=round(rng.uniform(0.0, 0.6) if kind == "prompt" else rng.uniform(0.3, 0.9), 2),
                 norm=rng.random() < 0.6, static=kind == "decode" and rng.random() < 0.3)
        if (top_k * inter <= 12288 and experts * _payload(c) <= 900e6
                and 6.0 * tokens * top_k * hidden * inter <= 3.1e11):
            return c


# ---- inputs ----

def _u8(t):
    return t.contiguous().view(torch.uint8).reshape(*t.shape[:-1], -1)


def _half(x):
    return x.to(torch.float16)


def _encode(fmt, w):
    """Blocks [n, bytes per block] of the weights w [n, weights per block]."""
    if fmt == "q8_0":
        d = _half(w.abs().amax(1, keepdim=True) / 127)
        q = torch.round(w / d.float()).clamp(-127, 127).to(torch.int8)
        return torch.cat([_u8(d), _u8(q)], 1)
    if fmt == "q4_0":
        d = _half(w.abs().amax(1, keepdim=True) / 7)
        q = (torch.round(w / d.float()) + 8).clamp(0, 15).to(torch.uint8)
        return torch.cat([_u8(d), q[:, :16] | (q[:, 16:] << 4)], 1)
    n = w.shape[0]
    if fmt == "q4_k":
        w = w.view(n, 8, 32)
        low = (-w.amin(2)).clamp(min=0)
        step = (w.amax(2) + low) / 15
        d, dmin = _half(step.amax(1, keepdim=True) / 63), _half(low.amax(1, keepdim=True) / 63)
        sc = torch.round(step / d.float()).clamp(1, 63)
        m = torch.round(low / dmin.float()).clamp(0, 63)
        q = torch.round((w + (dmin.float() * m)[..., None]) / (d.float() * sc)[..., None]).clamp(0, 15).to(torch.uint8)
        sc, m = sc.to(torch.uint8), m.to(torch.uint8)
        scales = torch.cat([sc[:, :4] | ((sc[:, 4:] >> 4) << 6), m[:, :4] | ((m[:, 4:] >> 4) << 6),
                            (sc[:, 4:] & 15) | ((m[:, 4:] & 15) << 4)], 1)
        q = q.view(n, 4, 2, 32)
        return torch.cat([_u8(d), _u8(dmin), scales, (q[:, :, 0] | (q[:, :, 1] << 4)).reshape(n, 128)], 1)
    w = w.view(n, 16, 16)  # q6_k
    s = w.abs().amax(2) / 31
    d = _half(s.amax(1, keepdim=True) / 127)
    sc = torch.round(s / d.float()).clamp(1, 127)
    q = (torch.round(w / (d.float() * sc)[..., None]) + 32).clamp(0, 63).to(torch.uint8).view(n, 2, 4, 32)
    ql = (q[:, :, :2] & 15) | ((q[:, :, 2:] & 15) << 4)
    qh = (q[:, :, 0] >> 4) | ((q[:, :, 1] >> 4) << 2) | ((q[:, :, 2] >> 4) << 4) | ((q[:, :, 3] >> 4) << 6)
    return torch.cat([ql.reshape(n, 128), qh.reshape(n, 64), _u8(sc.to(torch.int8)), _u8(d)], 1)


def _decode(fmt, b):
    """The weights [n, weights per block] in 64 bits of the blocks b [n, bytes per block]."""
    n = b.shape[0]
    half = lambda lo: b[:, lo:lo + 2].contiguous().view(torch.float16).double()
    signed = lambda t: t.contiguous().view(torch.int8).double()
    if fmt == "q8_0":
        return half(0) * signed(b[:, 2:])
    if fmt == "q4_0":
        return half(0) * (torch.cat([b[:, 2:] & 15, b[:, 2:] >> 4], 1).double() - 8)
    if fmt == "q4_k":
        s = b[:, 4:16]
        sc = torch.cat([s[:, :4] & 63, (s[:, 8:] & 15) | ((s[:, :4] >> 6) << 4)], 1).double()
        m = torch.cat([s[:, 4:8] & 63, (s[:, 8:] >> 4) | ((s[:, 4:8] >> 6) << 4)], 1).double()
        q = b[:, 16:].reshape(n, 4, 1, 32)
        q = torch.cat([q & 15, q >> 4], 2).reshape(n, 8, 32).double()
        return ((half(0) * sc)[..., None] * q - (half(2) * m)[..., None]).reshape(n, 256)
    ql, qh = b[:, :128].reshape(n, 2, 2, 32), b[:, 128:192].reshape(n, 2, 1, 32)
    low = torch.cat([ql & 15, ql >> 4], 2)
    high = torch.cat([(qh >> s) & 3 for s in (0, 2, 4, 6)], 2)
    q = (low | (high << 4)).reshape(n, 16, 16).double() - 32
    return ((half(208) * signed(b[:, 192:208]))[..., None] * q).reshape(n, 256)


def _matrix(fmt, rows, cols, gen):
    w = torch.randn(rows * cols // FORMATS[fmt][1], FORMATS[fmt][1], device="cuda", generator=gen) * WEIGHT_SIGMA
    return _encode(fmt, w)


def _store(c, gen):
    """Expert payloads [layers * experts, payload bytes] on the GPU: gate, up, down."""
    gu, dn = MIXES.get(c["qtype"], (c["qtype"], c["qtype"]))
    H, I, E = c["hidden"], c["inter"], c["experts"]
    out = torch.empty(c["layers"] * E, _payload(c), dtype=torch.uint8, device="cuda")
    at = 0
    while at < out.shape[0]:
        n = min(16, out.shape[0] - at)
        both = _matrix(gu, n * 2 * I, H, gen).view(n, -1)
        out[at:at + n, :both.shape[1]] = both
        out[at:at + n, both.shape[1]:] = _matrix(dn, n * H, I, gen).view(n, -1)
        at += n
    return out


def _routes(c, x, w):
    """Per token: the chosen experts by descending logit, their weights, and the margin of the choice."""
    x = x.double()
    if c["norm"]:
        x = x / (x.square().mean(1, keepdim=True) + 1e-6).sqrt()
    z, ids = (x @ w.double()).sort(dim=1, descending=True, stable=True)
    k = c["top_k"]
    gap = z[:, k - 1] - z[:, k] if k < c["experts"] else torch.ones_like(z[:, 0])
    return x, ids[:, :k], torch.softmax(z[:, :k], 1), gap


def _tokens(c, w, gen):
    """Inputs [calls, layers, tokens, hidden].  A token whose choice of experts hangs on the rounding
    of a sum is drawn again: either choice would be right for it."""
    n, H = c["calls"] * c["tokens"], c["hidden"]
    noise = torch.randn(n, c["layers"], H, device="cuda", generator=gen)
    if c["kind"] == "prompt":
        common = torch.randn(1, c["layers"], H, device="cuda", generator=gen)
        x = c["rho"] * common + math.sqrt(1 - c["rho"] ** 2) * noise
    else:
        x = noise
        for t in range(1, n):
            x[t] = c["rho"] * x[t - 1] + math.sqrt(1 - c["rho"] ** 2) * noise[t]
    for l in range(c["layers"]):
        for _ in range(20):
            close = (_routes(c, x[:, l], w[l])[3] < 1e-4).nonzero()[:, 0]
            if not close.numel():
                break
            x[close, l] = torch.randn(close.numel(), H, device="cuda", generator=gen)
    return x.view(c["calls"], c["tokens"], c["layers"], H).transpose(1, 2).contiguous()


def _inputs(c, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    w = torch.randn(c["layers"], c["hidden"], c["experts"], device="cuda", generator=gen) * ROUTER_SIGMA
    return w, _tokens(c, w, gen), _store(c, gen)


def prepare(case, seed):
    c = dict(DEFAULTS, **case)
    w, x, dev = _inputs(c, seed)
    store = HostBuffer(dev.numel())
    torch.from_numpy(store.array).copy_(dev.view(-1))
    del dev
    cache = MoeCache(c["layers"], c["experts"], c["top_k"], c["hidden"], c["inter"], c["qtype"], store.ptr,
                     store.nbytes, c["slots"], stream=torch.cuda.current_stream(), residual=c["norm"],
                     prenorm=c["norm"])
    if c["slots"] == c["experts"]:  # a served model has long met all of its experts
        warm = torch.randn(max(64, 40 * c["experts"] // c["top_k"]), c["hidden"], device="cuda",
                           generator=torch.Generator(device="cuda").manual_seed(seed + 1))
        for l in range(c["layers"]):
            cache.layer_forward(warm, w[l], l, torch.empty_like(warm))
    y = torch.empty_like(x)
    calls = [(x[i, l], w[l], l, y[i, l]) for i in range(c["calls"]) for l in range(c["layers"])]
    return {"cache": cache, "store": store, "w": w, "x": x, "y": y, "calls": calls,
            "forward": cache.layer_forward_static if c["static"] else cache.layer_forward}


def run(state):
    forward = state["forward"]
    for x, w, layer, y in state["calls"]:
        forward(x, w, layer, y)
    return state["y"]


def work(case):
    """The chosen experts' weights (of a multi-token call: as many as tokens that choose evenly and
    independently meet), the router's, the inputs and the outputs; two operations per weight and token."""
    c = dict(DEFAULTS, **case)
    H, I, E, k, T = c["hidden"], c["inter"], c["experts"], c["top_k"], c["tokens"]
    n = c["calls"] * c["layers"]
    met = E * (1 - (1 - k / E) ** T)
    return {"bytes": n * (met * _payload(c) + 4.0 * H * E + 8.0 * T * H),
            "flops": n * T * (6.0 * k * H * I + 2.0 * H * E)}


def tolerance(case):
    """About four times what the path is off its value in 64 bits.  Calls of one token, and of up to
    eight with their experts resident, are accurate to 32 bits (3e-7 seen); larger ones round the
    weights to bfloat16 (3e-3 seen for the layer alone, 4e-4 to 8e-4 with the residual added), and so
    may a window whose experts do not fit the slots."""
    c = dict(DEFAULTS, **case)
    if c["tokens"] == 1 or (c["tokens"] <= 8 and c["slots"] == c["experts"]):
        return {"rel": 1.5e-6, "max": 3e-5}
    return {"rel": 3e-3, "max": 6e-2} if c["norm"] else {"rel": 1e-2, "max": 1e-1}


def exact(case, seed):
    c = dict(DEFAULTS, **case)
    gu, dn = MIXES.get(c["qtype"], (c["qtype"], c["qtype"]))
    H, I, E = c["hidden"], c["inter"], c["experts"]
    w, x, dev = _inputs(c, seed)
    gate_bytes = I * H // FORMATS[gu][1] * FORMATS[gu][0]
    y = torch.zeros(x.shape, dtype=torch.float64, device="cuda")
    for l in range(c["layers"]):
        tok = x[:, l].reshape(-1, H)
        xn, ids, p, _ = _routes(c, tok, w[l])
        out = tok.double() if c["norm"] else torch.zeros(tok.shape, dtype=torch.float64, device="cuda")
        for e in range(E):
            t, j = (ids == e).nonzero(as_tuple=True)
            if not t.numel():
                continue
            b = dev[l * E + e]
            both = _decode(gu, b[:2 * gate_bytes].view(-1, FORMATS[gu][0])).view(2, I, H)
            down = _decode(dn, b[2 * gate_bytes:].view(-1, FORMATS[dn][0])).view(H, I)
            a = xn[t]
            h = torch.nn.functional.silu(a @ both[0].t()) * (a @ both[1].t())
            out.index_add_(0, t, p[t, j][:, None] * (h @ down.t()))
        y[:, l] = out.view(c["calls"], c["tokens"], H)
    return y
