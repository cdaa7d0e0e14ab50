"""The work whose speed this framework answers for, as cases that can be timed and compared.

A case is one call pattern of a program that uses the framework:

  prefill    the prompts of a batch through a stack of layers (K/V caches filled, hidden states out)
  decode     `steps` incremental steps of a batch whose K/V caches already hold the sequences
  encode     a batch through the layers as a bidirectional encoder (padding skipped, no sequence mask)
  generate   the model around a stack: prompt ids in, logits out, then `steps` tokens, each chosen outside the library

All tensors are fp16, as everywhere in the library.  Sequence lengths are part of a case (`len_lo` .. `len_hi`, spread over
the batch), so its work is known; weights, activations, caches and token ids come from the seed.
"""
from __future__ import annotations

import math

import torch

from paper_2104_12470_amd import eet

DEVICE = "cuda:0"
GPT2_VOCAB = 50257
_streams = {}


def _case(name, kind, hidden, heads, ffn, layers, batch, len_lo, len_hi, steps=0):
    return {"name": name, "kind": kind, "hidden": hidden, "heads": heads, "ffn": ffn, "layers": layers, "batch": batch,
            "len_lo": len_lo, "len_hi": len_hi, "steps": steps}


def listed():
    return [
        # a handful of short requests through one GPT-2-small layer: the smallest call, launches and latency
        _case("short prompts 768", "prefill", 768, 12, 3072, 1, 4, 16, 64),
        # one user of a GPT-2-medium-sized model: a short prompt, then token after token
        _case("one reply 24x1024", "generate", 1024, 16, 4096, 24, 1, 37, 37, 16),
        # a batch of prompts, and the tokens that follow, of a GPT-2-medium-sized stack
        _case("prompts 24x1024", "prefill", 1024, 16, 4096, 24, 8, 256, 512),
        _case("tokens 24x1024", "decode", 1024, 16, 4096, 24, 8, 384, 768, 16),
        # sentences of half the padded length through an encoder of the same size
        _case("sentences 24x1024", "encode", 1024, 16, 4096, 24, 16, 64, 192),
        # one layer of a 7B-sized model: a small batch of prompts, its tokens, and a server's batch of tokens
        _case("prompts 4096", "prefill", 4096, 32, 16384, 1, 4, 512, 1024),
        _case("tokens 4096", "decode", 4096, 32, 16384, 1, 4, 512, 1279, 16),
        _case("server tokens 4096", "decode", 4096, 32, 16384, 1, 48, 100, 1500, 16),
        # long documents
        _case("long prompts 2048", "prefill", 2048, 16, 8192, 1, 2, 2048, 4096),
        _case("long tokens 2048", "decode", 2048, 16, 8192, 1, 2, 2048, 4160, 16),
        # one layer of GPT-3's width, full batch: the largest work
        _case("prompts 12288", "prefill", 12288, 96, 49152, 1, 16, 1024, 2048),
        _case("tokens 12288", "decode", 12288, 96, 49152, 1, 16, 1024, 2104, 8),
    ]


def _log_between(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: widths of 256 to 12288 with heads of 64 or 128, 1 to 24 layers, batches of 1 to
    128, sequences of 1 to 4096 tokens; feed-forward widths of four times the layer's or of eight thirds of it."""
    largest = _flops(listed()[-2])
    while True:
        kind = rng.choice(["prefill", "prefill", "decode", "decode", "encode", "generate"])
        d = rng.choice([64, 128])
        heads = max(1, _log_between(rng, 256, 12288 if kind != "generate" else 2048) // d)
        hidden = heads * d
        ffn = 4 * hidden if rng.random() < 0.75 else max(64, int(hidden * 8 / 3) // 64 * 64)
        layers = _log_between(rng, 1, 24)
        batch = _log_between(rng, 1, 128)
        len_hi = _log_between(rng, 8, 4096)
        len_lo = max(1, int(len_hi * rng.choice([0.1, 0.25, 0.5, 0.75, 1.0])))
        steps = rng.randrange(4, 17) if kind in ("decode", "generate") else 0
        c = _case("", kind, hidden, heads, ffn, layers, batch, len_lo, len_hi, steps)
        del c["name"]
        params = layers * (4 * hidden * hidden + 2 * hidden * ffn)
        rows = batch * (len_hi if kind != "decode" else 16)
        cache = 2 * layers * batch * (len_hi + steps) * hidden
        if params > 1.9e9 or rows * (5 * hidden + ffn) > 3e9 or cache > 2e9 or rows > 65536:
            continue                              # a state stays a small part of the card
        if _flops(c) > largest or work(c)["bytes"] > 30e9:
            continue                              # no more work than the largest of the list
        return c


def _lens(c):
    """Lengths of the batch, spread over [len_lo, len_hi] without order; the longest is len_hi."""
    lo, hi, n = c["len_lo"], c["len_hi"], c["batch"]
    out = [lo + int((hi - lo + 1) * ((0.618034 * b + 0.3) % 1.0)) for b in range(n)]
    out[n // 2] = hi
    return out


def _params(c):
    H, F = c["hidden"], c["ffn"]
    return 4 * H * H + 2 * H * F


def _flops(c):
    H, L = c["hidden"], _lens(c)
    dense = 2.0 * _params(c) * c["layers"]
    head = 2.0 * GPT2_VOCAB * H * c["batch"]
    if c["kind"] == "decode":
        return sum(dense * c["batch"] + c["layers"] * sum(4.0 * H * (n + s + 1) for n in L) for s in range(c["steps"]))
    window = (lambda n: 4.0 * H * n * n) if c["kind"] == "encode" else (lambda n: 2.0 * H * n * (n + 1))
    total = dense * sum(L) + c["layers"] * sum(window(n) for n in L)
    if c["kind"] == "generate":
        total += head + sum(dense * c["batch"] + head + c["layers"] * sum(4.0 * H * (n + s + 1) for n in L) for s in range(c["steps"]))
    return total


def work(case):
    """Weights once per call, inputs and outputs once; a token's step reads the keys and values it sees and adds its own."""
    H, B, L, n = case["hidden"], case["batch"], _lens(case), case["layers"]
    weights = 2.0 * n * (_params(case) + 9 * H + case["ffn"])
    rows = sum(L)
    cached = lambda s: n * 4.0 * H * sum(m + s + 1 for m in L)          # noqa: E731
    if case["kind"] == "decode":
        nbytes = sum(weights + cached(s) + n * 4.0 * H * B + 4.0 * H * B for s in range(case["steps"]))
    elif case["kind"] == "generate":
        wte, out = 2.0 * GPT2_VOCAB * H, 2.0 * GPT2_VOCAB * B
        nbytes = weights + wte + out + n * 4.0 * H * rows + 4.0 * H * rows
        nbytes += sum(weights + wte + out + cached(s) for s in range(case["steps"]))
    else:
        nbytes = weights + 4.0 * H * rows + (n * 4.0 * H * rows if case["kind"] == "prefill" else 0.0)
    return {"bytes": nbytes, "flops": _flops(case)}


def tolerance(case):
    """fp16 with fp32 sums: each layer rounds its intermediates a few times, and the differences add up over the layers.
    Four times the distance from the same arithmetic in float64 (one layer: rel 3.1e-4 to 4.7e-4, max 1.1e-3 to 2.8e-3;
    24 layers: rel 1.4e-3 to 1.5e-3, max 5.2e-3 to 8.2e-3)."""
    return {"rel": 1.8e-3 + 1.8e-4 * case["layers"], "max": 0.01 + 1e-3 * case["layers"]}


def _stream():
    """The program's one working stream (a decode step of a stack is replayed as a graph, which the null stream does not allow)."""
    if "s" not in _streams:
        _streams["s"] = torch.cuda.Stream()
    return _streams["s"]


class _Draws:
    """Normal fp16 tensors from one seeded generator on the device."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEVICE)
        self.g.manual_seed(seed)

    def normal(self, shape, sigma=1.0, mean=0.0):
        return torch.empty(shape, dtype=torch.float16, device=DEVICE).normal_(mean, sigma, generator=self.g)

    def ids(self, shape):
        return torch.randint(0, GPT2_VOCAB, shape, dtype=torch.int32, device=DEVICE, generator=self.g)


def _layer_weights(r, c):
    H, F = c["hidden"], c["ffn"]
    s = 0.02 if H <= 4096 else 0.006
    return {"ln1_g": r.normal((H,), 0.1, 1.0), "ln1_b": r.normal((H,), 0.1), "w_qkv": r.normal((3 * H, H), s), "b_qkv": r.normal((3 * H,), s),
            "w_o": r.normal((H, H), s), "b_o": r.normal((H,), s), "ln2_g": r.normal((H,), 0.1, 1.0), "ln2_b": r.normal((H,), 0.1),
            "w_fc1": r.normal((F, H), s), "b_fc1": r.normal((F,), s), "w_fc2": r.normal((H, F), s), "b_fc2": r.normal((H,), s)}


def _inputs(c, seed):
    """Weights, activations, caches and token ids of a case, from the seed alone."""
    r = _Draws(seed)
    H, B, lens, steps = c["hidden"], c["batch"], _lens(c), c["steps"]
    prompt, room = _room(c)
    d = {"weights": [_layer_weights(r, c) for _ in range(c["layers"])]}
    if c["kind"] == "generate":
        d["head"] = {"wte": r.normal((GPT2_VOCAB, H), 0.02), "wpe": r.normal((room, H), 0.01), "lnf_g": r.normal((H,), 0.1, 1.0), "lnf_b": r.normal((H,), 0.1)}
        d["prompt"] = r.ids((B, prompt))
        d["next"] = r.ids((steps, B))
    elif c["kind"] == "decode":
        sigma = (0.02 if H <= 4096 else 0.006) * math.sqrt(H)          # what the K and V projections of normalised rows give
        d["kv"] = r.normal((c["layers"] * 2 * B * room * H,), sigma)
        d["x"] = r.normal((steps, B, H))
    else:
        d["x"] = r.normal((B, prompt, H))
    return d


def _room(c):
    """Padded prompt length and cache rows per sequence; a decode-only program never sees a prompt longer than a token, so
    its scratch stays small."""
    longest = max(_lens(c))
    return (1 if c["kind"] == "decode" else longest), longest + c["steps"]


def prepare(case, seed):
    c, d = case, _inputs(case, seed)
    prompt, room = _room(c)
    cfg = eet.make_config(c["hidden"], c["heads"], c["ffn"], c["batch"], prompt, room)
    s = {"kind": c["kind"], "lens": _lens(c), "steps": c["steps"], "stream": _stream(), "layers": c["layers"]}
    if c["kind"] == "generate":
        s["model"] = eet.DecoderModel(cfg, d["weights"], d["head"], GPT2_VOCAB, device=DEVICE)
        s["prompt"], s["next"] = d["prompt"], d["next"]
        return s
    # one layer on its own is a layer handle; several are a stack
    s["net"] = eet.DecoderLayer(cfg, d["weights"][0], device=DEVICE) if c["layers"] == 1 else eet.DecoderStack(cfg, d["weights"], device=DEVICE)
    s["x"] = d["x"]
    s["out"] = torch.empty_like(s["x"])
    if c["kind"] == "decode":
        s["net"].kv_cache.copy_(d["kv"])
        s["tok"], s["row"] = torch.empty_like(s["x"][0]), torch.empty_like(s["x"][0])
    return s


def _exact_layer(w, heads, x, kv, rows, causal):
    """One pre-LN layer in 64 bits.  x: the packed rows [T, H]; rows: per sequence its rows of x and its cached length before
    them; kv: [2, B, heads, room, d] to write keys and values into, or None (the rows see one another only)."""
    F = torch.nn.functional
    H = x.shape[1]
    d = H // heads
    g = lambda name: w[name].double()                                  # noqa: E731
    a = F.layer_norm(x, (H,), g("ln1_g"), g("ln1_b"), 1e-5)
    qkv = F.linear(a, g("w_qkv"), g("b_qkv"))
    ctx = torch.empty_like(x)
    for b, (r0, r1, n0) in enumerate(rows):
        q, k, v = (qkv[r0:r1, i * H:(i + 1) * H].view(r1 - r0, heads, d).transpose(0, 1).contiguous() for i in range(3))
        if kv is not None:
            kv[0, b, :, n0:n0 + r1 - r0] = k
            kv[1, b, :, n0:n0 + r1 - r0] = v
            k, v = (kv[i, b, :, :n0 + r1 - r0].contiguous() for i in range(2))
        seen = torch.ones((q.shape[1], k.shape[1]), dtype=torch.bool, device=x.device).tril(n0) if causal else None
        for h in range(0, heads, 16):
            s = torch.matmul(q[h:h + 16], k[h:h + 16].transpose(1, 2).contiguous()) / math.sqrt(d)
            if seen is not None:
                s.masked_fill_(~seen, -math.inf)
            o = torch.matmul(torch.softmax(s, -1), v[h:h + 16])
            ctx[r0:r1, h * d:(h + o.shape[0]) * d] = o.transpose(0, 1).reshape(r1 - r0, -1)
    y = x + F.linear(ctx, g("w_o"), g("b_o"))
    del qkv, ctx
    a = F.layer_norm(y, (H,), g("ln2_g"), g("ln2_b"), 1e-5)
    a = F.gelu(F.linear(a, g("w_fc1"), g("b_fc1")), approximate="tanh")
    return y + F.linear(a, g("w_fc2"), g("b_fc2"))


def exact(case, seed):
    """What run() returns for these inputs, by plain torch in 64 bits."""
    if _flops(case) > 1.5e14:
        return None
    c, d = case, _inputs(case, seed)
    H, B, heads, lens, n = c["hidden"], c["batch"], c["heads"], _lens(c), c["layers"]
    prompt, room = _room(c)
    kv = None
    if c["kind"] != "encode":
        kv = d["kv"].double() if c["kind"] == "decode" else torch.zeros(n * 2 * B * room * H, dtype=torch.float64, device=DEVICE)
        kv = kv.view(n, 2, B, heads, room, H // heads)

    def through(x, rows, causal=True):
        for i, w in enumerate(d["weights"]):
            x = _exact_layer(w, heads, x, None if kv is None else kv[i], rows, causal)
        return x

    def steps_of(inputs):
        return [through(x, [(b, b + 1, lens[b] + k) for b in range(B)]) for k, x in enumerate(inputs)]

    ends = [sum(lens[:b + 1]) for b in range(B)]
    packed = [(e - m, e, 0) for e, m in zip(ends, lens)]
    if c["kind"] == "generate":
        head = {k: v.double() for k, v in d["head"].items()}

        def logits(x):
            x = torch.nn.functional.layer_norm(x, (H,), head["lnf_g"], head["lnf_b"], 1e-5)
            return torch.nn.functional.pad(x @ head["wte"].T, (0, -GPT2_VOCAB % 64))     # columns up to the next multiple of 64 are zero rows of the table

        x = torch.cat([head["wte"][d["prompt"][b, :m].long()] + head["wpe"][:m] for b, m in enumerate(lens)])
        got = [logits(through(x, packed)[[e - 1 for e in ends]])]
        at = torch.tensor(lens, device=DEVICE)
        got += [logits(y) for y in steps_of([head["wte"][d["next"][k].long()] + head["wpe"][at + k] for k in range(c["steps"])])]
        return {"logits": got, "kv": kv.reshape(-1)}
    if c["kind"] == "decode":
        return {"out": torch.stack(steps_of(d["x"].double())), "kv": kv.reshape(-1)}
    x = through(torch.cat([d["x"][b, :m] for b, m in enumerate(lens)]).double(), packed, c["kind"] == "prefill")
    out = torch.zeros((B, prompt, H), dtype=torch.float64, device=DEVICE)                # pad rows come back as zeros
    for b, (r0, r1, _) in enumerate(packed):
        out[b, :r1 - r0] = x[r0:r1]
    return {"out": out} if kv is None else {"out": out, "kv": kv.reshape(-1)}


def run(state):
    s = state
    with torch.cuda.stream(s["stream"]):
        if s["kind"] == "generate":
            m = s["model"]
            logits = [m.prefill(s["prompt"], s["lens"])[0]]
            for k in range(s["steps"]):
                logits.append(m.decode_step(s["next"][k])[0])
            return {"logits": logits, "kv": m.stack.kv_cache}
        net = s["net"]
        if s["kind"] == "prefill":
            net.prefill(s["x"], s["lens"], s["out"])
            return {"out": s["out"], "kv": net.kv_cache}
        if s["kind"] == "encode":
            net.encode(s["x"], s["lens"], s["out"])
            return {"out": s["out"]}
        # decode: take the sequences up where they were, then step by step
        if s["layers"] == 1:
            eet.eet_restore(net.handle, s["lens"])
            for k in range(s["steps"]):
                net.decode_step(s["x"][k], s["out"][k])
        else:
            eet.eet_stack_restore(net.handle, s["lens"])
            for k in range(s["steps"]):
                s["tok"].copy_(s["x"][k])             # fixed buffers: the step is recorded once and replayed
                net.decode_step(s["tok"], s["row"])
                s["out"][k].copy_(s["row"])
        return {"out": s["out"], "kv": net.kv_cache}
