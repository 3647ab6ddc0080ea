"""The calls whose time matters for a stage: what a program that serves with it does, over the range of its sizes.

A case is one pass through the library's entry points (``paper_2512_21835_amd``): a whole request, one round of decode
steps, the prefill of one or several prompts, or a move of K/V between two devices.  Shapes are the ones of the
repository's workloads (tiny, 8B- and 70B-shaped) and of the two other models that the paper serves (13B-shaped, with a
KV head per query head, and 32B-shaped); most cases run one or two layers of a stage, the first two a whole stage.

Fields of a case: ``kind``; ``shape`` and ``layers``; ``mb`` micro-batches of ``batch`` sequences; ``ctx`` tokens held
per sequence before the call; ``ragged``: sequences of different lengths, from half of ``ctx`` up; ``together``: one
call for all micro-batches, or one call each in turn; ``tokens`` of a prompt and ``chunk``, the tokens per prefill
call; ``fp32``: an fp32 KV cache; ``streamed`` layers kept in pinned host memory, two slots.
"""
import math

import torch

import paper_2512_21835_amd as P

DEV = "cuda"
EPS, THETA = 1e-5, 10000.0
GENERATED = 256   # decode steps of one request, after which the next one takes its place

# hidden, query heads, KV heads, head width, FFN width
SHAPES = {
    "tiny": (256, 4, 2, 64, 688),
    "8b": (4096, 32, 8, 128, 14336),
    "13b": (5120, 40, 40, 128, 13824),
    "32b": (5120, 64, 8, 128, 25600),
    "70b": (8192, 64, 8, 128, 28672),
}
_STREAM = []


class _Shape:
    """The fields that config_for reads."""

    def __init__(self, name, layers):
        self.hidden, self.n_q_heads, self.n_kv_heads, self.head_dim, self.ffn = SHAPES[name]
        self.n_layers, self.rope_theta, self.rms_eps = layers, THETA, EPS

    def tensors(self):
        h, qd, kvd, f = self.hidden, self.n_q_heads * self.head_dim, self.n_kv_heads * self.head_dim, self.ffn
        return {"wq": (qd, h), "wk": (kvd, h), "wv": (kvd, h), "wo": (h, qd), "wg": (f, h), "wu": (f, h), "wd": (h, f),
                "g1": (h,), "g2": (h,)}

    def layer_params(self):
        return sum(math.prod(s) for s in self.tensors().values())


def _case(name, kind, shape, layers, mb=1, batch=1, ctx=0, ragged=False, together=True, tokens=0, chunk=0, fp32=False,
          streamed=0):
    return {"name": name, "kind": kind, "shape": shape, "layers": layers, "mb": mb, "batch": batch, "ctx": ctx,
            "ragged": ragged, "together": together, "tokens": tokens, "chunk": chunk, "fp32": fp32,
            "streamed": streamed}


def listed():
    return [
        # The smallest stage end to end: a 16-token prompt, then 16 decode steps that take the stage's own output.
        # Every launch is a few microseconds: latency and launches count.
        _case("tiny_request", "request", "tiny", 2, tokens=16),
        # One request on a whole 8B-shaped stage: one decode step of one sequence.
        _case("decode_8b_1row", "decode", "8b", 8, ctx=1024),
        # The interleaved schedule: four micro-batches of one sequence, one call each in turn.
        _case("decode_70b_round_robin", "decode", "70b", 1, mb=4, ctx=2048, together=False),
        # KV pressure: eight micro-batches of two sequences near the end of an 8192-token context, in one call.
        _case("decode_70b_16rows_long", "decode", "70b", 1, mb=8, batch=2, ctx=7900),
        # As many sequences as one call takes, of different lengths.
        _case("decode_8b_64rows_ragged", "decode", "8b", 2, mb=8, batch=8, ctx=1100, ragged=True),
        # Weights beyond the HBM budget: four micro-batches decode in one call while two layers stream from the host.
        _case("decode_8b_streamed", "decode", "8b", 3, mb=4, ctx=1024, streamed=2),
        # A short prompt, the commonest prefill of an interactive program.
        _case("prefill_8b_short", "prefill", "8b", 2, tokens=37, chunk=37),
        # An ordinary prompt.
        _case("prefill_8b_1024", "prefill", "8b", 2, tokens=1024, chunk=1024),
        # The largest call: four long prompts at once.
        _case("prefill_70b_4x2048", "prefill", "70b", 1, mb=4, tokens=2048, chunk=2048),
        # A long prompt cut into chunks, so that other requests' decode steps can go between them.
        _case("prefill_32b_chunked", "prefill", "32b", 1, tokens=3500, chunk=500),
        # A cache kept in fp32, with a KV head for every query head.
        _case("prefill_13b_fp32_cache", "prefill", "13b", 1, mb=2, tokens=600, chunk=600, fp32=True),
        # The tail of a sequence's cache leaves for another device and comes back (device buffers on this side).
        _case("kv_transfer_70b", "kv", "70b", 16, ctx=2000, tokens=500),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["request", "decode", "decode", "decode", "prefill", "prefill", "prefill", "kv"])
    if kind == "request":
        return _unnamed("request", "tiny", rng.randint(1, 4), tokens=_log(rng, 2, 48))
    if kind == "kv":
        shape = rng.choice(["8b", "13b", "70b"])
        tokens = _log(rng, 16, 1024)
        return _unnamed("kv", shape, 4 if shape == "13b" else rng.randint(4, 16), ctx=tokens + _log(rng, 16, 2048),
                        tokens=tokens)
    shape = rng.choice(["8b", "13b", "32b", "70b"])
    if kind == "decode":
        rows = _log(rng, 1, 64)
        batch = rng.choice([b for b in (1, 2, 4, 8) if b <= rows])
        mb = min(rows // batch, 64 // batch)
        # bounded by the cache of one layer: rows x context x bytes per token
        per_token = 4 * SHAPES[shape][2] * SHAPES[shape][3]
        most = min(8000, int(3e9 / (per_token * mb * batch)))
        fp32 = rng.random() < 0.15
        streamed = int(rng.random() < 0.12)
        return _unnamed("decode", shape, 1 + streamed, mb=mb, batch=batch, ctx=_log(rng, 16, most),
                        ragged=rng.random() < 0.5, together=mb * batch > 4 or rng.random() < 0.5, fp32=fp32,
                        streamed=streamed)
    mb = rng.choice([1, 1, 2, 4])
    tokens = _log(rng, 8, 4096 // mb)
    fp32 = tokens <= 1024 and rng.random() < 0.25
    chunk = tokens if rng.random() < 0.7 else max(2, -(-tokens // rng.randint(2, 6)))
    return _unnamed("prefill", shape, 1, mb=mb, tokens=tokens, chunk=chunk, fp32=fp32)


def _unnamed(*a, **k):
    c = _case("", *a, **k)
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs
def _lengths(case):
    """Tokens that each sequence (mb, b) holds before the call."""
    n = case["mb"] * case["batch"]
    if not case["ragged"]:
        return [case["ctx"]] * n
    half = max(1, case["ctx"] // 2)
    return [case["ctx"] - int(i * 0.6180339887 % 1.0 * half) for i in range(n)]


def _generator(seed, part):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1_000_003 + part) % (1 << 62))
    return g


def _weights(shape, layer, seed):
    g = _generator(seed, 1 + layer)
    w = {}
    for name, size in shape.tensors().items():
        t = torch.empty(size, dtype=torch.bfloat16, device=DEV)
        w[name] = t.normal_(1.0 if len(size) == 1 else 0.0, 0.02, generator=g)
    return w


def _cached(case, seq, n, seed):
    """K and V [layers][n][KV heads][d] that sequence `seq` holds, in the cache's type."""
    shape = _Shape(case["shape"], case["layers"])
    g = _generator(seed, 1000 + seq)
    size = (2, shape.n_layers, n, shape.n_kv_heads, shape.head_dim)
    kv = torch.empty(size, dtype=torch.float32 if case["fp32"] else torch.bfloat16, device=DEV).normal_(generator=g)
    return kv[0], kv[1]


def _hidden(case, seed):
    shape = _Shape(case["shape"], case["layers"])
    rows = case["tokens"] if case["kind"] in ("prefill", "request") else 1
    g = _generator(seed, 500)
    return torch.empty((case["mb"], case["batch"], rows, shape.hidden), device=DEV).normal_(generator=g)


class _State:
    """A stage and its inputs; the stage goes with the last reference."""

    def __init__(self, case, seed):
        self.case, self.handle = case, None
        if not _STREAM:
            _STREAM.append(torch.cuda.Stream())
        shape = _Shape(case["shape"], case["layers"])
        kind, seqs = case["kind"], case["mb"] * case["batch"]
        most = case["ctx"] + case["tokens"] + (GENERATED if kind == "decode" else 16)
        cfg = P.config_for(shape, max_microbatches=case["mb"], max_batch=case["batch"], max_context=most,
                           n_resident_max=shape.n_layers - case["streamed"], kv_fp32=case["fp32"],
                           compute_stream=_STREAM[0].cuda_stream)
        self.handle = P.stage_init(cfg)
        if kind != "kv":
            for layer in range(shape.n_layers):
                w = _weights(shape, layer, seed)
                torch.cuda.synchronize()
                P.stage_load_layer(self.handle, layer, w, int(layer < shape.n_layers - case["streamed"]))
        self.ids = list(range(case["mb"]))
        self.lengths = _lengths(case)
        self.cached = [_cached(case, i, n, seed) for i, n in enumerate(self.lengths) if n] if kind != "prefill" else []
        self.steps = 0
        if kind == "kv":
            size = (shape.n_layers, case["tokens"], shape.n_kv_heads, shape.head_dim)
            self.k = torch.empty(size, dtype=torch.int16, device=DEV)
            self.v = torch.empty_like(self.k)
        else:
            self.x = _hidden(case, seed)
            if kind == "prefill":   # one input per call, [mb][batch][tokens of the call][hidden]
                self.x = [c.contiguous() for c in self.x.split(case["chunk"], 2)]
                self.y = [torch.empty_like(c) for c in self.x]
            elif kind == "request":
                self.y = torch.empty_like(self.x)
                self.out = torch.empty((16, shape.hidden), device=DEV)
            else:
                self.x = self.x[:, :, 0].contiguous()
                self.y = torch.empty_like(self.x)
        torch.cuda.synchronize()
        if self.cached:
            self.arrive()

    def reset(self):
        for mb in self.ids:
            for b in range(self.case["batch"]):
                P.stage_reset_sequence(self.handle, mb, b)

    def arrive(self):
        """Requests whose cache was computed elsewhere: their K/V is appended."""
        for i, (k, v) in enumerate(self.cached):
            P.stage_kv_append(self.handle, i // self.case["batch"], i % self.case["batch"], k.shape[1], k, v)

    def __del__(self):
        if self.handle is not None:
            P.stage_destroy(self.handle)
            self.handle = None


def prepare(case, seed):
    return _State(case, seed)


# ------------------------------------------------------------------ the passes
def run(state):
    case, h = state.case, state.handle
    kind = case["kind"]
    if kind == "kv":
        P.stage_kv_export_tail(h, 0, 0, case["tokens"], state.k, state.v, True)
        P.stage_kv_append(h, 0, 0, case["tokens"], state.k, state.v)
        return state.k, state.v
    if kind == "decode":
        if state.steps == GENERATED:   # the requests have ended: others take their places
            state.reset()
            state.arrive()
            state.steps = 0
        state.steps += 1
        if case["together"]:
            P.stage_decode(h, state.ids, case["batch"], state.x, state.y)
        else:
            for mb in state.ids:
                P.stage_decode(h, [mb], case["batch"], state.x[mb], state.y[mb])
        return state.y
    state.reset()
    if kind == "prefill":
        for x, y in zip(state.x, state.y):
            P.stage_prefill(h, state.ids, case["batch"], x.shape[2], x, y)
        return state.y
    P.stage_prefill(h, [0], 1, case["tokens"], state.x, state.y)
    last = state.y[0, 0, case["tokens"] - 1]
    for i in range(16):
        P.stage_decode(h, [0], 1, last, state.out[i])
        last = state.out[i]
    return state.y, state.out


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    shape = _Shape(case["shape"], case["layers"])
    layers, h = shape.n_layers, shape.hidden
    kv_token = 2 * shape.n_kv_heads * shape.head_dim * (4 if case["fp32"] else 2)   # bytes per layer
    if case["kind"] == "kv":   # out and back, each read and written
        return {"bytes": 4.0 * layers * case["tokens"] * kv_token, "flops": 0.0}
    params = shape.layer_params()
    seqs, qd = case["mb"] * case["batch"], shape.n_q_heads * shape.head_dim
    if case["kind"] == "decode":
        held = sum(_lengths(case))
        calls = 1 if case["together"] else case["mb"]
        return {"bytes": float(calls * layers * params * 2 + layers * (held + seqs) * kv_token + seqs * 8 * h),
                "flops": float(layers * (2 * params * seqs + 4 * qd * (held + seqs)))}
    n = case["tokens"]
    steps = 16 if case["kind"] == "request" else 0
    calls = -(-n // case["chunk"]) if case["kind"] == "prefill" else 1 + steps
    pairs = seqs * (n * (n + 1) // 2 + steps * n + steps * (steps + 1) // 2)
    return {"bytes": float(calls * layers * params * 2 + layers * seqs * (n + steps) * kv_token + seqs * (n + steps) * 8 * h),
            "flops": float(layers * (2 * params * seqs * (n + steps) + 4 * qd * pairs))}


def tolerance(case):
    """About four times the largest difference from `exact` over the listed cases and some 60 drawn ones.

    With an fp32 cache, what fp32 sums and 16-bit operand pairs leave: up to 1.1e-5 (largest element 5.6e-5 rms).  With
    a bf16 cache, a K or V element whose exact value lies near the middle of two bf16 values may be rounded to either,
    one bf16 step apart: prefill 3.7e-4 (6.7e-3), decode, where only a row's newest token can differ, 1.6e-4 (3.0e-3),
    the tiny stage's fed-back steps 7.0e-5 (3.5e-4).
    """
    if case["kind"] == "kv":
        return "exact"
    if case["fp32"]:
        return {"rel": 5e-5, "max": 3e-4}
    return {"request": {"rel": 3e-4, "max": 1.5e-3}, "decode": {"rel": 6e-4, "max": 0.012},
            "prefill": {"rel": 1.5e-3, "max": 0.03}}[case["kind"]]


# ------------------------------------------------------------------ the same in float64
def _rms(x, g):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * g


def _rope(x, pos):
    """x [n, heads, d] at positions pos [n]: rotate-half pairs."""
    half = x.shape[-1] // 2
    inv = torch.tensor([THETA ** (-2.0 * i / x.shape[-1]) for i in range(half)], dtype=torch.float64, device=x.device)
    ang = pos.double()[:, None] * inv
    c, s = ang.cos()[:, None], ang.sin()[:, None]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, a * s + b * c], -1)


def _layer(shape, w, seqs, cache, fp32):
    """One layer over sequences [(x [n, H])], their caches [(k, v) [held, KV heads, d]] extended in place."""
    hq, hkv, d = shape.n_q_heads, shape.n_kv_heads, shape.head_dim
    x = torch.cat(seqs)
    y = _rms(x, w["g1"].double())
    q, k, v = (y @ w[t].double().t() for t in ("wq", "wk", "wv"))
    att, at = torch.empty_like(q), 0
    for i, s in enumerate(seqs):
        n = s.shape[0]
        held = cache[i][0].shape[0]
        pos = torch.arange(held, held + n, device=x.device)
        qi = _rope(q[at:at + n].view(n, hq, d), pos)
        ki, vi = _rope(k[at:at + n].view(n, hkv, d), pos), v[at:at + n].view(n, hkv, d)
        if not fp32:   # the cache element is the contract: bf16
            ki, vi = ki.float().bfloat16().double(), vi.float().bfloat16().double()
        cache[i] = (torch.cat([cache[i][0], ki]), torch.cat([cache[i][1], vi]))
        later = torch.arange(held + n, device=x.device)[None, :] > pos[:, None]
        for hd in range(hq):
            kk, vv = cache[i][0][:, hd * hkv // hq], cache[i][1][:, hd * hkv // hq]
            sc = (qi[:, hd] @ kk.t()) / math.sqrt(d)
            att[at:at + n, hd * d:(hd + 1) * d] = torch.softmax(sc.masked_fill(later, -math.inf), -1) @ vv
        at += n
    x = x + att @ w["wo"].double().t()
    y = _rms(x, w["g2"].double())
    g = y @ w["wg"].double().t()
    x = x + (g / (1 + torch.exp(-g)) * (y @ w["wu"].double().t())) @ w["wd"].double().t()
    return list(x.split([s.shape[0] for s in seqs]))


def exact(case, seed):
    if case["kind"] == "kv":
        return None
    shape = _Shape(case["shape"], case["layers"])
    n_seq, h = case["mb"] * case["batch"], shape.hidden
    x = _hidden(case, seed).double()
    seqs = [x[i // case["batch"], i % case["batch"]] for i in range(n_seq)]
    empty = torch.zeros((0, shape.n_kv_heads, shape.head_dim), dtype=torch.float64, device=DEV)
    caches = [[(empty, empty)] * n_seq for _ in range(shape.n_layers)]
    if case["kind"] == "decode":
        for i, n in enumerate(_lengths(case)):
            k, v = _cached(case, i, n, seed)
            for layer in range(shape.n_layers):
                caches[layer][i] = (k[layer].double(), v[layer].double())

    def forward(seqs):
        for layer in range(shape.n_layers):
            seqs = _layer(shape, _weights(shape, layer, seed), seqs, caches[layer], case["fp32"])
        return seqs

    out = forward(seqs)
    if case["kind"] == "decode":
        return torch.stack(out).view(case["mb"], case["batch"], h)
    y = torch.stack(out).view(case["mb"], case["batch"], -1, h)
    if case["kind"] == "prefill":
        return [c.contiguous() for c in y.split(case["chunk"], 2)]
    steps, last = [], out[0][-1:]
    for _ in range(16):
        last = forward([last])[0]
        steps.append(last[0])
    return y, torch.stack(steps)
