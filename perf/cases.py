"""The calls a serving program makes of the cache manager, as cases to time and compare.

A case is a cache (layers, batch, heads, head size, budgets, windows, variants) and a way of using it:

  decode   one pass = `steps` decode steps on a cache in its steady state: conf_kv_attend once per layer,
           conf_kv_step on the step's logits, conf_kv_evict_compact.  With `graph` the steps were recorded
           into a HIP graph by `prepare` and a pass replays it, as launch-bound serving loops do.
  chunk    the same with `chunk` tokens per attention call (prompt chunks, draft tokens that are kept).
  prompt   one pass = conf_kv_load_prefill of every layer (the hand-over from the model's prefill), with
           `observe` the prompt-phase importance of every layer, and then `steps` decode steps, the first of
           which cuts the cache to its budget.

`confident` makes the last step of a pass a confident one for every other sequence (one token takes nearly all
of the probability): those sequences then live a few tokens above the tight budget and give up several tokens
at once, the others live at the loose budget and give up one token per step.

A pass returns the attention output of every layer and step, the confidence scores and the budget choices.
Kept tokens and stored codes show in it: a step attends to what the steps before it kept, and `prepare` has
already run one pass of the decode kinds.
"""
import math

import torch

from paper_2605_24786_amd import ConfKV

HEAVY_PROB, HEAVY_GAIN = 0.02, 3.0      # share of the keys that lean towards the queries, and by how much

_DEFAULTS = dict(kind="decode", layers=32, batch=1, q_heads=32, kv_heads=8, head_dim=128, vocab=128256, prompt=1024,
                 window=128, protected=128, tight=512, loose=1024, tight_last=0, steps=4, confident=True, graph=False,
                 chunk=1, observe=False, scales="token", scope="kv_head", page=0, layout="contiguous")


def _case(name=None, **kw):
    c = dict(_DEFAULTS, **kw)
    return c if name is None else dict(c, name=name)


def listed():
    return [
        # The smallest model in use: multi-head attention, 64 channels, FP16-only cache, one sequence, one token at a
        # time.  Latency: a dozen launches of a megabyte or two each.
        _case("gpt2_b1_decode", layers=12, q_heads=12, kv_heads=12, head_dim=64, vocab=50257, prompt=512, window=-1,
              protected=64, tight=256, loose=512, steps=1, confident=False),
        # One chat user on an 8B-class model with a ragged prompt; the serving loop replays a recorded step.
        _case("llama8b_b1_graph_decode", prompt=1003, tight=512, loose=971, graph=True),
        # A small batch at the middle of the range, eager calls.
        _case("llama8b_b8_decode", batch=8, prompt=4096, tight=1024, loose=2048),
        # The same batch arriving: prompt hand-over, the step that evicts half of every cache, the step behind it.
        _case("llama8b_b8_prompt", kind="prompt", batch=8, prompt=4096, tight=1024, loose=2048, steps=2),
        # A 32B-class model (64 layers, five query heads per kv-head), one sequence, long generation.
        _case("qwen32b_b1_decode", layers=64, q_heads=40, vocab=152064, prompt=4096, window=64, tight=512, loose=2048,
              steps=2, confident=False),
        # Retrieval over a long document: 32768 prompt tokens handed over and cut to the loose budget.
        _case("llama8b_b1_prompt32k", kind="prompt", prompt=32768, tight=512, loose=4096, steps=2, confident=False),
        # A long context that stays: the cache holds some sixteen thousand tokens of one sequence.
        _case("llama8b_b1_decode16k", prompt=16384, tight=8192, loose=16001, steps=2, confident=False),
        # The largest decode step: 32 sequences, pyramidal budgets falling over the layers.
        _case("llama8b_b32_pyramid_decode", batch=32, prompt=2048, window=64, protected=64, tight=1024, tight_last=128,
              loose=2048, steps=2),
        # Draft tokens kept four at a time.
        _case("llama8b_b8_chunk4", kind="chunk", batch=8, prompt=4096, tight=1024, loose=2048, steps=1, chunk=4,
              confident=False),
        # Sixteen tokens per call: chunks of a late prompt, 64 query rows per kv-head.
        _case("llama8b_b8_chunk16", kind="chunk", batch=8, prompt=4096, tight=1024, loose=2048, steps=1, chunk=16,
              confident=False),
        # Prompt-phase importance: every query of a ragged prompt observes the prompt before the first step.
        _case("llama8b_b1_observe", kind="prompt", layers=8, prompt=3001, tight=512, loose=1024, steps=2, chunk=32,
              observe=True, confident=False),
        # The paper's literal bookkeeping: scales per channel, one kept set per layer; an odd batch and length.
        _case("llama8b_b5_literal_decode", batch=5, prompt=3001, tight=700, loose=1777, steps=2, scales="channel",
              scope="layer"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: batch 1 .. 32, caches of 64 .. 32768 tokens, 1 .. 8 query heads per kv-head."""
    most = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(["decode", "decode", "decode", "chunk", "prompt"])
        D = rng.choice([64, 128, 128, 128])
        G = rng.choice([1, 2, 4, 4, 5, 7, 8])
        Hkv = rng.choice([2, 4, 8, 8, 12])
        window = rng.choice([-1, 32, 64, 128, 128])
        c = _case(kind=kind, layers=rng.choice([2, 8, 12, 24, 32, 48, 64]), batch=_log_int(rng, 1, 32), q_heads=G * Hkv,
                  kv_heads=Hkv, head_dim=D, vocab=rng.choice([32000, 50257, 128256, 152064]), window=window,
                  prompt=_log_int(rng, 64, 32768), protected=rng.choice([16, 64, 128]), confident=rng.random() < 0.5,
                  steps=rng.choice([1, 2, 4]))
        c["loose"] = max(32, int(c["prompt"] * rng.uniform(0.3, 1.1)))
        c["tight"] = max(16, int(c["loose"] * rng.uniform(0.3, 0.8)))
        if rng.random() < 0.25:
            c["tight_last"] = max(8, c["tight"] // 8)
        if kind == "decode":
            c["graph"] = rng.random() < 0.25
            variant = rng.choice(["", "", "", "channel", "layer", "paged"])
            if variant == "channel" and D == 128 and window >= 0:
                c["scales"] = "channel"
            elif variant == "layer":
                c["scope"] = "layer"
            elif variant == "paged" and D == 128 and window >= 0 and G > 1:
                # (one launch has to hold a unit's scores on chip in this layout)
                c.update(layout="paged", page=rng.choice([8, 16, 32]), window=min(window, c["protected"]),
                         prompt=min(c["prompt"], 1500), loose=min(c["loose"], 1500), tight=min(c["tight"], 1000))
        elif kind == "chunk":
            if D != 128:
                continue
            c.update(chunk=min(rng.choice([2, 3, 4, 8, 16, 32]), 128 // G), steps=1)
        else:
            c["steps"] = 2
            if rng.random() < 0.25 and D == 128:
                c.update(observe=True, chunk=min(32, 128 // G), prompt=min(c["prompt"], 3001))
        if _cost(c) <= most and _prompt_bytes(c) <= 9 << 30 and _capacity(c) * c["layers"] * c["batch"] * Hkv <= 1 << 25:
            return c


# ---- shapes ----

def _budgets(c):
    """(tight, loose) per layer: constant, or falling linearly from `tight` to `tight_last` over the layers."""
    L = c["layers"]
    first, last = c["tight"], c["tight_last"] or c["tight"]
    tight = [round(first + (last - first) * l / max(1, L - 1)) for l in range(L)]
    return tight, [max(t, t * c["loose"] // first) for t in tight]


def _capacity(c):
    slack = c["page"] - 1 if c["page"] > 1 else 0
    longest = max(c["prompt"], max(_budgets(c)[1]), c["protected"] + slack) + max(1, c["chunk"])
    if c["layout"] == "paged":
        longest += c["window"] + 16 + c["page"]
    return -(-longest // 64) * 64


def _prompt_bytes(c):
    return 4 * c["layers"] * c["batch"] * c["kv_heads"] * c["prompt"] * c["head_dim"] if c["kind"] == "prompt" else 0


def _tokens(c):
    return c["chunk"] if c["kind"] == "chunk" else 1


def _is_confident(c, b, step):
    return c["confident"] and step == c["steps"] - 1 and b % 2 == 0


def _lengths(c):
    """Cache length seen by the attention of (layer, sequence, step), averaged over sequences: [layer][step]."""
    tq, (tight, loose), P = _tokens(c), _budgets(c), c["protected"]
    out = []
    for l in range(c["layers"]):
        row = []
        for s in range(c["steps"]):
            tot = 0
            for b in range(c["batch"]):
                if c["kind"] == "prompt" and s == 0:
                    n = c["prompt"]
                elif c["kind"] != "prompt" and c["confident"] and b % 2 == 0:
                    n = min(max(loose[l], P), max(tight[l], P) + s * tq)
                elif c["kind"] == "prompt":
                    n = min(c["prompt"] + s, max(loose[l], P))
                else:
                    n = max(loose[l], P)
                tot += n + tq
            row.append(tot / c["batch"])
        out.append(row)
    return out


def work(c):
    """Bytes and operations one pass cannot do without: cached rows and logits read once, the importance of every
    cached token read and written, prompts read and stored once, queries, outputs and new rows once; two operations
    per multiply-add of the two contractions (of the score contraction alone where a prompt query only observes)."""
    D, B, H, Hq, T, tq = c["head_dim"], c["batch"], c["kv_heads"], c["q_heads"], c["prompt"], _tokens(c)
    nbytes = flops = 0.0
    row8 = 2 * D + (4 if c["scales"] == "token" else 0)
    for row in _lengths(c):
        for n in row:
            n16 = n if c["window"] < 0 else min(n, c["window"] + tq)
            nbytes += B * H * ((n - n16) * row8 + n16 * 4 * D + 8 * n + tq * 8 * D) + B * Hq * tq * 4 * D
            flops += 4.0 * B * Hq * tq * n * D
        if c["kind"] == "prompt":
            n16 = T if c["window"] < 0 else min(T, c["window"])
            nbytes += B * H * (T * 4 * D + (T - n16) * row8 + n16 * 4 * D + 8 * T)
            if c["observe"]:
                nbytes += B * (H * ((T - n16) * (D + 2) + n16 * 2 * D + 8 * T) + Hq * T * 2 * D)
                flops += B * Hq * float(T) * T * D
    return {"bytes": nbytes + c["steps"] * 4.0 * B * c["vocab"], "flops": flops}


def _cost(c):
    w = work(c)
    return max(w["bytes"], w["flops"] / 50)


def tolerance(c):
    """fp16 outputs of fp16 / INT8 operands with fp32 sums.  Measured on these cases with other split counts of the
    sums: up to 2.9e-4 relative (the rounding of output and probabilities), 2.8e-3 at most; the larger `max` leaves
    room for a token whose score ties with the eviction's cut-off."""
    return {"rel": 1.2e-3, "max": 0.05}


# ---- inputs ----

class _State:
    pass


def _inputs(c, seed):
    """What the model hands over: the steps' queries, keys, values and logits, and prompt(l), called once per layer
    in order, then prompt_q(l) the same way."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1000003 + 17)
    L, B, Hq, H, D, T, V = (c[k] for k in ("layers", "batch", "q_heads", "kv_heads", "head_dim", "prompt", "vocab"))
    S, tq = c["steps"], _tokens(c)
    st = _State()
    st.case = c

    def normal(*shape, dtype=torch.float16):
        return torch.randn(shape, generator=g, device="cuda", dtype=dtype)

    def keys(direction, *shape):
        """Keys of which a few lean along their head's direction; `direction` broadcasts against shape + (D,)."""
        k = normal(*shape, D)
        heavy = torch.rand(shape, generator=g, device="cuda") < HEAVY_PROB
        return k.add_(heavy[..., None] * (HEAVY_GAIN * direction).to(k.dtype))

    u = torch.nn.functional.normalize(normal(L, H, D, dtype=torch.float32), dim=-1)
    mean = (math.sqrt(D) * u).repeat_interleave(Hq // H, dim=1).to(torch.float16)          # [L][Hq][D]
    toks = (B,) if c["kind"] != "chunk" else (B, tq)
    mid = (None,) * len(toks)
    st.q = normal(S, L, *toks, Hq, D).add_(mean[(slice(None), *mid)])
    st.k = keys(u[(slice(None), *mid)], S, L, *toks, H)
    st.v = normal(S, L, *toks, H, D)
    st.logits = normal(S, B, V, dtype=torch.float32).mul_(0.5)
    for s in range(S):
        for b in range(B):
            if _is_confident(c, b, s):
                st.logits[s, b, (7919 * (b + 1) + s) % V] += 25.0
    prompt = lambda l: (keys(u[l][None, :, None, :], B, H, T), normal(B, H, T, D))
    prompt_q = lambda l: normal(B, T, Hq, D).add_(mean[l])
    return st, prompt, prompt_q


def prepare(c, seed):
    L, B = c["layers"], c["batch"]
    tight, loose = _budgets(c)
    st, prompt, prompt_q = _inputs(c, seed)
    st.kv = ConfKV(n_layers=L, batch=B, n_q_heads=c["q_heads"], n_kv_heads=c["kv_heads"], head_dim=c["head_dim"],
                   vocab=c["vocab"], capacity=_capacity(c), fp16_window=c["window"], protected_window=c["protected"],
                   n_tight=tight, n_loose=loose, scale_mode=c["scales"], rank_scope=c["scope"],
                   max_chunk=c["chunk"] if c["chunk"] > 1 else 0, evict_page=c["page"], layout=c["layout"])
    st.out = torch.empty_like(st.q)
    st.conf = torch.empty(c["steps"], B, dtype=torch.float32, device="cuda")
    st.sel = torch.empty(c["steps"], B, dtype=torch.uint8, device="cuda")
    # what the model's layers hold when they call: one tensor per layer and argument
    st.calls = [[(l, st.q[s, l], st.k[s, l], st.v[s, l], st.out[s, l]) for l in range(L)] for s in range(c["steps"])]
    st.scored = [(st.logits[s], st.conf[s], st.sel[s]) for s in range(c["steps"])]
    if c["kind"] == "prompt":
        st.prompt = [prompt(l) for l in range(L)]
        st.prompt_q = [prompt_q(l) for l in range(L)] if c["observe"] else None
        return st
    for l in range(L):
        st.kv.load_prefill(l, *prompt(l))
    if c["graph"]:
        st.kv.static_plan(True)
    _steps(st)                       # the step that cuts the prompt to its budget belongs to no steady-state pass
    if c["graph"]:
        torch.cuda.synchronize()
        st.graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(st.graph):
            _steps(st)
    return st


def _steps(st):
    kv, c = st.kv, st.case
    attend = kv.attend_chunk if c["kind"] == "chunk" else kv.attend
    for layers, scored in zip(st.calls, st.scored):
        for args in layers:
            attend(*args)
        kv.step(*scored)
        kv.evict_compact()


def run(st):
    c = st.case
    if c["kind"] == "prompt":
        for l, (k, v) in enumerate(st.prompt):
            st.kv.load_prefill(l, k, v)
            if c["observe"]:
                st.kv.observe_prompt(l, st.prompt_q[l])
    if c["graph"]:
        st.graph.replay()
    else:
        _steps(st)
    return {"out": st.out, "conf": st.conf, "sel": st.sel}


# ---- the same in 64 bits ----

TAU, ALPHA, DECAY = (float(torch.tensor(x)) for x in (0.7, 0.65, 0.9))      # the manager's defaults, held as fp32


def _exact_confidence(logits):
    """0.4 (1 - H / log V) + 0.3 sigmoid(margin of the two largest) + 0.3 p_max, with the manager's fp32 weights."""
    wh, wm, wp = (float(torch.tensor(x)) for x in (0.4, 0.3, 0.3))
    x = logits.double()
    logp = torch.log_softmax(x, -1)
    p = logp.exp()
    top = x.topk(2, -1).values
    h = -(p * logp).sum(-1) / math.log(x.shape[-1])
    return wh * (1 - h) + wm * torch.sigmoid(top[..., 0] - top[..., 1]) + wp * p.amax(-1)


def _stored_int8(x, scale):
    """What INT8 storage keeps of fp16 rows x: codes times fp16 scales, exact in fp32."""
    s = scale.float()
    ok = (s > 0) & s.isfinite()
    codes = (x.double() / torch.where(ok, s, 1.0).double()).round().clamp(-127, 127)
    return torch.where(ok, codes.float() * s, 0.0)


class _Unit:
    """The cache of one (layer, sequence) over all its kv-heads: rows in order of position, kept rows as indices."""

    def __init__(self, c, k, v):
        self.c = c
        self.raw = [k, v]
        fixed = c["scales"] == "channel"
        amax = [x.abs().amax(1 if fixed else -1, keepdim=True) for x in self.raw]
        self.scale = [(a.float() / 127.0).half() if fixed else None for a in amax]
        H, T = k.shape[:2]
        self.q8 = [self._int8(i, x) for i, x in enumerate(self.raw)]
        self.idx = torch.arange(T, device=k.device).repeat(H, 1)
        self.ema = torch.zeros(H, T, dtype=torch.float32, device=k.device)
        self.is16 = torch.ones(H, T, dtype=torch.bool, device=k.device)
        self._demote()

    def _int8(self, i, x):
        s = self.scale[i]
        return _stored_int8(x, (x.abs().amax(-1, keepdim=True).float() / 127.0).half() if s is None else s)

    def _demote(self):
        W = self.c["window"]
        if W >= 0:
            self.is16 &= self.is16.flip(1).cumsum(1).flip(1) <= W

    def _rows(self, i):
        at = self.idx[..., None].expand(-1, -1, self.raw[i].shape[-1])
        return torch.where(self.is16[..., None], self.raw[i].gather(1, at).float(), self.q8[i].gather(1, at)).double()

    def attend(self, q, k=None, v=None):
        """Causal attention of the tokens q [tq][Hq][D]: the appended ones, or (no k) the last tq cached ones."""
        H, tq, dev = self.idx.shape[0], q.shape[0], q.device
        G, D = q.shape[1] // H, q.shape[2]
        if k is not None:
            first, new = self.raw[0].shape[1], [k.transpose(0, 1), v.transpose(0, 1)]
            self.q8 = [torch.cat([a, self._int8(i, b)], 1) for i, (a, b) in enumerate(zip(self.q8, new))]
            self.raw = [torch.cat([a, b], 1) for a, b in zip(self.raw, new)]
            self.idx = torch.cat([self.idx, torch.arange(first, first + tq, device=dev).repeat(H, 1)], 1)
            self.ema = torch.cat([self.ema, torch.zeros(H, tq, device=dev)], 1)
            self.is16 = torch.cat([self.is16, torch.ones(H, tq, dtype=torch.bool, device=dev)], 1)
        n = self.idx.shape[1]
        qd = q.double().reshape(tq, H, G, D).permute(1, 2, 0, 3).reshape(H, G * tq, D)
        s = torch.bmm(qd, self._rows(0).transpose(1, 2).contiguous()).reshape(H, G, tq, n) * float(torch.tensor(1 / math.sqrt(D)))
        s += torch.full((tq, n), -math.inf, dtype=torch.float64, device=dev).triu(n - tq + 1)
        p = torch.softmax(s, -1)
        late = DECAY ** torch.arange(tq - 1, -1, -1, dtype=torch.float64, device=dev)
        mass = (p.sum(1) * late[:, None]).sum(1)
        self.ema = (DECAY ** tq * self.ema.double() + (1 - DECAY) * mass).float()
        out = torch.bmm(p.reshape(H, G * tq, n), self._rows(1))
        return out.reshape(H, G, tq, D).permute(2, 0, 1, 3).reshape(tq, H * G, D)

    def evict(self, budget):
        H, n = self.idx.shape
        cand = n - min(self.c["protected"], n)
        e = min(n - budget, cand)
        if e > 0:
            a, pos = self.ema[:, :cand].double(), self.idx[:, :cand].double()
            if self.c["scope"] == "layer":
                a = a.sum(0, keepdim=True).expand(H, -1)
            unit = lambda x: (x - x.amin(1, keepdim=True)) / (x.amax(1, keepdim=True) - x.amin(1, keepdim=True)).clamp(min=1e-300)
            score = ALPHA * unit(a) + (1 - ALPHA) * unit(pos)
            keep = torch.cat([score.sort(dim=1, stable=True).indices[:, e:].sort(1).values,
                              torch.arange(cand, n, device=a.device).repeat(H, 1)], 1)
            self.idx, self.ema, self.is16 = (x.gather(1, keep) for x in (self.idx, self.ema, self.is16))
        self._demote()


def exact(c, seed):
    """The pass in float64 (codes, scales and stored importance as the formats define them): confidence, choices and
    the attention outputs; no outputs where pages are evicted whole, or where it takes too long."""
    st, prompt, prompt_q = _inputs(c, seed)
    L, B, S = c["layers"], c["batch"], c["steps"]
    tight, loose = _budgets(c)
    conf = _exact_confidence(st.logits)
    sel = conf >= TAU
    res = {"out": None, "conf": conf, "sel": sel.to(torch.uint8)}
    passes = 1 if c["kind"] == "prompt" else 2       # `prepare` has run one pass of the decode kinds
    if c["page"] or L * B * S * passes > 6000 or (c["observe"] and L * B * c["q_heads"] * c["prompt"] ** 2 > 2e10):
        return res
    choice = sel.tolist()
    out = torch.empty(st.q.shape, dtype=torch.float64, device="cuda")
    prompts = [prompt(l) for l in range(L)] if c["observe"] else (prompt(l) for l in range(L))
    for l, (k, v) in enumerate(prompts):
        pq = prompt_q(l) if c["observe"] else None
        for b in range(B):
            unit = _Unit(c, k[b], v[b])
            if c["observe"]:
                unit.attend(pq[b])
            for _ in range(passes):
                for s in range(S):
                    at = (s, l, b) if c["kind"] == "chunk" else (s, l, b, None)
                    out[s, l, b] = unit.attend(st.q[at], st.k[at], st.v[at]).reshape(out.shape[3:])
                    unit.evict(tight[l] if choice[s][b] else loose[l])
    return dict(res, out=out)
