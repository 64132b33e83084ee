"""The calls a program that serves agents makes of this library, over the
sizes it meets, each with its inputs, its least work and its exact result.

One case is one of five kinds ("op"):

  decode  one decode call of a layer: main threads, each perhaps with an
          auxiliary thread forked from it, over a paged cache
  step    one token for each thread through every layer: fork, sq_step_begin,
          sq_step_attn per layer, release
  extend  causal attention of a chunk that has just been appended
  append  a fork of a cached thread and a chunk of new tokens for it, all layers
          ("turn": 1 adds the chunk's attention and one decode step, which makes
          it the whole turn of an auxiliary thread)
  evict   spans leave the cache: on a fork (out of place), on a thread that was
          appended to first (in place), or masked first and compacted later

A pass leaves the store as it found it (what it forks or creates it releases),
so it can be repeated; the pages it writes are the ones after the prepared
threads' pages, and are returned whole.  K and V are N(0, 1) in bf16 with four
channels per KV head scaled by 8, the outliers that cached keys and values of
trained models show.  Head shapes are the ones of the benchmark (32 query and 8
KV heads of 128; 64 and 8 of 64 with sinks and windows).
"""

import math

import numpy as np
import torch

from paper_2602_22603_amd import sq, workload

P = 16
KV_SCALE = (1.0 / 16, 1.0 / 16)  # of an 8-bit store: 28 is its largest value


# ---------------------------------------------------------------------------
# The cases.
def _case(name, op, **kw):
    c = dict(name=name, op=op, hq=32, hkv=8, d=128, kv8=False, sinks=False, window=0, layers=1)
    c.update(kw)
    return c


def listed():
    return [
        # a short task: main and auxiliary thread right after the first fork
        _case("decode_small", "decode", tasks=1, aux=True, lo=2048, hi=2048, back=48, private=48),
        # eight tasks of 128K tokens, each with an auxiliary thread: the
        # largest batch the benchmark runs (4.3 GB of keys and values)
        _case("decode_128k", "decode", tasks=8, aux=True, lo=131072, hi=131072, back=256, private=512),
        # a mixed batch on an 8-bit cache: threads of every age, no two alike
        _case("decode_mixed_8bit", "decode", tasks=12, aux=False, lo=3001, hi=61003, back=0,
              private=0, kv8=True),
        # one task's next token through the layers after an eviction left
        # 22.7K tokens: main and auxiliary thread
        _case("step_compacted", "step", tasks=1, aux=True, lo=22673, hi=22673, back=17, private=211,
              layers=12),
        # the same for a model whose layers alternate between a window of 128
        # keys and all of them, with sinks
        _case("step_windowed", "step", tasks=4, aux=False, lo=9000, hi=33333, back=0, private=0,
              layers=12, hq=64, d=64, sinks=True, window=128),
        # a turn's tool response of 8192 tokens after the first 16K, over the layers
        _case("append_turn", "append", base=16389, n=8192, layers=24, turn=False),
        # an auxiliary thread from its fork to its first token on an 8-bit
        # cache: the prompt stored, its attention, one step
        _case("aux_turn_8bit", "append", base=30011, n=512, layers=8, turn=True, kv8=True),
        # the first tool responses of a 64K context leave it (65%)
        _case("evict_64k", "evict", length=65536, pairs=40, frac=0.65, how="oneshot", layers=6, shape=3),
        # a 16K thread is built, and stale spans leave it in its own pages
        _case("evict_inplace", "evict", length=16411, pairs=12, frac=0.5, how="inplace", layers=6, shape=5),
        # the attention of an 8192-token chunk over that compacted context
        _case("extend_8k", "extend", base=22673, n=8192),
        # a short tool response (or a batch of draft tokens) late in a task
        _case("extend_short", "extend", base=60547, n=77),
        # a reasoning chunk of a model of 64-channel heads with sinks
        _case("extend_sinks_d64", "extend", base=20011, n=1999, hq=64, d=64, sinks=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["decode", "decode", "step", "extend", "extend", "append", "evict"])
    hq, hkv, d = rng.choice([(32, 8, 128), (32, 8, 128), (64, 8, 64), (16, 8, 128), (8, 8, 64), (16, 2, 128)])
    c = _case(None, op, hq=hq, hkv=hkv, d=d, kv8=rng.random() < 0.3, sinks=rng.random() < 0.3)
    del c["name"]
    if op == "decode":
        tasks = _log(rng, 1, 16)
        hi = _log(rng, 500, min(131072, 600000 // tasks))
        c.update(tasks=tasks, aux=rng.random() < 0.5, lo=max(65, hi // _log(rng, 1, 12)), hi=hi,
                 back=rng.randrange(0, 60), private=rng.randrange(1, 600))
    elif op == "step":
        tasks = _log(rng, 1, 8)
        hi = _log(rng, 500, 100000 // tasks)
        c.update(tasks=tasks, aux=rng.random() < 0.5, lo=max(65, hi // _log(rng, 1, 6)), hi=hi,
                 back=rng.randrange(0, 60), private=rng.randrange(1, 300), layers=_log(rng, 4, 12),
                 window=rng.choice([0, 0, 128]))
    elif op == "extend":
        n = _log(rng, 3, 8192)
        c.update(base=_log(rng, 100, 22000 if n > 2000 else 60000), n=n, window=rng.choice([0, 0, 0, 128]))
    elif op == "append":
        turn = rng.random() < 0.5
        c.update(base=_log(rng, 50, 30000), n=_log(rng, 5, 700 if turn else 8192), layers=_log(rng, 2, 8 if turn else 24),
                 turn=turn)
    else:
        length = _log(rng, 1500, 65000)
        c.update(length=length, pairs=max(2, min(40, length // 900)), frac=round(rng.uniform(0.2, 0.7), 2),
                 how=rng.choice(["oneshot", "oneshot", "inplace", "chunked", "deferred"]),
                 layers=_log(rng, 1, 4 if length > 20000 else 6), shape=rng.randrange(1000), sinks=False)
    return c


# ---------------------------------------------------------------------------
# Sizes that follow from a case alone.
def _lengths(c):
    """The main threads' lengths: spread over [lo, hi] by their logarithm."""
    n, lo, hi = c["tasks"], c["lo"], c["hi"]
    return [int(hi * (lo / hi) ** (i / max(1, n - 1))) if n > 1 else hi for i in range(n)]


def _threads(c):
    """(task, shared tokens, private tokens) of every thread of a batch."""
    out = []
    for t, n in enumerate(_lengths(c)):
        out.append((t, n, 0))
        if c["aux"]:
            out.append((t, n - c["back"], c["private"]))
    return out


def _spans(c):
    """Reasoning and tool spans in turn; the tool spans that leave."""
    rng = np.random.default_rng([2602, c["shape"]])
    n, pairs = c["length"], c["pairs"]
    reasoning = workload.lognormal_lengths(rng, pairs, 6.0, 0.4, n // 4)
    tool = workload.lognormal_lengths(rng, pairs, 7.0, 0.8, n - n // 4)
    spans, pos = [], 0
    for r, t in zip(reasoning, tool):
        spans.append((pos + r, pos + r + t))
        pos += r + t
    chosen, gone = workload.choose_until(rng, spans, list(range(pairs)), c["frac"] * n)
    return spans, chosen, gone


def _pages(n):
    return (n + P - 1) // P


def _row_bytes(c):
    """K and V of one token of one layer."""
    return 2 * c["hkv"] * c["d"] * (1 if c["kv8"] else 2)


def _pair_flops(c, pairs):
    return 4.0 * c["d"] * c["hq"] * pairs


def _io_bytes(c, rows):
    return rows * c["hq"] * c["d"] * (2 + 4)


def _chunk_pairs(base, n, window):
    """(query, key) pairs of a causal chunk of n after base tokens."""
    if not window:
        return n * base + n * (n + 1) / 2
    return sum(min(window, base + j + 1) for j in range(n))


def work(case):
    c = case
    row = _row_bytes(c)
    if c["op"] in ("decode", "step"):
        new = 1 if c["op"] == "step" else 0
        bytes_ = flops = 0.0
        for layer in range(c["layers"]):
            w = _window(c, layer)
            for t, n in enumerate(_lengths(c)):
                bytes_ += min(w, n) * row if w else n * row  # a fork's shared tokens count once
            for t, shared, private in _threads(c):
                n = shared + private + new
                bytes_ += (0 if w else private * row) + new * 2 * row
                flops += _pair_flops(c, min(w, n) if w else n)
            bytes_ += _io_bytes(c, len(_threads(c)))
        return {"bytes": bytes_, "flops": flops}
    if c["op"] == "extend":
        keys = min(c["base"], c["window"]) + c["n"] if c["window"] else c["base"] + c["n"]
        return {"bytes": keys * row + _io_bytes(c, c["n"]),
                "flops": _pair_flops(c, _chunk_pairs(c["base"], c["n"], c["window"]))}
    if c["op"] == "append":
        bytes_ = c["layers"] * c["n"] * (row + 4.0 * c["hkv"] * c["d"])
        flops = 0.0
        if c["turn"]:
            n = c["base"] + c["n"]
            bytes_ += c["layers"] * (2 * n * row + _io_bytes(c, c["n"] + 1))
            flops = c["layers"] * _pair_flops(c, _chunk_pairs(c["base"], c["n"], 0) + n + 1)
        return {"bytes": bytes_, "flops": flops}
    spans, chosen, gone = _spans(c)
    first = min(spans[i][0] for i in chosen)
    moved = c["length"] - gone - first // P * P
    bytes_ = moved * (c["layers"] * 2.0 * row + 8)
    if c["how"] == "inplace":
        bytes_ += c["layers"] * c["length"] * (row + 4.0 * c["hkv"] * c["d"])
    if c["how"] == "deferred":
        bytes_ += c["length"] * row
    return {"bytes": bytes_, "flops": 0.0}


def tolerance(case):
    if case["op"] == "evict" and case["how"] != "deferred" or case["op"] == "append" and not case["turn"]:
        return "exact"
    # fp32 sums of bf16 products, weights of 16 bits: measured 7e-7 to 2.9e-6
    # of the 64-bit result (2-norm) over the listed and drawn cases
    return {"rel": 1e-5}


def _window(c, layer):
    """The window of a layer: every second one of a windowed step."""
    return c["window"] if c["op"] != "step" or layer % 2 == 0 else 0


# ---------------------------------------------------------------------------
# Inputs.
class _Draw:
    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(int(seed))
        self.outliers = None

    def normal(self, *shape):
        return torch.randn(shape, generator=self.gen, device="cuda", dtype=torch.float32)

    def kv(self, c, n):
        """K or V of n tokens: bf16 [layers, n, hkv, d]."""
        if self.outliers is None:
            self.outliers = torch.ones(c["hkv"], c["d"], device="cuda")
            at = torch.rand(c["hkv"], c["d"], generator=self.gen, device="cuda").argsort(1)[:, :4]
            self.outliers.scatter_(1, at, 8.0)
        x = torch.empty(c["layers"], n, c["hkv"], c["d"], device="cuda", dtype=torch.bfloat16)
        for layer in range(c["layers"]):
            x[layer] = self.normal(n, c["hkv"], c["d"]) * self.outliers
        return x

    def q(self, c, *shape):
        return self.normal(*shape, c["hq"], c["d"]).to(torch.bfloat16)

    def sinks(self, c):
        return self.normal(c["hq"]) if c["sinks"] else None


def _store(c, pages, seqs, longest, **kw):
    return sq.Store(num_layers=c["layers"], num_q_heads=c["hq"], num_kv_heads=c["hkv"],
                    head_dim=c["d"], num_pages=pages, max_seqs=seqs,
                    max_pages_per_seq=_pages(longest) + 1,
                    kv_scales=[KV_SCALE] * c["layers"] if c["kv8"] else None, **kw)


def _inputs(c, seed):
    """Everything a case is given, in a fixed order of draws."""
    g = _Draw(seed)
    x = {}
    if c["op"] in ("decode", "step"):
        x["main"] = [(g.kv(c, n), g.kv(c, n)) for n in _lengths(c)]
        x["private"] = [(g.kv(c, p), g.kv(c, p)) if p else None for _, _, p in _threads(c)]
        b = len(_threads(c))
        x["q"] = g.q(c, c["layers"], b)
        if c["op"] == "step":
            x["new"] = (g.kv(c, b), g.kv(c, b))
    elif c["op"] == "extend":
        n = c["base"] + c["n"]
        x["kv"] = (g.kv(c, n), g.kv(c, n))
        x["q"] = g.q(c, c["n"])
    elif c["op"] == "append":
        x["base"] = (g.kv(c, c["base"]), g.kv(c, c["base"]))
        x["chunk"] = (g.kv(c, c["n"]), g.kv(c, c["n"]))
        if c["turn"]:
            x["q"] = g.q(c, c["layers"], c["n"])
            x["new"] = (g.kv(c, 1), g.kv(c, 1))
            x["q1"] = g.q(c, c["layers"], 1)
    else:
        x["kv"] = (g.kv(c, c["length"]), g.kv(c, c["length"]))
        x["q"] = g.q(c, 1)
    x["sinks"] = g.sinks(c)
    return x


def prepare(case, seed):
    c = dict(case)
    x = _inputs(c, seed)
    s = {"case": c, "sinks": x["sinks"]}
    if c["op"] in ("decode", "step"):
        lengths, threads = _lengths(c), _threads(c)
        grown = sum(_pages(n) + 1 for n in lengths) + sum(_pages(p) + 3 for _, _, p in threads)
        st = _store(c, grown + 2 * len(threads), 2 * len(threads) + len(lengths),
                    max(lengths) + max(p for _, _, p in threads) + 16)
        mains = [st.seq_create() for _ in lengths]
        for h, (k, v) in zip(mains, x["main"]):
            st.append(h, k, v)
        s["seqs"] = []
        for (t, shared, private), kv in zip(threads, x["private"]):
            if not private:
                s["seqs"].append(mains[t])
                continue
            s["seqs"].append(st.fork(mains[t], shared))
            st.append(s["seqs"][-1], *kv)
        s["q"] = x["q"]
        s["out"] = torch.empty(x["q"].shape, dtype=torch.float32, device="cuda")
        if c["op"] == "step":
            s["k"], s["v"] = x["new"]
            s["lengths"] = [a + b for _, a, b in threads]
            s["first_new"] = st.num_pages - st.stats()["free_pages"]
    elif c["op"] == "extend":
        n = c["base"] + c["n"]
        st = _store(c, _pages(n) + 1, 1, n)
        s["seq"] = st.seq_create()
        st.append(s["seq"], *x["kv"])
        s["q"] = x["q"]
        s["out"] = torch.empty(x["q"].shape, dtype=torch.float32, device="cuda")
    elif c["op"] == "append":
        n = c["base"] + c["n"] + 1
        st = _store(c, _pages(c["base"]) + _pages(c["n"]) + 4, 2, n)
        s["seq"] = st.seq_create()
        st.append(s["seq"], *x["base"])
        s["k"], s["v"] = x["chunk"]
        s["first_new"] = _pages(c["base"])
        if c["turn"]:
            s["q"], s["q1"], s["new"] = x["q"], x["q1"], x["new"]
            s["out"] = torch.empty(x["q"].shape, dtype=torch.float32, device="cuda")
            s["out1"] = torch.empty(x["q1"].shape, dtype=torch.float32, device="cuda")
    else:
        spans, s["chosen"], gone = _spans(c)
        kept = _pages(c["length"] - gone)
        inplace = c["how"] == "inplace"
        st = _store(c, _pages(c["length"]) + (1 if inplace else kept + 2), 2, c["length"],
                    evict_inplace=inplace, evict_chunk_pages=64 if c["how"] == "chunked" else 0)
        s["spans"] = spans
        s["q"] = x["q"]
        s["out"] = torch.empty(x["q"].shape, dtype=torch.float32, device="cuda")
        if inplace:
            s["k"], s["v"] = x["kv"]
            s["first_new"] = 0
        else:
            s["seq"] = st.seq_create()
            st.append(s["seq"], *x["kv"])
            for i, (a, b) in enumerate(spans):
                st.span_mark(s["seq"], i, a, b)
            s["first_new"] = _pages(c["length"])
    s["store"] = st
    return s


# ---------------------------------------------------------------------------
# One pass.
def _written(s):
    """The pages a pass writes: all after the prepared threads' pages."""
    st, p = s["store"], s["first_new"]
    return {"k": st.k_pool[:, :, p:], "v": st.v_pool[:, :, p:], "pos": st.pos_pool[p:]}


def run(s):
    return _RUN[s["case"]["op"]](s)


def _run_decode(s):
    c = s["case"]
    return s["store"].decode(0, s["seqs"], s["q"][0], out=s["out"][0], window=c["window"], sinks=s["sinks"])


def _run_step(s):
    c, st = s["case"], s["store"]
    seqs = [st.fork(h, n) for h, n in zip(s["seqs"], s["lengths"])]
    st.step_begin(seqs, window=c["window"])
    for layer in range(c["layers"]):
        st.step_attn(layer, s["k"][layer], s["v"][layer], s["q"][layer], out=s["out"][layer],
                     window=_window(c, layer), sinks=s["sinks"])
    for h in seqs:
        st.release(h)
    return {"out": s["out"], **_written(s)}


def _run_extend(s):
    c = s["case"]
    return s["store"].extend(0, s["seq"], s["q"], out=s["out"], window=c["window"], sinks=s["sinks"])


def _run_append(s):
    c, st = s["case"], s["store"]
    h = st.fork(s["seq"], c["base"])
    st.append(h, s["k"], s["v"])
    got = {}
    if c["turn"]:
        for layer in range(c["layers"]):
            st.extend(layer, h, s["q"][layer], out=s["out"][layer], sinks=s["sinks"])
        st.step_begin([h])
        for layer in range(c["layers"]):
            st.step_attn(layer, s["new"][0][layer], s["new"][1][layer], s["q1"][layer], out=s["out1"][layer],
                         sinks=s["sinks"])
        got = {"out": s["out"], "out1": s["out1"]}
    st.release(h)
    return {**got, **_written(s)}


def _run_evict(s):
    c, st = s["case"], s["store"]
    got = {}
    if c["how"] == "inplace":
        h = st.seq_create()
        st.append(h, s["k"], s["v"])
        for i, (a, b) in enumerate(s["spans"]):
            st.span_mark(h, i, a, b)
    else:
        h = st.fork(s["seq"], c["length"])
    if c["how"] == "deferred":
        st.evict(h, s["chosen"], deferred=True)
        got["out"] = st.decode(0, [h], s["q"], out=s["out"])
        stats = st.compact(h)
    else:
        stats = st.evict(h, s["chosen"])
    st.release(h)
    return {"stats": stats, **got, **_written(s)}


_RUN = {"decode": _run_decode, "step": _run_step, "extend": _run_extend, "append": _run_append,
        "evict": _run_evict}


# ---------------------------------------------------------------------------
# The exact results, in 64 bits.
def _held(c, x):
    """The values a store of the case holds for x, in 64 bits."""
    if not c["kv8"]:
        return x.double()
    y = (x.float() * float(np.float32(1.0 / np.float32(KV_SCALE[0])))).clamp(-448.0, 448.0)
    return y.to(torch.float8_e4m3fn).double() * KV_SCALE[0]


def _attend(c, q, k, v, first, last, sinks):
    """q [n, hq, d], k and v [L, hkv, d] (64 bits): row j over keys first[j] .. last[j]."""
    n, g = q.shape[0], c["hq"] // c["hkv"]
    out = torch.empty(q.shape, dtype=torch.float64, device=q.device)
    at = torch.arange(k.shape[0], device=q.device)
    step = max(1, 60_000_000 // k.shape[0])
    for h in range(c["hq"]):
        kh, vh = k[:, h // g].contiguous(), v[:, h // g].contiguous()
        for j in range(0, n, step):
            x = (q[j:j + step, h].double() @ kh.T) / math.sqrt(c["d"])
            seen = (at >= first[j:j + step, None]) & (at <= last[j:j + step, None])
            x.masked_fill_(~seen, -math.inf)
            m = x.amax(1, keepdim=True)
            if sinks is not None:
                m = torch.maximum(m, sinks[h].double())
            w = torch.exp(x - m)
            den = w.sum(1, keepdim=True)
            if sinks is not None:
                den = den + torch.exp(sinks[h].double() - m)
            out[j:j + step, h] = (w @ vh) / den
    return out


def _rows(n, base, window, device):
    last = base + torch.arange(n, device=device)
    return (last - window + 1 if window else torch.zeros_like(last)), last


def _exact_batch(c, x, layer, new):
    """One layer of a decode call or step (new: its tokens join)."""
    out = []
    w = _window(c, layer)
    for b, (t, shared, private) in enumerate(_threads(c)):
        parts = []
        for i in (0, 1):
            rows = [x["main"][t][i][layer, :shared]]
            if private:
                rows.append(x["private"][b][i][layer])
            if new:
                rows.append(x["new"][i][layer, b:b + 1])
            parts.append(_held(c, torch.cat(rows)))
        n = parts[0].shape[0]
        first, last = _rows(1, n - 1, w, "cuda")
        out.append(_attend(c, x["q"][layer, b:b + 1], *parts, first, last, x["sinks"]))
    return torch.cat(out)


def exact(case, seed):
    c = dict(case)
    none = {"k": None, "v": None, "pos": None}
    if c["op"] == "evict" and c["how"] != "deferred" or c["op"] == "append" and not c["turn"]:
        return None  # bytes that move
    x = _inputs(c, seed)
    if c["op"] == "decode":
        return _exact_batch(c, x, 0, False)
    if c["op"] == "step":
        return {"out": torch.stack([_exact_batch(c, x, layer, True) for layer in range(c["layers"])]), **none}
    if c["op"] == "extend":
        first, last = _rows(c["n"], c["base"], c["window"], "cuda")
        return _attend(c, x["q"], _held(c, x["kv"][0][0]), _held(c, x["kv"][1][0]), first, last, x["sinks"])
    if c["op"] == "append":
        out, out1 = [], []
        n = c["base"] + c["n"]
        for layer in range(c["layers"]):
            k, v = (_held(c, torch.cat([x["base"][i][layer], x["chunk"][i][layer], x["new"][i][layer]])) for i in (0, 1))
            first, last = _rows(c["n"], c["base"], 0, "cuda")
            out.append(_attend(c, x["q"][layer], k[:n], v[:n], first, last, x["sinks"]))
            first, last = _rows(1, n, 0, "cuda")
            out1.append(_attend(c, x["q1"][layer], k, v, first, last, x["sinks"]))
        return {"out": torch.stack(out), "out1": torch.stack(out1), **none}
    spans, chosen, _ = _spans(c)
    keep = torch.ones(c["length"], dtype=torch.bool, device="cuda")
    for i in chosen:
        keep[spans[i][0]:spans[i][1]] = False
    k, v = (_held(c, x["kv"][i][0][keep]) for i in (0, 1))
    first, last = _rows(1, k.shape[0] - 1, 0, "cuda")
    stats = {n: None for n, _ in sq.EvictStats._fields_}
    return {"stats": stats, "out": _attend(c, x["q"], k, v, first, last, x["sinks"]), **none}
