"""Performance cases of the paged multi-LoRA delta, through the public entry points of PagedLoraPool.

A case is one step of a serving program: translate the batch's token -> adapter map (batch_begin), add
the adapters' delta to the outputs of the projections of one or more transformer layers (delta, in the
slot ranges such a program has inputs for at a time), end the batch.  One case also replaces adapters
in the pool on the way.  A layer's projections are q, k, v, o and, where `ffn` is set, up and down; q, k,
v and up read the same hidden states.

Fields of a case
  dtype        element type of weights, x and y: bf16, fp16 or fp32
  layers, hidden, kv, ffn   projection shapes: q, o hidden -> hidden, k, v hidden -> kv, up / down (0 = none)
  calls        "layer": one call per layer; "inputs": one call for q, k, v and one for o (and one each for
               up and down), as a program calls that has o's input only after attention; "all": one call
  decode       tokens that are one request each (adapter drawn by Zipf over ids)
  prefill      tokens that come as whole requests of len_lo .. len_hi tokens
  none         share of the decode tokens without an adapter
  adapters, ranks, zipf, max_rank, page_kib   the resident set
  swap         adapters replaced (evict, load from page-locked memory) before each batch
"""
import math

import numpy as np
import torch

from paper_2512_20210_amd import binding as plora

DTYPES = {"fp16": (torch.float16, plora.PLORA_F16, 2), "bf16": (torch.bfloat16, plora.PLORA_BF16, 2),
          "fp32": (torch.float32, plora.PLORA_F32, 4)}


def _case(name=None, **kw):
    c = dict(dtype="bf16", layers=1, hidden=4096, kv=4096, ffn=0, calls="layer", decode=0, prefill=0, len_lo=64,
             len_hi=256, none=0.0, adapters=64, ranks="8,16,32,64", zipf=1.0, max_rank=64, page_kib=64, swap=0)
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: one 1024 -> 1024 projection, 16 decode tokens over 4 adapters; all latency
        _case("one_projection_16tok_fp16", dtype="fp16", hidden=1024, kv=0, calls="all", decode=16, adapters=4,
              ranks="8,16", zipf=0.0, max_rank=16, page_kib=16),
        # a handful of interactive users: 4 tokens through all layers of a 7B-shaped model, call by call
        _case("decode_4tok_32layers", layers=32, calls="inputs", decode=4, adapters=16, ranks="8,16,32,64"),
        # the usual decode step of a 7B-shaped model in a serving program: 256 tokens, 64 adapters,
        # layer by layer because each layer's input is the previous one's output
        _case("decode_256tok_32layers", layers=32, calls="inputs", decode=256),
        # the same step as one call over all 128 slots: the shape of bench.py's headline workload
        _case("decode_256tok_all_slots", layers=32, calls="all", decode=256),
        # grouped-query attention shapes (k, v 4096 -> 1024) in fp16, a ragged number of tokens, some
        # of them of the plain base model
        _case("decode_gqa_101tok_fp16", dtype="fp16", layers=32, kv=1024, calls="layer", decode=101, none=0.1,
              adapters=40, ranks="8,16,32,64"),
        # one 13B-shaped layer with its MLP, 1024 tokens over 1000 resident adapters: hardly any reuse of weights
        _case("decode_13b_layer_1000adapters", hidden=5120, kv=5120, ffn=13824, calls="layer", decode=1024,
              adapters=1000, ranks="16,32,64,128", zipf=0.8, max_rank=128, page_kib=128),
        # prefill of some 30 prompts of a 7B-shaped layer
        _case("prefill_5k_layer", calls="layer", prefill=5120, adapters=128, ranks="8,16,32,64,128", zipf=1.2, max_rank=128),
        # long prompts through a 13B-shaped layer with its MLP, fp16
        _case("prefill_16k_13b_layer_fp16", dtype="fp16", hidden=5120, kv=5120, ffn=13824, calls="inputs", prefill=16384,
              len_lo=512, len_hi=4096, adapters=32, ranks="16,32,64,128", zipf=1.0, max_rank=128, page_kib=128),
        # continuous batching on ragged shapes: a chunk of prefill next to decode tokens, arbitrary ranks,
        # projections that are no multiple of any tile
        _case("mixed_ragged_4layers", layers=4, hidden=2056, kv=520, calls="inputs", decode=93, prefill=900, len_lo=17,
              len_hi=300, none=0.2, adapters=48, ranks="3,5,12,20,33,48,77,100", max_rank=100),
        # fp32 adapters: a decode step and a prefill
        _case("decode_64tok_fp32", dtype="fp32", layers=8, hidden=2048, kv=2048, calls="inputs", decode=64, adapters=32),
        _case("prefill_2k_fp32", dtype="fp32", hidden=2048, kv=2048, calls="layer", prefill=2048, adapters=32),
        # churn: before every batch of 512 decode tokens two adapters of the batch are replaced in the pool
        _case("swap_2_decode_512tok", calls="layer", decode=512, adapters=256, ranks="4,8,16,32,64,128", max_rank=128, swap=2),
    ]


def _spread(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    most = max(work(c)["bytes"] for c in listed())
    while True:
        dtype = rng.choice(["bf16", "bf16", "bf16", "fp16", "fp16", "fp32"])
        hidden = 8 * _spread(rng, 96, 640)
        kv = hidden if rng.random() < 0.6 else 8 * max(16, hidden // 32)
        ffn = 8 * int(hidden * rng.uniform(2.0, 3.5) / 8) if rng.random() < 0.25 else 0
        kind = rng.choice(["decode", "decode", "prefill", "mixed"])
        ranks = rng.choice(["8,16", "8,16,32,64", "16,32,64,128", "3,5,12,20,33,48,77,100", "8,16,32,64,128"])
        c = _case(dtype=dtype, hidden=hidden, kv=kv, ffn=ffn, calls=rng.choice(["layer", "inputs", "inputs", "all"]),
                  layers=_spread(rng, 1, 32), decode=_spread(rng, 1, 1024) if kind != "prefill" else 0,
                  prefill=_spread(rng, 100, 16384) if kind != "decode" else 0,
                  none=rng.choice([0.0, 0.0, 0.1, 0.3]), adapters=_spread(rng, 2, 512), ranks=ranks,
                  zipf=rng.choice([0.0, 0.8, 1.0, 1.2]), max_rank=max(int(r) for r in ranks.split(",")),
                  page_kib=rng.choice([16, 64, 64, 128]))
        c["len_lo"] = _spread(rng, 1, 512)
        c["len_hi"] = c["len_lo"] * rng.choice([1, 2, 4, 8])
        weights = c["adapters"] * _mean_rank(c) * sum(a + b for a, b in _slots(c)) * DTYPES[dtype][2]
        if weights < 8e9 and work(c)["bytes"] <= most:
            return c


# ---- shapes -------------------------------------------------------------------------------------------

def _layer_slots(c):
    h, kv, f = c["hidden"], c["kv"], c["ffn"]
    if kv == 0:  # a single projection
        return [(h, h)]
    return [(h, h), (h, kv), (h, kv), (h, h)] + ([(h, f), (f, h)] if f else [])


def _slots(c):
    return _layer_slots(c) * c["layers"]


def _x_of(c):
    """For every projection of a layer, which of the layer's input buffers it reads."""
    n = len(_layer_slots(c))
    return {1: [0], 4: [0, 0, 0, 1], 6: [0, 0, 0, 1, 2, 3]}[n]


def _x_dims(c):
    n = len(_layer_slots(c))
    h, f = c["hidden"], c["ffn"]
    return {1: [h], 4: [h, h], 6: [h, h, h, f]}[n]


def _call_ranges(c):
    """(first slot, slots) of every delta call of a step."""
    per = len(_layer_slots(c))
    if c["calls"] == "all":
        return [(0, per * c["layers"])]
    if c["calls"] == "layer" or per == 1:
        return [(per * l, per) for l in range(c["layers"])]
    split = [(0, 3), (3, 1)] + ([(4, 1), (5, 1)] if per == 6 else [])
    return [(per * l + a, n) for l in range(c["layers"]) for a, n in split]


def _mean_rank(c):
    r = [int(v) for v in c["ranks"].split(",")]
    return sum(r) / len(r)


def _zipf(rng, n, s, size):
    p = (np.arange(n) + 1.0) ** -s
    return rng.choice(n, size=size, p=p / p.sum())


def _draw_batch(c, seed):
    """(rank of every adapter, token -> adapter map): host arrays, the sizes fixed by the case."""
    rng = np.random.default_rng(seed)
    ranks = rng.choice([int(v) for v in c["ranks"].split(",")], size=c["adapters"])
    parts = []
    left = c["prefill"]
    while left > 0:
        n = min(left, int(rng.integers(c["len_lo"], c["len_hi"] + 1)))
        parts.append(np.full(n, _zipf(rng, c["adapters"], c["zipf"], 1)[0]))
        left -= n
    d = _zipf(rng, c["adapters"], c["zipf"], c["decode"])
    if c["none"] > 0:
        d[rng.random(c["decode"]) < c["none"]] = -1
    parts.append(d)
    return ranks.astype(np.int64), np.concatenate(parts).astype(np.int32)


def work(case):
    """Every used adapter's weights read once, x read once, y read and written once, v written once (means over draws)."""
    elt = DTYPES[case["dtype"]][2]
    per_layer = _layer_slots(case)
    elems = sum(a + b for a, b in per_layer) * case["layers"]
    nbytes = flops = 0.0
    draws = 4
    for k in range(draws):
        ranks, t2a = _draw_batch(case, 1000 + k)
        used = np.unique(t2a[t2a >= 0])
        active = int((t2a >= 0).sum())
        nbytes += ranks[used].sum() * elems * elt
        nbytes += case["layers"] * active * elt * (sum(_x_dims(case)) + 2 * sum(b for _, b in per_layer))
        nbytes += case["layers"] * len(per_layer) * len(t2a) * case["max_rank"] * 4
        flops += 2.0 * ranks[t2a[t2a >= 0]].sum() * elems
    return {"bytes": nbytes / draws, "flops": flops / draws}


# ---- inputs -------------------------------------------------------------------------------------------

def _gen(seed, k):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + k) & 0x7FFFFFFFFFFF)
    return g


def _blob(c, seed, aid, rank):
    """Adapter `aid`'s weights on the GPU: slot after slot [A: rank x d_in | B: rank x d_out], A ~ N(0, 1/d_in), B ~ N(0, 1/rank)."""
    dt = DTYPES[c["dtype"]][0]
    per = _layer_slots(c)
    w = torch.randn(c["layers"], rank * sum(a + b for a, b in per), generator=_gen(seed, 16 + aid), device="cuda", dtype=dt)
    o = 0
    for a, b in per:
        w[:, o:o + rank * a] *= a ** -0.5
        o += rank * a
        w[:, o:o + rank * b] *= rank ** -0.5
        o += rank * b
    return w


def _scale(rank):
    return 16.0 / rank


def _activations(c, seed, n_tok):
    """x: per input buffer of a layer [layers, tokens, d_in]; y: per projection [layers, tokens, d_out] (what the base model left there)."""
    dt = DTYPES[c["dtype"]][0]
    x = [torch.randn(c["layers"], n_tok, d, generator=_gen(seed, i), device="cuda", dtype=dt) for i, d in enumerate(_x_dims(c))]
    y = [torch.randn(c["layers"], n_tok, b, generator=_gen(seed, 8 + i), device="cuda", dtype=dt)
         for i, (_, b) in enumerate(_layer_slots(c))]
    return x, y


class _State:
    def __init__(self, case, seed):
        c = self.case = case
        dt, code, elt = DTYPES[c["dtype"]]
        ranks, self.t2a = _draw_batch(c, seed)
        slots = _slots(c)
        elems = sum(a + b for a, b in slots)
        page = c["page_kib"] * 1024
        n_pages = int(sum(-(-int(r) * elems * elt // page) for r in ranks))
        self.pool = plora.PagedLoraPool(page, n_pages, [a for a, _ in slots], [b for _, b in slots], code, len(ranks),
                                        c["max_rank"])
        host = [torch.empty(int(ranks.max()) * elems, dtype=dt, pin_memory=True) for _ in range(2)]
        last = [None, None]
        for i, r in enumerate(ranks):
            k = i % 2
            if last[k] is not None:
                plora.plora_sync_adapter(self.pool.h, last[k])  # its page-locked buffer is free again
            w = _blob(c, seed, i, int(r)).reshape(-1)
            h = host[k][:w.numel()]
            h.copy_(w)
            self.pool.load(i, int(r), _scale(int(r)), h)
            last[k] = i
        for i in last:
            if i is not None:
                plora.plora_sync_adapter(self.pool.h, i)
        self.x, self.y = _activations(c, seed, len(self.t2a))
        self.v = torch.empty(len(slots), len(self.t2a), c["max_rank"], device="cuda", dtype=torch.float32)
        per, xo = len(_layer_slots(c)), _x_of(c)
        xs = [self.x[xo[s % per]][s // per] for s in range(len(slots))]
        ys = [self.y[s % per][s // per] for s in range(len(slots))]
        self.calls = [(a, xs[a:a + n], [self.v[s] for s in range(a, a + n)], ys[a:a + n]) for a, n in _call_ranges(c)]
        # adapters of the batch that are replaced before it, in turn, and their page-locked weights
        used = [int(i) for i in np.unique(self.t2a) if i >= 0]
        self.swap_ids = used[:8 * c["swap"]]
        self.swap_host = {}
        for i in self.swap_ids:
            h = torch.empty(int(ranks[i]) * elems, dtype=dt, pin_memory=True)
            h.copy_(_blob(c, seed, i, int(ranks[i])).reshape(-1))
            self.swap_host[i] = (int(ranks[i]), h)
        self.at = 0
        self.copy_stream = torch.cuda.Stream() if c["swap"] else None

    def __del__(self):
        if getattr(self, "pool", None) is not None:
            self.pool.close()


def prepare(case, seed):
    return _State(case, seed)


def run(s):
    pool = s.pool
    for _ in range(s.case["swap"]):
        i = s.swap_ids[s.at % len(s.swap_ids)]
        s.at += 1
        rank, h = s.swap_host[i]
        if not pool.ready(i):  # its last load is still on its way: nothing else can be evicted for it
            plora.plora_sync_adapter(pool.h, i)
        pool.evict(i)
        pool.load(i, rank, _scale(rank), h, s.copy_stream.cuda_stream)
    stream = torch.cuda.current_stream().cuda_stream
    b = pool.batch_begin(s.t2a, stream)
    for slot0, x, v, y in s.calls:
        pool.delta(b, slot0, x, v, y, stream)
    pool.batch_end(b)
    return {"y": s.y, "v": s.v}


# ---- what is right ------------------------------------------------------------------------------------

def tolerance(case):
    # About four times what was measured against exact().  The rounding of y to the element type decides for the
    # 16-bit types (2-norm: bf16 1.7e-3, fp16 2.1e-4; one ulp at most for a single value); fp32 pools and v (sums of
    # up to 13824 terms in fp32) show up to 2.6e-7.
    return {"bf16": {"rel": 7e-3, "max": 4e-2}, "fp16": {"rel": 9e-4, "max": 5e-3}, "fp32": {"rel": 1e-6, "max": 1e-5}}[case["dtype"]]


def exact(case, seed):
    c = case
    ranks, t2a = _draw_batch(c, seed)
    per, xo = _layer_slots(c), _x_of(c)
    x, y0 = _activations(c, seed, len(t2a))
    y = [t.double() for t in y0]
    v = torch.zeros(c["layers"] * len(per), len(t2a), c["max_rank"], device="cuda", dtype=torch.float64)
    for i in np.unique(t2a[t2a >= 0]):
        r = int(ranks[i])
        w = _blob(c, seed, int(i), r)
        tok = torch.from_numpy(np.nonzero(t2a == i)[0]).cuda()
        for l in range(c["layers"]):
            o = 0
            for s, (a, b) in enumerate(per):
                wa = w[l, o:o + r * a].double().view(r, a)
                wb = w[l, o + r * a:o + r * (a + b)].double().view(r, b)
                o += r * (a + b)
                vs = x[xo[s]][l][tok].double() @ wa.t()
                v[l * len(per) + s, tok, :r] = vs
                y[s][l].index_add_(0, tok, (vs @ wb) * _scale(r))
    return {"y": y, "v": v}
