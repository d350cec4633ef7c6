"""What is timed: the calls a serving program makes of this library, one layer (or a few) at a time.

Three kinds of work, each through the public entry points of paper_2512_17910_amd.binding:

  qkv    the masked multi-adapter QKV projection with the paged K/V write (alora_qkv_forward, _ex, _static, or the
         recorded graph), over `layers` layers that share one token batch: the first call groups the batch, the
         others reuse the grouping, as a model's layers do.  Decode-sized cases run four layers, each with weights
         of its own, because a model's next layer never finds its weights in the on-package cache.
  attn   the reader of the paged cache (alora_paged_attention, _split, _suffix or _suffix_split), one layer.
  turn   one layer of a turn of a conversation: the new tokens are projected, then attend over the cached context
         and over each other.

Shapes are those of the repository's configurations (8B: hidden 4096, 32 query / 8 K/V heads of 128; 70B: hidden
8192, 64 / 8 heads; the small fp32 layer) and one generic shape in between.  Requests are base-model ones, standard
LoRAs (active from their first token) and activated LoRAs whose activation point lies in or before the projected
rows, in the mixture of the configurations.  Values: x ~ N(0,1), W, A ~ N(0, 1/hidden), B ~ N(0, 1/rank),
q, K, V ~ N(0, 1).  A state is drawn on the GPU from the seed alone.
"""
import math

import numpy as np
import torch

from paper_2512_17910_amd import binding as ab

SHAPES = {              # hidden, query heads, K/V heads, head size
    "8b": (4096, 32, 8, 128),
    "70b": (8192, 64, 8, 128),
    "3b": (3072, 24, 8, 128),
    "small": (256, 4, 2, 64),
}
MAX_POS = 32768         # rows of the rotary tables a model of these shapes keeps


def listed():
    return [
        # one conversation is being answered: one token a step.  The smallest call: launches and the host count
        {"name": "qkv-decode-1", "kind": "qkv", "shape": "8b", "dtype": "bf16", "rows": 1, "seqs": 1, "adapters": 4, "rank": 32,
         "base": 0.0, "layers": 4, "rope": True, "bias": False, "mixed": False, "via": "static"},
        # a quiet server: a few dozen requests decode together, the layers replayed as recorded graphs (Sec. 3)
        {"name": "qkv-decode-37", "kind": "qkv", "shape": "8b", "dtype": "bf16", "rows": 37, "seqs": 37, "adapters": 8, "rank": 32,
         "base": 0.25, "layers": 4, "rope": True, "bias": False, "mixed": False, "via": "graph"},
        # a busy server: 256 requests decode together, a quarter of them base-model ones (configuration 3)
        {"name": "qkv-decode-256", "kind": "qkv", "shape": "8b", "dtype": "bf16", "rows": 256, "seqs": 256, "adapters": 16, "rank": 32,
         "base": 0.25, "layers": 4, "rope": False, "bias": False, "mixed": False, "via": "plain"},
        # a step of chunked prefill: a few ragged pieces of prompts, adapters of two ranks and a layer bias
        {"name": "qkv-chunk-777", "kind": "qkv", "shape": "8b", "dtype": "bf16", "rows": 777, "seqs": 5, "adapters": 8, "rank": 32,
         "base": 0.25, "layers": 2, "rope": True, "bias": True, "mixed": True, "via": "plain"},
        # a prefill step of 8 prompts (configuration 2)
        {"name": "qkv-prefill-4096", "kind": "qkv", "shape": "8b", "dtype": "bf16", "rows": 4096, "seqs": 8, "adapters": 8, "rank": 32,
         "base": 0.0, "layers": 1, "rope": False, "bias": False, "mixed": False, "via": "plain"},
        # the uncached suffixes of four long conversations, many adapters (configuration 5), rotary embedding fused
        {"name": "qkv-suffix-13757", "kind": "qkv", "shape": "8b", "dtype": "bf16", "rows": 13757, "seqs": 4, "adapters": 32, "rank": 16,
         "base": 0.0, "layers": 1, "rope": True, "bias": False, "mixed": False, "via": "plain"},
        # a large prefill step of the large model, activation near the end (configuration 4)
        {"name": "qkv-prefill-8192-70b", "kind": "qkv", "shape": "70b", "dtype": "bf16", "rows": 8192, "seqs": 4, "adapters": 4, "rank": 64,
         "base": 0.0, "layers": 1, "rope": False, "bias": False, "mixed": False, "via": "plain"},
        # reference precision: a small fp32 layer, projected and attended (configuration 1)
        {"name": "turn-f32-64", "kind": "turn", "shape": "small", "dtype": "f32", "rows": 64, "seqs": 2, "context": 32, "adapters": 2,
         "rank": 8, "rope": False},
        # decode attention of the busy server: 256 requests at contexts of 2 .. 2047 positions
        {"name": "attn-decode-256", "kind": "attn", "via": "row", "dtype": "bf16", "hq": 32, "hkv": 8, "d": 128, "bs": 16,
         "seqs": 256, "rows": 1, "ctx_lo": 2, "ctx_hi": 2047},
        # decode attention of a few long conversations (an adapter evaluated on each)
        {"name": "attn-decode-long-8", "kind": "attn", "via": "split", "dtype": "bf16", "hq": 32, "hkv": 8, "d": 128, "bs": 16,
         "seqs": 8, "rows": 1, "ctx_lo": 32768, "ctx_hi": 65536},
        # long uncached suffixes attend over a long cached prefix
        {"name": "attn-suffix-2048", "kind": "attn", "via": "suffix", "dtype": "bf16", "hq": 32, "hkv": 8, "d": 128, "bs": 16,
         "seqs": 4, "rows": 2048, "ctx_lo": 16384, "ctx_hi": 16384},
        # the turn the method is about: four requests each add a short invocation to a 16K conversation whose blocks
        # the base model wrote; 4 x 64 rows are projected and attend over the reused context
        {"name": "turn-4x64-16k", "kind": "turn", "shape": "8b", "dtype": "bf16", "rows": 256, "seqs": 4, "context": 16384, "adapters": 4,
         "rank": 32, "rope": True},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    u = rng.random()
    if u < 0.55:
        shape = rng.choice(["8b", "8b", "3b", "70b"])
        rows = _log_int(rng, 1, 8192 if shape == "70b" else 13757)
        decode = rows <= 256 and rng.random() < 0.7          # a row per sequence; otherwise pieces of prompts
        seqs = rows if decode else rng.randint(1, min(8, rows))
        via = "plain"
        if rows <= 64:
            via = rng.choice(["plain", "static", "graph"])
        return {"kind": "qkv", "shape": shape, "dtype": "bf16", "rows": rows, "seqs": seqs,
                "adapters": rng.choice([1, 2, 4, 8, 16, 32]), "rank": rng.choice([8, 16, 32, 64]),
                "base": rng.choice([0.0, 0.25, 0.5, 1.0]), "layers": 4 if rows <= 256 else 2 if rows <= 1024 else 1,
                "rope": rng.random() < 0.6, "bias": rng.random() < 0.3, "mixed": rng.random() < 0.3, "via": via}
    if u < 0.63:
        seqs = rng.randint(1, 4)
        return {"kind": "turn", "shape": "small", "dtype": "f32", "rows": seqs * _log_int(rng, 1, 128), "seqs": seqs,
                "context": rng.randint(128, 640), "adapters": rng.choice([1, 2, 4]), "rank": rng.choice([4, 8, 16]), "rope": rng.random() < 0.5}
    if u < 0.75:
        seqs = rng.randint(1, 8)
        return {"kind": "turn", "shape": rng.choice(["8b", "3b"]), "dtype": "bf16", "rows": seqs * _log_int(rng, 1, 256), "seqs": seqs,
                "context": _log_int(rng, 1024, 16384), "adapters": rng.choice([1, 4, 8]), "rank": rng.choice([16, 32]),
                "rope": rng.random() < 0.8}
    hkv = 8
    hq = hkv * rng.choice([1, 2, 4, 4, 8])
    via = rng.choice(["row", "split", "suffix", "suffix", "suffix_split", "suffix_split"])
    case = {"kind": "attn", "via": via, "dtype": "bf16", "hq": hq, "hkv": hkv, "d": 128, "bs": rng.choice([16, 16, 32, 64])}
    if via == "row":
        hi = rng.randint(64, 4096)
        case.update(seqs=_log_int(rng, 32, 256), rows=1, ctx_lo=rng.randint(1, hi), ctx_hi=hi)
    elif via == "split":
        hi = _log_int(rng, 2048, 65536)
        case.update(seqs=rng.randint(1, 12), rows=1, ctx_lo=hi // rng.randint(1, 3), ctx_hi=hi)
    elif via == "suffix":
        hi = _log_int(rng, 2048, 16384)
        case.update(seqs=rng.randint(1, 4), rows=_log_int(rng, 256, 2048), ctx_lo=max(2048, hi // rng.randint(1, 2)), ctx_hi=hi)
        if hq > 32:
            case["rows"] = min(case["rows"], 1024)
    else:
        hi = _log_int(rng, 1024, 32768)
        case.update(seqs=rng.randint(1, 6), rows=_log_int(rng, 1, 200), ctx_lo=max(256, hi // rng.randint(1, 3)), ctx_hi=hi)
    return case


# ---- inputs -------------------------------------------------------------------------------------
def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


class _Values:
    """Normally distributed tensors, one generator on the GPU."""

    def __init__(self, seed, dtype):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)
        self.dtype = torch.bfloat16 if dtype == "bf16" else torch.float32

    def __call__(self, shape, std=1.0):
        return torch.randn(shape, device="cuda", generator=self.g, dtype=torch.float32).mul_(std).to(self.dtype)


def _rope_tables():
    i = torch.arange(64, device="cuda", dtype=torch.float64)
    angle = torch.arange(MAX_POS, device="cuda", dtype=torch.float64)[:, None] * (10000.0 ** (-i / 64.0))[None, :]
    return torch.cos(angle).float(), torch.sin(angle).float()


def _cut(rng, total, parts):
    """`total` rows cut into `parts` ragged pieces, none empty."""
    cuts = np.sort(rng.choice(np.arange(1, total), size=parts - 1, replace=False)) if parts > 1 else np.zeros(0, np.int64)
    return np.diff(np.concatenate([[0], cuts, [total]])).astype(np.int64)


class _Batch:
    """The flattened token batch a scheduler hands over: rows of every sequence, who is adapted, where K/V go."""

    def __init__(self, rng, lens, first, adapters, base, start_of, bs=16):
        n = len(lens)
        owner = rng.integers(0, adapters, n)
        owner[rng.permutation(n)[: int(round(base * n))]] = -1
        start = np.array([start_of(int(f), int(l)) for f, l in zip(first, lens)], np.int32)
        seg = np.repeat(np.arange(n, dtype=np.int32), lens)
        pos = np.concatenate([np.arange(f, f + l) for f, l in zip(first, lens)]).astype(np.int32)
        # cache blocks: only those the batch's own rows fall into, dealt by a permutation (what lies in front of a
        # sequence's first row was written by earlier calls, and this call does not touch it)
        b0, b1 = first // bs, (first + lens - 1) // bs + 1
        perm = rng.permutation(int(lens.sum()) // bs + 2 * n + 2)      # (a size that the row count gives, with some blocks to spare)
        at = np.concatenate([[0], np.cumsum(b1 - b0)])[:-1]
        slot = perm[at[seg] + pos // bs - b0[seg]].astype(np.int64) * bs + pos % bs
        self.n_seqs, self.n_slots, self.bs = n, len(perm) * bs, bs
        self.aid_host, self.seg_host, self.pos_host, self.start_host = owner[seg].astype(np.int32), seg, pos, start
        self.aid, self.seg, self.pos, self.start, self.slot = (_dev(a) for a in (self.aid_host, seg, pos, start, slot))


class _Layer:
    def __init__(self, values, hidden, N, adapters, ranks, bias):
        self.W = values((hidden, N), hidden ** -0.5)
        self.A = [values((hidden, r), hidden ** -0.5) for r in ranks]
        self.B = [values((r, N), r ** -0.5) for r in ranks]
        self.bias = values((N,)) if bias else None


def _ranks(case):
    L, r = case["adapters"], case["rank"]
    return [r if (i % 2 == 0 or not case.get("mixed")) else 8 for i in range(L)]


class _Qkv:
    """`layers` projection calls over one batch."""

    def __init__(self, case, seed):
        rng = np.random.default_rng(seed)
        values = _Values(seed, case["dtype"])
        hidden, hq, hkv, d = SHAPES[case["shape"]]
        N, T, n = (hq + 2 * hkv) * d, case["rows"], case["seqs"]
        if T == n:          # decode: one row each, somewhere in its sequence, past the activation point
            lens, first = np.ones(n, np.int64), rng.integers(1, 2048, n)
            start_of = lambda f, l: int(rng.integers(0, f + 1))
        else:               # pieces of prompts: a LoRA is active from its first token on, an aLoRA from the last part of its piece on
            lens, first = _cut(rng, T, n), 16 * rng.integers(0, 512, n)
            start_of = lambda f, l: 0 if rng.random() < 0.25 else f + int(rng.integers((9 * l) // 10 if T > 6000 else l // 2, l + 1))
        self.batch = b = _Batch(rng, lens, first, case["adapters"], case["base"], start_of)
        ranks = _ranks(case)
        self.ranks = ranks if case["mixed"] else None
        self.layers = [_Layer(values, hidden, N, case["adapters"], ranks, case["bias"]) for _ in range(case["layers"])]
        self.x = values((T, hidden))
        self.rope = _rope_tables() if case["rope"] else None
        self.out = [tuple(torch.zeros(s, device="cuda", dtype=values.dtype) for s in ((T, hq * d), (b.n_slots, hkv * d), (b.n_slots, hkv * d)))
                    for _ in self.layers]
        self.dims = ab.make_dims(ab.ALORA_BF16 if case["dtype"] == "bf16" else ab.ALORA_F32, T, hidden, hq, hkv, d, case["adapters"],
                                 case["rank"], b.n_seqs, b.n_slots, b.seg, b.pos)
        self.via = case["via"]
        self.ws = None if self.via == "static" else ab.alloc_workspace(self.dims)
        self.plain = self.rope is None and self.ranks is None and not case["bias"] and case["layers"] == 1
        self.graphs = []
        if self.via == "graph":
            for y, (q, kc, vc) in zip(self.layers, self.out):
                self.graphs.append(ab.alora_qkv_graph_create(self.x, b.aid, b.start, y.W, y.A, y.B, q, kc, vc, b.slot, b.bs, self.dims,
                                                             self.ws, bias=y.bias, adapter_ranks=self.ranks, rope=self.rope))

    def __del__(self):
        for g in getattr(self, "graphs", ()):
            ab.alora_qkv_graph_destroy(g)

    def run(self):
        b = self.batch
        if self.via == "graph":
            for g in self.graphs:
                ab.alora_qkv_graph_launch(g)
            return self.out
        for i, (y, (q, kc, vc)) in enumerate(zip(self.layers, self.out)):
            if self.via == "static":
                ab.alora_qkv_forward_static(self.x, b.aid, b.start, y.W, y.A, y.B, q, kc, vc, b.slot, b.bs, self.dims, bias=y.bias,
                                            adapter_ranks=self.ranks, rope=self.rope)
            elif self.plain:
                ab.alora_qkv_forward(self.x, b.aid, b.start, y.W, y.A, y.B, q, kc, vc, b.slot, b.bs, self.dims, self.ws)
            else:
                ab.alora_qkv_forward_ex(self.x, b.aid, b.start, y.W, y.A, y.B, q, kc, vc, b.slot, b.bs, self.dims, self.ws, bias=y.bias,
                                        adapter_ranks=self.ranks, rope=self.rope, reuse_grouping=i > 0)
        return self.out


def _lens(case, rng):
    return rng.integers(case["ctx_lo"], case["ctx_hi"] + 1, case["seqs"])


class _Reader:
    """One call of the cache reader: the last `rows` positions of every sequence are query rows."""

    def __init__(self, via, values, rng, lens, rows, hq, hkv, d, bs, kv=None):
        n = len(lens)
        nb = (lens + bs - 1) // bs
        self.table = np.full((n, int(nb.max())), -1, np.int32)
        perm, at = rng.permutation(int(nb.sum())).astype(np.int32), 0
        for s in range(n):
            self.table[s, : nb[s]] = perm[at: at + nb[s]]
            at += int(nb[s])
        rows = np.minimum(rows, lens)
        self.seq_host = np.repeat(np.arange(n, dtype=np.int32), rows)
        self.pos_host = np.concatenate([np.arange(l - r, l, dtype=np.int32) for l, r in zip(lens, rows)])
        self.kc, self.vc = (values((len(perm) * bs, hkv * d)) for _ in range(2))
        self.q = values((len(self.seq_host), hq * d))
        self.out = torch.empty_like(self.q)
        self.bt, self.seq, self.pos = _dev(self.table), _dev(self.seq_host), _dev(self.pos_host)
        self.dims = ab.make_attn_dims(self.q, self.kc, self.bt, hq, hkv, d, bs)
        self.call = {"row": ab.alora_paged_attention, "split": ab.alora_paged_attention_split, "suffix": ab.alora_paged_attention_suffix,
                     "suffix_split": ab.alora_paged_attention_suffix_split}[via]
        self.more = ()
        if via in ("split", "suffix_split"):
            size = (ab.alora_paged_attention_workspace_bytes if via == "split" else ab.alora_paged_attention_suffix_workspace_bytes)(self.dims)
            self.more = (torch.empty(max(size, 16), dtype=torch.uint8, device="cuda"),)

    def run(self):
        self.call(self.q, self.kc, self.vc, self.bt, self.seq, self.pos, self.out, self.dims, *self.more)
        return self.out


class _Turn:
    """One layer of a turn: project the new rows (into the cache that holds the context), then attend."""

    def __init__(self, case, seed):
        rng = np.random.default_rng(seed)
        values = _Values(seed, case["dtype"])
        hidden, hq, hkv, d = SHAPES[case["shape"]]
        T, n, C, bs = case["rows"], case["seqs"], case["context"], 16
        each = T // n
        C = max(C, each)
        self.reader = r = _Reader("suffix_split" if case["dtype"] == "bf16" else "row", values, rng, np.full(n, C), each, hq, hkv, d, bs)
        self.slot = _dev(r.table[r.seq_host, r.pos_host // bs].astype(np.int64) * bs + r.pos_host % bs)
        self.aid = _dev((r.seq_host % case["adapters"]).astype(np.int32))
        # the invocation is the new rows: every one of them is adapted (fp32 layer: the last quarter)
        first = C - each if case["dtype"] == "bf16" else C - (each + 3) // 4
        self.start = _dev(np.full(n, first, np.int32))
        self.layer = _Layer(values, hidden, (hq + 2 * hkv) * d, case["adapters"], [case["rank"]] * case["adapters"], False)
        self.x = values((T, hidden))
        self.rope = None
        if case["rope"]:
            cos, sin = _rope_tables()
            self.rope = (cos[:, : d // 2].contiguous(), sin[:, : d // 2].contiguous())
        self.dims = ab.make_dims(ab.ALORA_BF16 if case["dtype"] == "bf16" else ab.ALORA_F32, T, hidden, hq, hkv, d, case["adapters"],
                                 case["rank"], n, r.kc.shape[0], r.seq, r.pos)
        self.ws = ab.alloc_workspace(self.dims)
        self.bs = bs

    def run(self):
        r, y = self.reader, self.layer
        ab.alora_qkv_forward_ex(self.x, self.aid, self.start, y.W, y.A, y.B, r.q, r.kc, r.vc, self.slot, self.bs, self.dims, self.ws, rope=self.rope)
        return {"attention": r.run(), "q": r.q, "k_cache": r.kc, "v_cache": r.vc}


def prepare(case, seed):
    if case["kind"] == "qkv":
        return _Qkv(case, seed)
    if case["kind"] == "turn":
        return _Turn(case, seed)
    rng = np.random.default_rng(seed)
    return _Reader(case["via"], _Values(seed, case["dtype"]), rng, _lens(case, rng), case["rows"], case["hq"], case["hkv"], case["d"], case["bs"])


def run(state):
    return state.run()


# ---- what a pass cannot do without --------------------------------------------------------------
def _qkv_work(hidden, N, Nq, T, T_act, used, rank, e):
    flops = 2.0 * T * hidden * N + 2.0 * T_act * rank * (hidden + N)
    data = e * (T * hidden + hidden * N + used * rank * (hidden + N) + T * N) + T * 20
    return data, flops


def work(case):
    e = 2 if case["dtype"] == "bf16" else 4
    if case["kind"] == "attn":
        # expected values of the drawn contexts: the cached rows of every sequence once, 4 flops per (query head, position, element)
        mean, n, width = (case["ctx_lo"] + case["ctx_hi"]) / 2, case["seqs"], case["hkv"] * case["d"]
        rows = min(case["rows"], mean)
        return {"bytes": e * (2 * n * mean * width + 2 * n * rows * case["hq"] * case["d"]),
                "flops": 4.0 * n * rows * (mean - (rows - 1) / 2) * case["hq"] * case["d"]}
    hidden, hq, hkv, d = SHAPES[case["shape"]]
    N, Nq, T = (hq + 2 * hkv) * d, hq * d, case["rows"]
    if case["kind"] == "turn":
        n, C = case["seqs"], max(case["context"], T // case["seqs"])
        act = T if case["dtype"] == "bf16" else n * ((T // n + 3) // 4)
        data, flops = _qkv_work(hidden, N, Nq, T, act, min(case["adapters"], n), case["rank"], e)
        rows = T // n
        return {"bytes": data + e * (2 * n * (C - rows) * hkv * d + T * Nq),       # the call's own q, K, V need not come back from memory
                "flops": flops + 4.0 * n * rows * (C - (rows - 1) / 2) * hq * d}
    adapted = 1.0 - case["base"]
    act = T * adapted * (1.0 if T == case["seqs"] else 0.44 if T <= 6000 else 0.29)     # expected share of active rows
    used = min(case["adapters"], max(1.0, case["seqs"] * adapted)) if adapted else 0.0
    rank = sum(_ranks(case)) / len(_ranks(case))
    data, flops = _qkv_work(hidden, N, Nq, T, act, used, rank, e)
    return {"bytes": case["layers"] * data, "flops": case["layers"] * flops}


def tolerance(case):
    # About four times what the path shows against the same computation in fp64: fp32 2.7e-7 in the 2-norm (sums in
    # another order); bf16 1.7e-3, largest 3.9e-3 (one rounding to bf16); readers 2.3e-3, largest 9.4e-3 (the suffix
    # reader's softmax weights are bf16 too).
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 2e-5}
    if case["kind"] == "qkv":
        return {"rel": 7e-3, "max": 1.6e-2}
    return {"rel": 1e-2, "max": 4e-2}
