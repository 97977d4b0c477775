"""The workloads whose time is followed: what a serving or evaluation program has this library do.

Geometry throughout: GQA 32:4 with D = 128 unless a case says otherwise, spans of about sqrt(L) tokens,
random inputs of the scale that the search and the softmax meet (unit variance for the joint softmax, a
third of that where the raw search scores gate the spans, so that the gate spreads over several of them).
Every call goes through paper_2601_18401_amd.binding as a program calls it: outputs are allocated by the
call, the scratch is the binding's own workspace.
"""
import math

import torch

from paper_2601_18401_amd import binding as B

DEV = "cuda"

# one entry per kind of call; sizes in tokens
_LISTED = [
    # one decode step against a short, odd-sized cache: launches and latency are everything
    {"name": "decode_16k", "kind": "decode", "form": "joint", "dtype": "bf16", "L": 16411, "Hq": 32, "Hkv": 4, "D": 128,
     "S": 128, "topk": 8, "std": 1.0},
    # the headline decode step: a million tokens, sixteen spans of 1024
    {"name": "decode_1m", "kind": "decode", "form": "joint", "dtype": "bf16", "L": 1048576, "Hq": 32, "Hkv": 4, "D": 128,
     "S": 1024, "topk": 16, "std": 1.0},
    # the longest cache: ten million tokens, spans of 4096
    {"name": "decode_10m", "kind": "decode", "form": "joint", "dtype": "bf16", "L": 10485760, "Hq": 32, "Hkv": 4, "D": 128,
     "S": 4096, "topk": 16, "std": 1.0},
    # one decode step on the paper's own stride pattern with its kernel configuration, gated
    {"name": "anchor_decode_1m", "kind": "anchor_decode", "dtype": "bf16", "L": 1000003, "Hq": 32, "Hkv": 4, "D": 128,
     "topk": 2, "window": 1088, "back": 4, "fwd": 2, "root": 2, "std": 0.35},
    # a serving batch: eight sequences, from 300000 tokens down to a fifth of that, one step for all
    {"name": "decode_batch", "kind": "decode_batch", "form": "joint", "dtype": "bf16", "B": 8, "L": 300007, "Hq": 32,
     "Hkv": 4, "D": 128, "S": 512, "topk": 16, "std": 1.0},
    # span-search of a 64K prompt
    {"name": "search_64k", "kind": "search", "dtype": "bf16", "L": 65536, "Lq": 65536, "Hq": 32, "Hkv": 4, "D": 128,
     "S": 256, "topk": 8, "std": 1.0, "scores": False},
    # span-attention of a 256K prompt with planted needle spans: the largest prefill
    {"name": "prefill_256k", "kind": "prefill", "form": "joint", "dtype": "bf16", "L": 262144, "Lq": 262144, "Hq": 32,
     "Hkv": 4, "D": 128, "S": 512, "A": 512, "topk": 8, "std": 1.0, "needles": 16},
    # chunked prefill while serving: 4000 new rows behind a cache of 196000 tokens, gated, sixteen spans
    {"name": "prefill_chunk", "kind": "prefill", "form": "gated", "dtype": "bf16", "L": 200000, "Lq": 4000, "Hq": 32,
     "Hkv": 4, "D": 128, "S": 512, "A": 512, "topk": 16, "std": 0.35, "needles": 0},
    # span-search of a prompt on the paper's own stride pattern (the gate wants the scores)
    {"name": "anchor_search_48k", "kind": "anchor_search", "dtype": "bf16", "L": 49157, "Lq": 49157, "Hq": 32, "Hkv": 4,
     "D": 128, "topk": 2, "window": 1088, "back": 4, "fwd": 2, "root": 2, "std": 0.35},
    # span-attention of that prompt
    {"name": "anchor_prefill_48k", "kind": "anchor_prefill", "dtype": "bf16", "L": 49157, "Lq": 49157, "Hq": 32, "Hkv": 4,
     "D": 128, "topk": 2, "window": 1088, "back": 4, "fwd": 2, "root": 2, "std": 0.35},
    # a small model in fp32 (D = 64): what evaluations in full precision run
    {"name": "prefill_fp32", "kind": "prefill", "form": "joint", "dtype": "f32", "L": 4096, "Lq": 4096, "Hq": 4, "Hkv": 4,
     "D": 64, "S": 64, "A": 64, "topk": 4, "std": 1.0, "needles": 0},
    # a prompt whose span length is simply ceil(sqrt(L)), no multiple of anything
    {"name": "prefill_sqrt", "kind": "prefill", "form": "joint", "dtype": "bf16", "L": 20011, "Lq": 20011, "Hq": 32,
     "Hkv": 4, "D": 128, "S": 142, "A": 142, "topk": 8, "std": 1.0, "needles": 0},
]


def listed():
    return [dict(c) for c in _LISTED]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "anchor_decode", "decode_batch", "search", "prefill", "prefill", "prefill_chunk",
                       "anchor_search", "anchor_prefill", "prefill_fp32", "prefill_sqrt"])
    Hkv = rng.choice([2, 4, 4, 8])
    G = rng.choice([4, 8, 8]) if Hkv < 8 else 4
    heads = {"Hq": G * Hkv, "Hkv": Hkv, "D": 128}
    form = rng.choice(["joint", "joint", "gated"])
    if kind == "decode":
        L = _log_int(rng, 4000, 4000000)
        S = 64 * max(1, round(math.sqrt(L) / 64)) if rng.random() < 0.6 else math.ceil(math.sqrt(L))
        dt, D = rng.choice([("bf16", 128), ("bf16", 128), ("bf16", 64), ("f32", 128)])
        return {"kind": "decode", "form": form, "dtype": dt, "L": L, **heads, "D": D, "S": S, "topk": rng.choice([4, 8, 16]),
                "std": 1.0 if form == "joint" else 0.35}
    if kind == "anchor_decode":
        return {"kind": kind, "dtype": "bf16", "L": _log_int(rng, 4000, 4000000), **heads, "topk": rng.choice([1, 2, 3, 4]),
                "window": rng.choice([255, 1088]), "back": rng.choice([2, 3, 4]), "fwd": rng.choice([0, 1, 2]), "root": 2,
                "std": 0.35}
    if kind == "decode_batch":
        L = _log_int(rng, 8000, 400000)
        return {"kind": kind, "form": form, "dtype": "bf16", "B": rng.choice([2, 4, 7, 8]), "L": L, **heads,
                "S": 64 * max(1, round(math.sqrt(L) / 64)), "topk": rng.choice([8, 16]), "std": 1.0 if form == "joint" else 0.35}
    if kind in ("search", "prefill"):
        L = _log_int(rng, 3000, 130000)
        S = 64 * max(1, round(math.sqrt(L) / 64))
        Lq = L if rng.random() < 0.5 else rng.randint(L // 4, L)
        c = {"dtype": "bf16", "L": L, "Lq": Lq, **heads, "S": S, "topk": rng.choice([2, 4, 8, 8, 12]), "std": 1.0}
        if kind == "search":
            return {"kind": kind, **c, "scores": rng.random() < 0.5}
        # one in four: the redundant grid, spans that overlap by half
        A = S // 2 if rng.random() < 0.25 and S % 128 == 0 else S
        return {"kind": kind, "form": form, **c, "A": A, "std": 1.0 if form == "joint" else 0.35, "needles": rng.choice([0, 0, 12])}
    if kind == "prefill_chunk":
        L = _log_int(rng, 20000, 300000)
        S = 64 * max(1, round(math.sqrt(L) / 64))
        return {"kind": "prefill", "form": form, "dtype": "bf16", "L": L, "Lq": _log_int(rng, 256, 8192), **heads, "S": S,
                "A": S, "topk": rng.choice([8, 16]), "std": 1.0 if form == "joint" else 0.35, "needles": 0}
    if kind in ("anchor_search", "anchor_prefill"):
        L = _log_int(rng, 3000, 49000)
        Lq = L if rng.random() < 0.5 else rng.randint(L // 4, L)
        return {"kind": kind, "dtype": "bf16", "L": L, "Lq": Lq, **heads, "topk": rng.choice([1, 2, 3, 4]),
                "window": rng.choice([255, 1088]), "back": rng.choice([2, 3, 4]), "fwd": rng.choice([0, 1, 2]), "root": 2,
                "std": 0.35}
    if kind == "prefill_fp32":
        L = rng.randint(1500, 6000)
        S = rng.choice([64, math.ceil(math.sqrt(L))])
        c = {"dtype": "f32", "L": L, "Lq": L, "Hq": 4, "Hkv": rng.choice([1, 2, 4]), "D": rng.choice([64, 64, 128]), "S": S,
             "topk": rng.choice([2, 4, 8]), "std": 1.0}
        if rng.random() < 0.25:
            return {"kind": "search", **c, "scores": False}
        return {"kind": "prefill", "form": form, **c, "A": S, "std": 1.0 if form == "joint" else 0.35, "needles": 0}
    L = _log_int(rng, 2500, 20000)  # spans of ceil(sqrt(L)) tokens
    S = math.ceil(math.sqrt(L))
    return {"kind": "prefill", "form": form, "dtype": "bf16", "L": L, "Lq": L, **heads, "D": rng.choice([64, 128, 128]), "S": S,
            "A": S, "topk": rng.choice([4, 8]), "std": 1.0 if form == "joint" else 0.35, "needles": 0}


# ------------------------------------------------------------------------------------------ inputs

def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _randn(shape, gen, dtype, std):
    out = torch.empty(shape, dtype=dtype, device=DEV)
    step = 1 << 20
    for h in range(shape[0]):
        for t0 in range(0, shape[1], step):
            t1 = min(shape[1], t0 + step)
            out[h, t0:t1] = (torch.randn((t1 - t0, shape[2]), generator=gen, device=DEV) * std).to(dtype)
    return out


def _qkv(case, seed, L=None):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    L = case["L"] if L is None else L
    Lq = case.get("Lq", 1)
    dt, std, Hkv, D = _dtype(case), case["std"], case["Hkv"], case["D"]
    Q = _randn((case["Hq"], Lq, D), gen, dt, std)
    K = _randn((Hkv, L, D), gen, dt, std)
    V = _randn((Hkv, L, D), gen, dt, 1.0)
    if case.get("needles"):
        # spans whose keys lie close to one direction that every query of the group leans to
        S, G = case["S"], case["Hq"] // Hkv
        u = torch.randn((Hkv, D), generator=gen, device=DEV)
        for j in torch.randperm(max(1, L // S), generator=gen, device=DEV)[: case["needles"]].tolist():
            noise = torch.randn((Hkv, S, D), generator=gen, device=DEV)
            K[:, j * S:(j + 1) * S] = (std * (4.0 * u[:, None, :] + 0.1 * noise)).to(dt)
        for h in range(case["Hq"]):
            Q[h] = (Q[h].float() + std * u[h // G]).to(dt)
    return gen, Q, K, V


def _grid_selection(case, Q, K):
    """(idx, scores) of the top-k spans of every row, ascending, -1 / 0 in empty slots: what a search returned."""
    Hq, Lq, _ = Q.shape
    A, k, L, q0 = case["A"], case["topk"], case["L"], case["L"] - Q.shape[1]
    G, n = Hq // case["Hkv"], L // A
    idx = torch.full((Hq, Lq, k), -1, dtype=torch.int32, device=DEV)
    sc = torch.zeros((Hq, Lq, k), dtype=torch.float32, device=DEV)
    if n == 0:
        return idx, sc
    spans = torch.arange(n, device=DEV)
    kk = min(k, n)
    rows = max(1, (1 << 26) // n)
    for h in range(Hq):
        keys = K[h // G, A - 1:n * A:A].float()
        for r0 in range(0, Lq, rows):
            r1 = min(Lq, r0 + rows)
            c = (q0 + torch.arange(r0, r1, device=DEV)) // A
            s = Q[h, r0:r1].float() @ keys.t()
            s.masked_fill_(spans[None, :] >= c[:, None], -math.inf)
            v, j = torch.topk(s, kk, dim=1)
            j = torch.where(torch.isinf(v), n + 1, j)
            j, order = torch.sort(j, dim=1)
            v = torch.gather(v, 1, order)
            empty = j > n
            idx[h, r0:r1, :kk] = torch.where(empty, -1, j).to(torch.int32)
            sc[h, r0:r1, :kk] = torch.where(empty, 0.0, v)
    return idx, sc


def _anchor_selection(case, gen, Hq, Lq, q0):
    """Anchors and gate logits per row: distinct stride indices, nearest first, spread as random scores spread them."""
    k, s0 = case["topk"], math.isqrt(case["window"])
    an = torch.full((Hq, Lq, k), -1, dtype=torch.int32, device=DEV)
    sc = torch.zeros((Hq, Lq, k), dtype=torch.float32, device=DEV)
    i = q0 + torch.arange(Lq, device=DEV)
    smax = torch.sqrt((i + 1).double()).floor().long()  # (s+1)^2 <= i+1
    smax = smax - (smax * smax > i + 1).long() - 1
    c = (smax - s0 + 1).clamp(min=0)
    for h in range(Hq):
        u = torch.rand((Lq, k), generator=gen, device=DEV).sort(dim=1).values
        j = (u * (c - k + 1).clamp(min=1)[:, None]).long() + torch.arange(k, device=DEV)[None, :]
        t = i[:, None] - (s0 + j + 1) ** 2 + 1
        ok = (j < c[:, None]) & (t >= 0)
        an[h] = torch.where(ok, t, -1).to(torch.int32)
        sc[h] = torch.where(ok, torch.randn((Lq, k), generator=gen, device=DEV), 0.0)
    return an, sc


def _batch_lengths(case):
    L, nb = case["L"], case["B"]
    return [max(1, L - (4 * L * b) // (5 * max(1, nb - 1)) - 3 * b) for b in range(nb)]


def prepare(case, seed):
    st = {"case": case}
    kind = case["kind"]
    if kind == "decode_batch":
        Q, K, V, Ks = [], [], [], []
        for b, Lb in enumerate(_batch_lengths(case)):
            _, q, k, v = _qkv(case, seed * 64 + b, L=Lb)
            Q.append(q), K.append(k), V.append(v), Ks.append(B.sl_span_keys(k, case["S"]))
        st["batch"] = B.DecodeBatch(Q, Q, K, V, Ks, case["S"], case["topk"], want_scores=case["form"] == "gated")
        return st
    gen, st["Q"], st["K"], st["V"] = _qkv(case, seed)
    if kind in ("decode", "search"):
        st["Ks"] = B.sl_span_keys(st["K"], case["S"])
    elif kind == "prefill":
        st["idx"], st["scores"] = _grid_selection(case, st["Q"], st["K"])
    elif kind == "anchor_prefill":
        st["idx"], st["scores"] = _anchor_selection(case, gen, case["Hq"], case["Lq"], case["L"] - case["Lq"])
    return st


# ------------------------------------------------------------------------------------------ one pass

def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "decode_batch":
        b = state["batch"]
        if c["form"] == "gated":
            idx, sc = B.sl_span_search_decode_batched(b)
            return {"idx": idx, "scores": sc, "O": B.sl_span_attention_combined_decode_batched(b)}
        idx = B.sl_span_search_decode_batched(b)
        O, LSE = B.sl_span_attention_decode_batched(b)
        return {"idx": idx, "O": O, "LSE": LSE}
    Q, K, V = state["Q"], state["K"], state["V"]
    if kind == "decode":
        if c["form"] == "gated":
            idx, sc = B.sl_span_search_decode(Q, K, state["Ks"], c["S"], c["topk"], want_scores=True)
            return {"idx": idx, "scores": sc, "O": B.sl_span_attention_combined_decode(Q, K, V, idx, sc, c["S"])}
        idx = B.sl_span_search_decode(Q, K, state["Ks"], c["S"], c["topk"])
        O, LSE = B.sl_span_attention_decode(Q, K, V, idx, c["S"])
        return {"idx": idx, "O": O, "LSE": LSE}
    if kind == "anchor_decode":
        an, sc = B.sl_anchor_search_decode(Q, K, c["topk"], c["window"], want_scores=True, search_root=c["root"])
        O = B.sl_anchor_attention_decode(Q, K, V, an, sc, c["window"], c["back"], c["fwd"], search_root=c["root"])
        return {"idx": an, "scores": sc, "O": O}
    q0 = c["L"] - Q.shape[1]
    if kind == "search":
        r = B.sl_span_search_prefill(Q, K, state["Ks"], c["S"], c["topk"], q_pos0=q0, want_scores=c["scores"])
        return {"idx": r[0], "scores": r[1]} if c["scores"] else {"idx": r}
    if kind == "anchor_search":
        an, sc = B.sl_anchor_search_prefill(Q, K, c["topk"], c["window"], q_pos0=q0, want_scores=True, search_root=c["root"])
        return {"idx": an, "scores": sc}
    if kind == "anchor_prefill":
        return {"O": B.sl_anchor_attention_prefill(Q, K, V, state["idx"], state["scores"], c["window"], c["back"], c["fwd"],
                                                   q_pos0=q0, search_root=c["root"])}
    stride = 0 if c["A"] == c["S"] else c["A"]
    if c["form"] == "gated":
        return {"O": B.sl_span_attention_combined_prefill(Q, K, V, state["idx"], state["scores"], c["S"], q_pos0=q0,
                                                          span_stride=stride)}
    O, LSE = B.sl_span_attention_prefill(Q, K, V, state["idx"], c["S"], q_pos0=q0, span_stride=stride)
    return {"O": O, "LSE": LSE}


# ------------------------------------------------------------------------------------------ what a pass cannot do without

def _decode_work(c, L):
    """One decode step: the distinct rows that the heads of a group attend, read once, and the span keys."""
    e = 4 if c["dtype"] == "f32" else 2
    G, D = c["Hq"] // c["Hkv"], c["D"]
    n = (L - 1) // c["S"]
    k = min(c["topk"], n)
    distinct = n * (1 - (1 - k / n) ** G) if n else 0.0
    rows = c["Hkv"] * (distinct * c["S"] + (L - 1) % c["S"] + 1)
    pairs = c["Hq"] * (k * c["S"] + (L - 1) % c["S"] + 1)
    byts = rows * 2 * D * e + c["Hkv"] * n * D * e + 2 * c["Hq"] * D * e + c["Hq"] * (c["topk"] + 1) * 4
    return byts, pairs * 4 * D + c["Hq"] * n * 2 * D


def work(case):
    c, kind = case, case["kind"]
    e = 4 if c["dtype"] == "f32" else 2
    Hq, Hkv, D, L = c["Hq"], c["Hkv"], c["D"], c["L"]
    if kind == "decode":
        b, f = _decode_work(c, L)
        return {"bytes": b, "flops": f}
    if kind == "decode_batch":
        w = [_decode_work(c, Lb) for Lb in _batch_lengths(c)]
        return {"bytes": sum(x[0] for x in w), "flops": sum(x[1] for x in w)}
    s0 = math.isqrt(c["window"]) if "window" in c else 0
    if kind == "anchor_decode":
        n = max(0, math.isqrt(L) - s0)
        span = min(L, (c["back"] + c["fwd"]) * math.isqrt(L) + 1)
        k, w = min(c["topk"], n), min(L, c["window"])
        pairs = Hq * (k * span + w)
        rows = min(pairs, Hkv * L)
        return {"bytes": (Hq * k * span + Hkv * w if rows == pairs else rows) * 2 * D * e + Hkv * n * D * e + 2 * Hq * D * e,
                "flops": pairs * 4 * D + Hq * n * 2 * D}
    Lq = c.get("Lq", L)
    q0 = L - Lq
    step = max(1, Lq // 4096)
    pos = range(q0, L, step)
    if kind in ("anchor_search", "anchor_prefill"):
        cand = sum(max(0, math.isqrt(i + 1) - s0) for i in pos) / len(pos)
        if kind == "anchor_search":
            return {"bytes": Hq * Lq * D * e + Hkv * L * D * e + Hq * Lq * c["topk"] * 8, "flops": Hq * Lq * cand * 2 * D}
        att = sum(min(i + 1, min(i + 1, c["window"]) + (min(c["topk"], max(0, math.isqrt(i + 1) - s0))
                                                        * ((c["back"] + c["fwd"]) * math.isqrt(i) + 1))) for i in pos) / len(pos)
        return {"bytes": 2 * Hq * Lq * D * e + 2 * Hkv * L * D * e + Hq * Lq * c["topk"] * 8, "flops": Hq * Lq * att * 4 * D}
    A = c.get("A", c["S"])
    cand = sum(i // A for i in pos) / len(pos)
    att = sum(min(i + 1, min(c["topk"], i // A) * c["S"] + i % A + 1) for i in pos) / len(pos)
    if kind == "search":
        return {"bytes": Hq * Lq * D * e + Hkv * (L // A) * D * e + Hq * Lq * c["topk"] * (8 if c["scores"] else 4),
                "flops": Hq * Lq * cand * 2 * D}
    gated = c.get("form") == "gated"
    byts = 2 * Hq * Lq * D * e + 2 * Hkv * L * D * e + Hq * Lq * (c["topk"] * (8 if gated else 4) + (0 if gated else 4))
    return {"bytes": byts, "flops": Hq * Lq * att * 4 * D}


def tolerance(case):
    if case["kind"] in ("search", "anchor_search"):
        # Scores of exact products summed in 32 bits: 5e-8 off.  About one row in a million has its k-th and
        # next score closer than that; where it turns, the row's list shifts, which shows as 1.5e-5 over all scores.
        return {"rel": 1e-4, "max": 0.99, "differ": 1e-4}
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3, "differ": 1e-4}  # sums of 32-bit products in another order (2e-7 seen)
    # outputs rounded to bf16 (1.7e-3 seen), weights and partial outputs too on the matrix cores (2.5e-3 seen)
    return {"rel": 1e-2, "max": 0.1, "differ": 1e-4}


# ------------------------------------------------------------------------------------------ in 64 bits, plain torch

class _Rows:
    """Online softmax state of many rows: m, l [rows], o [rows, D] in 64 bits."""

    def __init__(self, rows, D):
        self.m = torch.full((rows,), -math.inf, dtype=torch.float64, device=DEV)
        self.l = torch.zeros((rows,), dtype=torch.float64, device=DEV)
        self.o = torch.zeros((rows, D), dtype=torch.float64, device=DEV)

    def add(self, at, q, k, v, scale, lo=None, hi=None, t0=0):
        """Rows `at` (each once) attend the keys k, v at tokens t0, t0 + 1, ...; lo, hi: a row's own range."""
        z = (q @ k.t()) * scale
        if lo is not None:
            t = t0 + torch.arange(k.shape[0], device=DEV)
            z.masked_fill_((t[None, :] < lo[:, None]) | (t[None, :] >= hi[:, None]), -math.inf)
        m0 = self.m[at]
        m = torch.maximum(m0, z.amax(dim=1))
        safe = torch.where(torch.isinf(m), 0.0, m)
        p = torch.exp(z - safe[:, None])
        f = torch.exp(m0 - safe)
        self.m[at] = m
        self.l[at] = self.l[at] * f + p.sum(dim=1)
        self.o[at] = self.o[at] * f[:, None] + p @ v

    def merged(self, other):
        m = torch.maximum(self.m, other.m)
        safe = torch.where(torch.isinf(m), 0.0, m)
        a, b = torch.exp(self.m - safe), torch.exp(other.m - safe)
        r = _Rows(0, self.o.shape[1])
        r.m, r.l, r.o = m, self.l * a + other.l * b, self.o * a[:, None] + other.o * b[:, None]
        return r


def _decode_exact(c, Q, K, V, L, anchor):
    """One decode step of one sequence: (scores [Hq, 1, k], O [Hq, 1, D], LSE [Hq, 1])."""
    Hq, D, k = c["Hq"], c["D"], c["topk"]
    G, i, scale = Hq // c["Hkv"], L - 1, 1 / math.sqrt(D)
    gated = anchor or c["form"] == "gated"
    sc = torch.full((Hq, 1, k), -math.inf, dtype=torch.float64, device=DEV)
    O = torch.zeros((Hq, 1, D), dtype=torch.float64, device=DEV)
    LSE = torch.zeros((Hq, 1), dtype=torch.float64, device=DEV)
    one = torch.zeros(1, dtype=torch.long, device=DEV)
    if anchor:
        s0, wlo = math.isqrt(c["window"]), max(0, i - c["window"] + 1)
        ell = math.isqrt(i) + (math.isqrt(i) ** 2 < i)
        s = torch.arange(s0, math.isqrt(i + 1), device=DEV)
        cand = i - (s + 1) ** 2 + 1
    else:
        wlo = i // c["S"] * c["S"]
        cand = (torch.arange(i // c["S"], device=DEV) + 1) * c["S"] - 1
    for h in range(Hq):
        q, Kh, Vh = Q[h].double(), K[h // G], V[h // G]
        z = (q @ Kh[cand].double().t())[0]
        kk = min(k, z.numel())
        pick = torch.topk(z, kk).indices.sort().values
        sc[h, 0, :kk] = z[pick]

        def part(lo, hi):
            r = _Rows(1, D)
            if hi > lo:
                r.add(one, q, Kh[lo:hi].double(), Vh[lo:hi].double(), scale)
            return r
        win = part(wlo, i + 1)
        states = []
        for t in cand[pick].tolist():
            if anchor:
                states.append(part(max(0, t - c["back"] * ell), min(min(i, t + c["fwd"] * ell) + 1, wlo)))
            else:
                states.append(part(t + 1 - c["S"], t + 1))
        if gated and states:
            g = torch.softmax(z[pick], 0)
            mixed = [s.merged(win) for s in states]
            O[h] = sum(g[a] * (r.o / r.l[:, None]) for a, r in enumerate(mixed))
        else:
            for s in states:
                win = win.merged(s)
            O[h] = win.o / win.l[:, None]
            LSE[h] = win.m + win.l.log()
    return sc, O, LSE


def _prefill_exact(c, Q, K, V, idx, scores, anchor):
    """(O, LSE or None) of a prefill pass on given selections."""
    Hq, Lq, D = Q.shape
    k, G, L, scale = c["topk"], Hq // c["Hkv"], c["L"], 1 / math.sqrt(D)
    gated = anchor or c.get("form") == "gated"
    q0 = L - Lq
    pos = q0 + torch.arange(Lq, device=DEV)
    if anchor:
        ell = torch.sqrt(pos.double()).floor().long()
        ell = ell - (ell * ell > pos).long()
        ell = ell + (ell * ell < pos).long()
        wlo = (pos - c["window"] + 1).clamp(min=0)
    else:
        A, S = c["A"], c["S"]
        wlo = pos // A * A
    O = torch.empty((Hq, Lq, D), dtype=torch.float64, device=DEV)
    LSE = None if gated else torch.empty((Hq, Lq), dtype=torch.float64, device=DEV)
    for kv in range(c["Hkv"]):
        Kh, Vh = K[kv], V[kv]
        R = G * Lq
        q = Q[kv * G:(kv + 1) * G].reshape(R, D)
        e = idx[kv * G:(kv + 1) * G].reshape(R, k).long()
        i = pos.repeat(G)
        w0 = wlo.repeat(G)
        if anchor:
            ok = (e >= 0) & (e <= i[:, None])
            lo = (e - c["back"] * ell.repeat(G)[:, None]).clamp(min=0)
            hi = torch.minimum(torch.minimum(e + c["fwd"] * ell.repeat(G)[:, None], i[:, None]) + 1, w0[:, None])
        else:
            ok = (e >= 0) & (e < (i // A)[:, None])
            hi = (e + 1) * A
            lo = (hi - S).clamp(min=0)
            if A < S and not gated:  # a token of the union counts once
                for a in range(k):
                    for b in range(k):
                        lower = ok[:, b] & (e[:, b] < e[:, a])
                        lo[:, a] = torch.where(lower, torch.maximum(lo[:, a], hi[:, b]), lo[:, a])
        some = ok & (hi > lo)
        win = _Rows(R, D)
        T = 512
        for r0 in range(0, Lq, T):
            r1 = min(Lq, r0 + T)
            at = (torch.arange(G, device=DEV)[:, None] * Lq + torch.arange(r0, r1, device=DEV)[None, :]).reshape(-1)
            a, b = int(wlo[r0]), q0 + r1
            win.add(at, q[at].double(), Kh[a:b].double(), Vh[a:b].double(), scale, w0[at], i[at] + 1, a)

        def add_pairs(state, where, pair_rows, pair_lo, pair_hi):
            # pairs sorted by where their range ends: neighbours share most of it.  A row may come twice.
            order = torch.argsort(pair_hi * (1 << 31) + where)
            where, pair_rows, pair_lo, pair_hi = (x[order] for x in (where, pair_rows, pair_lo, pair_hi))
            step = 2048 if anchor else 8192
            if anchor:
                cuts = list(range(0, where.numel(), step)) + [where.numel()]
            else:  # never across two spans
                ends = (torch.nonzero(pair_hi[1:] != pair_hi[:-1]).flatten() + 1).tolist()
                cuts = [0]
                for z in ends + [where.numel()]:
                    while z - cuts[-1] > step:
                        cuts.append(cuts[-1] + step)
                    if z > cuts[-1]:
                        cuts.append(z)
            for x, y in zip(cuts[:-1], cuts[1:]):
                if y <= x:
                    continue
                l0, h0 = pair_lo[x:y], pair_hi[x:y]
                a, b = (int(v) for v in torch.stack((l0.min(), h0.max())).tolist())
                state.add(where[x:y], q[pair_rows[x:y]].double(), Kh[a:b].double(), Vh[a:b].double(), scale, l0, h0, a)

        rows = torch.arange(R, device=DEV)
        if not gated:
            for a in range(k):  # a row's slots one after the other: each row once a call
                w = rows[some[:, a]]
                if w.numel():
                    add_pairs(win, w, w, lo[w, a], hi[w, a])
            O[kv * G:(kv + 1) * G] = (win.o / win.l[:, None]).reshape(G, Lq, D)
            LSE[kv * G:(kv + 1) * G] = (win.m + win.l.log()).reshape(G, Lq)
            continue
        g = torch.where(ok, scores[kv * G:(kv + 1) * G].reshape(R, k).double(), -math.inf)
        none = ~ok.any(dim=1)
        g = torch.softmax(torch.where(none[:, None], 0.0, g), dim=1)
        out = torch.where(none[:, None], win.o / win.l[:, None], 0.0)
        for a in range(k):
            st = _Rows(R, D)
            w = rows[some[:, a]]
            if w.numel():
                add_pairs(st, w, w, lo[w, a], hi[w, a])
            r = st.merged(win)
            out = out + torch.where((ok[:, a] & ~none)[:, None], g[:, a, None] * (r.o / r.l[:, None]), 0.0)
        O[kv * G:(kv + 1) * G] = out.reshape(G, Lq, D)
    return O, LSE


def exact(case, seed):
    c, kind = case, case["kind"]
    st = prepare(case, seed)
    if kind == "decode_batch":
        Q, _, K, V, _ = st["batch"].tensors
        got = [_decode_exact(c, Q[b], K[b], V[b], Lb, False) for b, Lb in enumerate(_batch_lengths(c))]
        sc, O, LSE = (torch.stack(x) for x in zip(*got))
        return {"idx": None, "scores": sc, "O": O} if c["form"] == "gated" else {"idx": None, "O": O, "LSE": LSE}
    Q, K, V = st["Q"], st["K"], st["V"]
    if kind == "anchor_decode":
        sc, O, _ = _decode_exact(c, Q, K, V, c["L"], True)
        return {"idx": None, "scores": sc, "O": O}
    if kind == "decode":
        sc, O, LSE = _decode_exact(c, Q, K, V, c["L"], False)
        return {"idx": None, "scores": sc, "O": O} if c["form"] == "gated" else {"idx": None, "O": O, "LSE": LSE}
    if kind == "anchor_prefill":
        return {"O": _prefill_exact(c, Q, K, V, st["idx"], st["scores"], True)[0]}
    if kind == "prefill":
        O, LSE = _prefill_exact(c, Q, K, V, st["idx"], st["scores"], False)
        return {"O": O} if LSE is None else {"O": O, "LSE": LSE}
    Hq, Lq, D = Q.shape
    G, k, q0 = Hq // c["Hkv"], c["topk"], c["L"] - Lq
    pos = q0 + torch.arange(Lq, device=DEV)
    if kind == "anchor_search":
        s0 = math.isqrt(c["window"])
        s = torch.arange(s0, max(s0, math.isqrt(c["L"])), device=DEV)
        sc = torch.full((Hq, Lq, k), -math.inf, dtype=torch.float64, device=DEV)
        kk = min(k, s.numel())
        for kv in range(c["Hkv"] if kk else 0):
            for r0 in range(0, Lq, 1024):
                r1 = min(Lq, r0 + 1024)
                t = pos[r0:r1, None] - (s[None, :] + 1) ** 2 + 1
                keys = K[kv][t.clamp(min=0)].double()
                z = torch.matmul(keys, Q[kv * G:(kv + 1) * G, r0:r1].permute(1, 2, 0).double().contiguous()).permute(2, 0, 1)
                z = z.masked_fill((t < 0)[None], -math.inf)
                pick = torch.topk(z, kk, dim=2).indices.sort(dim=2).values
                sc[kv * G:(kv + 1) * G, r0:r1, :kk] = torch.gather(z, 2, pick)
        return {"idx": None, "scores": sc}
    n = c["L"] // c["S"]
    kk = min(k, n)
    if not c["scores"]:
        return None  # spans only
    sc = torch.full((Hq, Lq, k), -math.inf, dtype=torch.float64, device=DEV)
    for h in range(Hq if kk else 0):
        keys = K[h // G, c["S"] - 1:n * c["S"]:c["S"]].double()
        for r0 in range(0, Lq, 16384):
            r1 = min(Lq, r0 + 16384)
            z = Q[h, r0:r1].double() @ keys.t()
            z.masked_fill_(torch.arange(n, device=DEV)[None, :] >= (pos[r0:r1] // c["S"])[:, None], -math.inf)
            v, j = torch.topk(z, kk, dim=1)
            j, order = torch.where(torch.isinf(v), n + 1, j).sort(dim=1)
            sc[h, r0:r1, :kk] = torch.gather(v, 1, order)
    return {"idx": None, "scores": sc}
