"""The work this library is called for, as measured cases.

Every case goes through the package's public calls, on device-resident
inputs made from a seed, with the buffers a serving program keeps
(``Buffers``, ``PositionBuffers``, scratch, outputs):

  pipeline  cb_pipeline: score, select and compact one receiver query against
            the caches of one or more senders
  score     cb_score alone, with the row normalisers
  message   cb_position_score, cb_select_spans and cb_gather_rows: the
            position-level selector and its continuous-row message
  select    cb_select_ws alone on given importance rows

Sizes are those of this repository's workloads and of its tests' ranges:
1 to 48 layers, 1 to 8 query heads per KV head, head width 64 or 128, a query
of 1 to 128 tokens, 256 to 131072 positions per sender, one to three senders,
bf16 or fp32, keep ratios 0.05 to 1.  A case's power p = 0 stands for p = infinity.

Where a call selects, the positions the query is relevant to come in passages
of whole 16-position blocks and number exactly what the call keeps, so that the
selection does not hang on the last bits of the scores.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2609_32046_amd as cb

DEV = "cuda"


def _case(name, kind, L, Hq, Hkv, D, T, m, S=1, dtype="bf16", keep=0.25, kdist="flat", lse=False,
          p=2.0, alpha=2.0):
    return {"name": name, "kind": kind, "L": L, "Hq": Hq, "Hkv": Hkv, "D": D, "T": T, "m": m,
            "S": S, "dtype": dtype, "keep": keep, "kdist": kdist, "lse": lse, "p": p,
            "alpha": alpha}


def listed():
    return [
        # The smallest configuration: one layer of a small fp32 model.  Launch
        # and latency bound.
        _case("tiny", "pipeline", 1, 4, 2, 64, 512, 16, dtype="f32", kdist="normal", lse=True),
        # One layer of the 8B shape, as a program makes it that scores each
        # layer when its cache arrives.
        _case("one-layer", "pipeline", 1, 32, 8, 128, 8192, 64, kdist="normal"),
        # A short question (8 tokens) to a narrow-headed model.
        _case("short-question", "pipeline", 24, 32, 8, 64, 4096, 8, keep=0.5, kdist="normal",
              lse=True),
        # The default workload: the 8B attention shape, 8192 positions.
        _case("8b-8k", "pipeline", 36, 32, 8, 128, 8192, 64),
        # Fan-in: three senders of 16384 positions and a 128-token query.
        _case("fanin-3x16k", "pipeline", 36, 32, 8, 128, 16384, 128, S=3),
        # Long context, five query heads per KV head, a small message.
        _case("longctx-32k", "pipeline", 48, 40, 8, 128, 32768, 64, keep=0.1, kdist="normal"),
        # Hybrid model: few attention layers, a very long sequence.
        _case("hybrid-64k", "pipeline", 8, 32, 8, 128, 65536, 32, kdist="normal"),
        # Sizes that divide nothing: seven query heads per KV head, a 50-token
        # query, 10007 positions, keys with outlier channels.
        _case("ragged", "score", 28, 28, 4, 128, 10007, 50, kdist="outliers", lse=True),
        # fp32 caches of a few layers, with positions that draw the attention.
        _case("fp32-layers", "score", 8, 32, 8, 128, 3000, 32, dtype="f32", kdist="peaked",
              lse=True),
        # The position-level selector of the 8B shape and its message of
        # 8 KiB rows.
        _case("message-8b-8k", "message", 36, 32, 8, 128, 8192, 64),
        # Three short senders, eight query heads per KV head, the general
        # score with another power.
        _case("message-3x3k", "message", 36, 64, 8, 128, 3001, 20, S=3, keep=0.125, p=3.0,
              alpha=1.0),
        # Selection alone on rows of the 8B shape at 100003 positions.
        _case("select-100k", "select", 36, 32, 8, 128, 100003, 64, keep=0.1),
    ]


def _cost(c):
    """Multiply-adds of the logits, or what the moved bytes are worth in them."""
    U = c["S"] * c["L"] * c["Hkv"]
    T = c["T"]
    if c["kind"] == "select":
        return U * T * 4 * 300.0
    R = (c["Hq"] // c["Hkv"]) * c["m"]
    heavy = 8.0 if c["dtype"] == "f32" else 1.0
    return max(U * R * T * c["D"] * heavy, U * T * c["D"] * 4 * 60.0)


def draw(rng):
    """A call of the same ranges, no dearer than the fan-in one."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    most = _cost(next(c for c in listed() if c["name"] == "fanin-3x16k"))
    kind = rng.choice(["pipeline", "pipeline", "pipeline", "score", "message", "select"])
    dtype = "f32" if rng.random() < 0.15 else "bf16"
    Hkv = rng.choice([1, 2, 4, 8])
    G = rng.choice([1, 2, 3, 4, 4, 5, 6, 7, 8])
    D = rng.choice([64, 128, 128])
    m = log_int(1, 128)
    T = log_int(256, 131072)
    S = rng.choice([1, 1, 1, 2, 3])
    L = log_int(1, 48)
    keep = rng.choice([0.05, 0.1, 0.25, 0.25, 0.5, 1.0])
    if kind == "message":
        m = min(m, 1024 // (4 if G <= 4 else 8))
        keep = rng.choice([1 / 16, 1 / 8, 1 / 4])
    kdist = "flat" if kind == "message" else rng.choice(["flat", "normal"])
    if kind == "score":
        kdist = rng.choice(["flat", "normal", "peaked", "outliers"])
    c = _case("", kind, L, G * Hkv, Hkv, D, T, m, S, dtype, keep, kdist, rng.random() < 0.5,
              *(rng.choice([(2.0, 2.0), (2.0, 2.0), (3.0, 1.0), (0.0, 1.0)])
                if kind == "message" else (2.0, 2.0)))
    del c["name"]
    while _cost(c) > most and c["L"] > 1:
        c["L"] = max(1, c["L"] // 2)
    while _cost(c) > most:
        c["T"] //= 2
    return c


# ---------------------------------------------------------------------------
# inputs


def _esize(c):
    return 4 if c["dtype"] == "f32" else 2


def _budget(c):
    """Kept positions per sender of a message (ceil of the fraction; position
    0 and the latents are always kept)."""
    n = cb.cb_budget_fanout(c["T"], round(1.0 / c["keep"]))
    return max(n, min(c["T"], _latents(c) + 1))


def _latents(c):
    return min(40, c["T"] // 8)


def _relevant(c, seed, count, first, last, run):
    """[S][T] mask: `count` positions of every sender in runs of `run` whole
    16-position blocks, within [first, last)."""
    out = np.zeros((c["S"], c["T"]), bool)
    step = 16 * run
    for s in range(c["S"]):
        rng = np.random.default_rng([seed, s, 77])
        left = count
        for b in rng.permutation((last - first + step - 1) // step):
            lo = first + int(b) * step
            n = min(left, last - lo, step)
            out[s, lo:lo + n] = True
            left -= n
            if left == 0:
                break
    return out


def _layout(c):
    return cb.layout(c["L"], c["Hq"], c["Hkv"], c["D"], c["m"], c["T"], senders=c["S"],
                     dtype=c["dtype"])


def _inputs(c, seed):
    """q, K, V and (message) the continuous rows, on the GPU."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    L, Hq, Hkv, D, T, m, S = (c[x] for x in ("L", "Hq", "Hkv", "D", "T", "m", "S"))

    def normal(*shape):
        return torch.randn(shape, generator=gen, device=DEV)

    R = Hq // Hkv * m
    q = normal(L, Hq, m, D)
    mask, chan, pull = None, 0, 0.0
    if c["kind"] in ("pipeline", "message"):
        # One channel carries the relevance: a fixed pull on the relevant
        # positions' logits, large against the spread of the others.
        spread = 0.12 if c["kdist"] == "flat" else 1.0
        pull = 1.5 + 8.0 * spread / math.sqrt(R)
        if c["kind"] == "pipeline":
            mask = _relevant(c, seed, cb.cb_keep_count(T, c["keep"]), 0, T, 1)
        else:
            first, last = 16, (T - _latents(c)) // 16 * 16
            rem = _budget(c) - _latents(c) - 1 - 15
            mask = _relevant(c, seed, max(0, min(rem, last - first) // 16 * 16), first,
                             max(first, last), 4)
        mask = torch.from_numpy(mask).to(DEV)
        chan = seed % D
        q[..., chan] = 4.0
    q = q.to(dt)
    shifted = None
    if c["kdist"] == "peaked":
        n = max(1, int(0.02 * T))
        shifted = torch.from_numpy(np.stack([np.random.default_rng([seed, s, 5]).choice(
            T, n, replace=False) for s in range(S)])).to(DEV)
    k = torch.empty((S, L, Hkv, T, D), dtype=dt, device=DEV)
    want_v = c["kind"] == "pipeline"
    v = torch.empty_like(k) if want_v else None
    for s in range(S):
        for l in range(L):
            x = normal(Hkv, T, D)
            if c["kdist"] == "flat":
                ch = torch.rand((Hkv, 1, D), generator=gen, device=DEV) * 1.5 + 0.5
                x *= ch / math.sqrt(D)
            elif c["kdist"] == "peaked":
                u = normal(Hkv, 1, D)
                x[:, shifted[s]] += u / u.norm(dim=-1, keepdim=True) * (3.0 * math.sqrt(D))
            elif c["kdist"] == "outliers":
                # Student-t(3) keys, four channels twenty times larger
                x /= (normal(3, Hkv, T, D) ** 2).mean(0).sqrt()
                x[..., torch.randperm(D, generator=gen, device=DEV)[:4]] *= 20.0
            if mask is not None:
                x[..., chan] = mask[s].to(torch.float32) * (pull * math.sqrt(D) / 4.0)
            k[s, l] = x
            if want_v:
                v[s, l] = normal(Hkv, T, D)
    rows = None
    if c["kind"] == "message":
        rows = torch.empty((S, T, Hq * D), dtype=dt, device=DEV)
        for s in range(S):
            rows[s] = normal(T, Hq * D)
    return q, k, v, rows


def _select_rows(c, seed):
    """Importance rows as near-uniform attention leaves them: log-normal
    around the mean weight."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    U = c["S"] * c["L"] * c["Hkv"]
    x = torch.randn((U, c["T"]), generator=gen, device=DEV)
    R = c["Hq"] // c["Hkv"] * c["m"]
    return torch.exp(x * 0.1) * (R / c["T"])


def prepare(case, seed):
    c = dict(case)
    if c["kind"] == "select":
        imp = _select_rows(c, seed)
        U, T = imp.shape
        idx = torch.empty((U, cb.cb_keep_count(T, c["keep"])), dtype=torch.int32, device=DEV)
        n = cb.cb_select_workspace_bytes(U, T)
        ws = torch.empty(n, dtype=torch.uint8, device=DEV) if n else None
        return {"c": c, "imp": imp, "idx": idx, "ws": ws}
    q, k, v, rows = _inputs(c, seed)
    lay = _layout(c)
    st = {"c": c, "q": q, "k": k, "v": v, "lay": lay}
    if c["kind"] == "message":
        n = _budget(c)
        st["rows"] = rows
        st["buf"] = cb.PositionBuffers(lay, device=DEV)
        st["idx"] = torch.empty((c["S"], n), dtype=torch.int32, device=DEV)
        st["out"] = torch.empty((c["S"] * n, rows.shape[-1]), dtype=rows.dtype, device=DEV)
    elif c["kind"] == "pipeline":
        st["buf"] = cb.Buffers(lay, c["keep"], device=DEV)
    else:
        st["imp"] = torch.empty(k.shape[:-1], dtype=torch.float32, device=DEV)
        st["lse"] = torch.empty((c["S"], c["L"], c["Hq"], c["m"]), dtype=torch.float32, device=DEV)
        st["ws"] = torch.empty(cb.cb_score_workspace_bytes(lay), dtype=torch.uint8, device=DEV)
    return st


def run(state):
    c = state["c"]
    if c["kind"] == "select":
        U, T = state["imp"].shape
        cb.cb_select_ws(state["imp"], U, T, c["keep"], state["idx"], state["ws"])
        return {"idx": state["idx"]}
    q, k, lay = state["q"], state["k"], state["lay"]
    if c["kind"] == "score":
        lse = state["lse"] if c["lse"] else None
        cb.cb_score(q, k, lay, state["imp"], lse, state["ws"])
        return {"importance": state["imp"], **({"lse": lse} if c["lse"] else {})}
    b = state["buf"]
    if c["kind"] == "pipeline":
        lse = b.row_lse if c["lse"] else None
        cb.cb_pipeline(q, k, state["v"], lay, c["keep"], b.importance, b.idx, b.k_out, b.v_out,
                       b.ws, row_lse=lse)
        return {"importance": b.importance, "idx": b.idx, "k": b.k_out, "v": b.v_out,
                **({"lse": lse} if c["lse"] else {})}
    S, T, n = c["S"], c["T"], state["idx"].shape[1]
    cb.cb_position_score(q, k, lay, b.score, b.ws, p=c["p"] or math.inf, alpha=c["alpha"], qscore=b.qscore,
                         corr=b.corr)
    cb.cb_select_spans(b.score, S, T, n, state["idx"], b.span_ws, n_latent=_latents(c))
    rows, out = state["rows"], state["out"]
    cb.cb_gather_rows(rows, S, T, rows.shape[-1] * rows.element_size(), state["idx"], n, out)
    return {"score": b.score, "q": b.qscore, "corr": b.corr, "idx": state["idx"], "rows": out}


def work(case):
    c = case
    U, T, D, es = c["S"] * c["L"] * c["Hkv"], c["T"], c["D"], _esize(c)
    imp = 4 * U * T
    if c["kind"] == "select":
        return {"bytes": imp + 4 * U * cb.cb_keep_count(T, c["keep"]), "flops": 0}
    R = c["Hq"] // c["Hkv"] * c["m"]
    read = (c["L"] * c["Hq"] * c["m"] * D + U * T * D) * es
    flops = 2 * U * R * T * D
    lse = 4 * U * R if c["lse"] else 0
    if c["kind"] == "score":
        return {"bytes": read + imp + lse, "flops": flops}
    if c["kind"] == "pipeline":
        n = cb.cb_keep_count(T, c["keep"])
        # kept V rows read, kept K (already read) and V rows written
        return {"bytes": read + imp + lse + 4 * U * n + 3 * U * n * D * es, "flops": flops}
    n = _budget(c) * c["S"]
    return {"bytes": read + 3 * 4 * c["S"] * T + 4 * n + 2 * n * c["Hq"] * D * es, "flops": flops}


def tolerance(case):
    """fp32 sums over fp32 logits: the error against 64 bits measures 3e-7 to
    5e-7 in every case, and four times that is stated.  A logit's rounding
    error moves its weight by a like factor, so it grows with the logits (the
    outlier channels' and the peaked positions' reach some tens), and the
    correction raises it to its power."""
    if case["kind"] == "select":
        return "exact"
    if case["kdist"] in ("outliers", "peaked"):
        return {"rel": 1e-5, "max": 1e-4}
    if case["kind"] == "message":
        return {"rel": 4e-6, "max": 4e-5}
    return {"rel": 2e-6, "max": 2e-5}


# ---------------------------------------------------------------------------
# the same in 64 bits, plain torch


def _weights64(q, k, c, s, l, g):
    """Softmax weights [G*m][T] of one unit, and the log normalisers."""
    G = c["Hq"] // c["Hkv"]
    qu = q[l, g * G:(g + 1) * G].reshape(-1, c["D"]).double()
    x = (qu @ k[s, l, g].double().t().contiguous()) / math.sqrt(c["D"])
    lse = torch.logsumexp(x, dim=1, keepdim=True)
    return torch.exp(x - lse), lse.reshape(G, c["m"])


def exact(case, seed):
    c = dict(case)
    if c["kind"] == "select":
        imp = _select_rows(c, seed)
        n = cb.cb_keep_count(c["T"], c["keep"])
        top = torch.sort(imp, dim=1, descending=True, stable=True)[1][:, :n]
        return {"idx": torch.sort(top, dim=1)[0].to(torch.int32)}
    q, k, v, _ = _inputs(c, seed)
    S, L, Hkv, T, D, m = (c[x] for x in ("S", "L", "Hkv", "T", "D", "m"))
    G = c["Hq"] // Hkv
    units = [(s, l, g) for s in range(S) for l in range(L) for g in range(Hkv)]
    if c["kind"] != "message":
        imp = torch.empty((S, L, Hkv, T), dtype=torch.float64, device=DEV)
        lse = torch.empty((S, L, c["Hq"], m), dtype=torch.float64, device=DEV)
        for s, l, g in units:
            w, z = _weights64(q, k, c, s, l, g)
            imp[s, l, g] = w.sum(0)
            lse[s, l, g * G:(g + 1) * G] = z
        got = {"importance": imp, **({"lse": lse} if c["lse"] else {})}
        if c["kind"] == "score":
            return got
        n = cb.cb_keep_count(T, c["keep"])
        top = torch.sort(imp, dim=-1, descending=True, stable=True)[1][..., :n]
        idx = torch.sort(top, dim=-1)[0]
        for name, x in (("k", k), ("v", v)):
            y = torch.empty((L, Hkv, S * n, D), dtype=x.dtype, device=DEV)
            for s, l, g in units:
                y[l, g, s * n:(s + 1) * n] = x[s, l, g][idx[s, l, g]]
            got[name] = y
        return {**got, "idx": idx.to(torch.int32)}

    def pool(x):   # maximum over positions t-3 .. t+3
        return torch.nn.functional.max_pool1d(x.reshape(-1, 1, T), 7, 1, 3).reshape(x.shape)

    p = c["p"] or math.inf
    Q = torch.zeros((S, T), dtype=torch.float64, device=DEV)
    num, den = torch.zeros_like(Q), torch.zeros_like(Q)
    for s, l, g in units:
        w, _ = _weights64(q, k, c, s, l, g)
        Q[s] += w.sum(0) / (m * c["Hq"])
        b = w.reshape(G, m, T).mean(0)
        if math.isinf(p):
            num[s] = torch.maximum(num[s], pool(b).amax(0))
            den[s] = torch.maximum(den[s], pool(b.mean(0)))
        else:
            num[s] += (pool(b) ** p).mean(0)
            den[s] += pool(b.mean(0)) ** p
    corr = num / den if math.isinf(p) else (num / den) ** (1.0 / (p - 1.0))
    Q = pool(Q)
    return {"score": Q * corr ** c["alpha"], "q": Q, "corr": corr, "idx": None, "rows": None}
