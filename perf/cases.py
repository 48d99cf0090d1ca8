"""Performance cases: the calls a serving program makes on this framework.

Four kinds of pass, each through the public binding (paper_2607_01237_amd.kara):

event      one compression interval: the tables are uploaded, the window's
           tokens appended (kv_append), and one compression event runs with the
           metadata commit (compress_window, compress_prefill with several
           windows, or the allocation-free entry).  The append rewrites every row
           compaction moved, so each pass compresses the same fresh window.
decode     one decoding step: lengths uploaded, one token per sequence
           appended, attention of one query per head over the paged cache.
attention  the recompute pass's causal attention of the window queries, one layer.
recompute  the window recompute pass (query projection, rotary embedding,
           attention, feed-forward), bf16 weights, fp32 residual stream.

Cache rows are returned as the bits they hold: the step moves rows, it never
computes them.  Inputs are N(0, 1) rows of the shapes the workloads in
kara_inputs name (model weights are not available); keys optionally carry 2 %
heavy hitters (4 x the norm) or a random rank-8 component.
"""
import math

import numpy as np
import torch

from paper_2607_01237_amd import kara

_DEV = "cuda:0"

_EVENT = dict(kind="event", entry="window", dtype="bf16", n_q=32, n_kv=8, d=128, window=1024, buffer=0, budget=205,
              alpha=16, gamma=8, queries=0, n_windows=1, seqs=8, idle=0, layers=1, prefix_lo=0, prefix_hi=2047, tail=0,
              block=16, keys="normal")
_DECODE = dict(kind="decode", dtype="bf16", n_q=32, n_kv=8, d=128, seqs=8, layers=1, len_lo=300, len_hi=4000, block=16)
_ATTN = dict(kind="attention", n_q=32, n_kv=8, d=128, window=1024, seqs=4, prefix_lo=3072, prefix_hi=15360, block=16)
_RECOMPUTE = dict(kind="recompute", n_q=32, n_kv=8, d=128, window=1024, seqs=1, layers=1, prefix_lo=3072,
                  prefix_hi=15360, block=16, hidden=4096, ffn=12288)


def listed():
    return [
        # a single small sequence in fp32: all launch latency and host work
        dict(_EVENT, name="event_tiny_f32", entry="noalloc", dtype="f32", n_q=4, n_kv=1, d=64, window=128, budget=26,
             alpha=4, gamma=4, seqs=1, prefix_lo=64, prefix_hi=64, tail=5),
        # one layer of a small batch, as a recompute forward hands layers over;
        # 2 % heavy-hitter keys per head, which trained models show
        dict(_EVENT, name="event_layer_heavy", seqs=8, tail=7, keys="heavy"),
        # the serving loop's event: 256-token blocks, three-block windows, a buffer
        dict(_EVENT, name="event_serve", window=768, buffer=32, budget=225, seqs=30, idle=34, layers=8,
             prefix_lo=64, prefix_hi=1500, tail=150, block=256),
        # the Qwen3-14B-shaped batch, whole windows scored by every query: the largest
        dict(_EVENT, name="event_14b", n_q=40, window=2048, budget=410, seqs=64, layers=4, prefix_lo=4096,
             prefix_hi=16384, tail=9, keys="lowrank"),
        # whole-cache top-k scored by a 32-token observation window: few queries, much compaction
        dict(_EVENT, name="event_observe", window=1280, buffer=32, budget=993, alpha=0, queries=32, seqs=128, layers=4,
             prefix_lo=0, prefix_hi=0),
        # an odd window of 64-wide heads with an unaligned block size
        dict(_EVENT, name="event_odd_d64", n_q=16, d=64, window=701, buffer=33, budget=134, seqs=21, layers=6,
             prefix_lo=1, prefix_hi=3001, tail=29, block=24),
        # prompts compressed before decoding, 16 windows each
        dict(_EVENT, name="prefill_16win", entry="prefill", n_windows=16, seqs=4, layers=4, prefix_lo=0, prefix_hi=0,
             tail=509),
        # one decoding layer of a small batch, and a long-context batch
        dict(_DECODE, name="decode_small"),
        dict(_DECODE, name="decode_long", n_q=40, seqs=128, layers=4, len_lo=7000, len_hi=8190),
        # the window recompute: attention alone, a small pass and a large one
        dict(_ATTN, name="attention_16seq", seqs=16),
        dict(_RECOMPUTE, name="recompute_1seq", window=768, prefix_lo=1200, prefix_hi=1200, layers=2, block=256),
        dict(_RECOMPUTE, name="recompute_8seq", seqs=8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# a drawn case's cost in seconds at rough rates stays under the largest listed one's
_MOST_S = 0.012


def draw(rng):
    kind = rng.choice(["event", "event", "event", "decode", "attention", "recompute"])
    block = rng.choice([16, 16, 256, 24])
    while True:
        if kind == "event":
            n_q, n_kv, d = rng.choice([(32, 8, 128), (40, 8, 128), (16, 8, 64), (8, 2, 128), (4, 1, 64)])
            window = _log_int(rng, 96, 4096)
            buffer = rng.choice([0, 0, 32, min(window // 3, rng.randrange(1, 64))])
            n = window - buffer
            budget = max(8, math.ceil(n * rng.choice([0.2, 0.2, 0.3, 0.75])))
            alpha = rng.choice([0, 16, 16]) if budget > 32 else 4
            prefill = rng.random() < 0.2 and window <= 1100
            lo = rng.randrange(0, 1000)
            c = dict(_EVENT, entry="prefill" if prefill else "window", dtype=rng.choice(["bf16", "bf16", "bf16", "f32"]),
                     n_q=n_q, n_kv=n_kv, d=d, window=window, buffer=buffer, budget=budget, alpha=alpha,
                     queries=buffer if buffer and rng.random() < 0.25 else 0,
                     n_windows=rng.randrange(2, 17) if prefill else 1, seqs=_log_int(rng, 1, 64),
                     layers=_log_int(rng, 1, 16), prefix_lo=lo, prefix_hi=lo + rng.randrange(0, 4000),
                     tail=rng.randrange(0, 300), block=block, keys=rng.choice(["normal", "normal", "heavy", "lowrank"]))
        elif kind == "decode":
            n_q, n_kv, d = rng.choice([(32, 8, 128), (40, 8, 128), (16, 2, 64), (8, 8, 128)])
            lo = _log_int(rng, 40, 6000)
            c = dict(_DECODE, dtype=rng.choice(["bf16", "bf16", "bf16", "f32"]), n_q=n_q, n_kv=n_kv, d=d,
                     seqs=_log_int(rng, 1, 128), layers=_log_int(rng, 1, 32), len_lo=lo, len_hi=lo + _log_int(rng, 1, 6000),
                     block=block)
        elif kind == "attention":
            n_q, n_kv, d = rng.choice([(32, 8, 128), (40, 8, 128), (16, 8, 64)])
            lo = _log_int(rng, 50, 8000)
            c = dict(_ATTN, n_q=n_q, n_kv=n_kv, d=d, window=_log_int(rng, 100, 2048), seqs=_log_int(rng, 1, 24),
                     prefix_lo=lo, prefix_hi=lo + rng.randrange(0, 8000), block=block)
        else:
            lo = _log_int(rng, 50, 8000)
            hidden, ffn, n_q = rng.choice([(4096, 12288, 32), (5120, 17408, 40), (1024, 3072, 16)])
            c = dict(_RECOMPUTE, n_q=n_q, hidden=hidden, ffn=ffn, window=_log_int(rng, 200, 2048),
                     seqs=_log_int(rng, 1, 8), layers=rng.randrange(1, 3), prefix_lo=lo,
                     prefix_hi=lo + rng.randrange(0, 4000), block=block)
        w = work(c)
        slow = 8 if c.get("dtype") == "f32" else 2 if c["d"] == 64 else 1
        if w["bytes"] / 2e12 + slow * w["flops"] / 5e14 <= _MOST_S:
            return c


# ---- geometry

def _lengths(c):
    """Tokens in each sequence before the pass: a fixed spread over the case's range."""
    lo, hi = (c["len_lo"], c["len_hi"]) if c["kind"] == "decode" else (c["prefix_lo"], c["prefix_hi"])
    n = c["seqs"] + c.get("idle", 0)
    lens = np.linspace(lo, hi, n).round().astype(np.int64) if n > 1 else np.array([(lo + hi) // 2])
    return np.random.default_rng(n).permutation(lens)


def _new_tokens(c):
    if c["kind"] == "event":
        return (c["n_windows"] - 1) * (c["window"] - c["buffer"]) + c["window"] + c["tail"]
    return {"decode": 1, "attention": c.get("window"), "recompute": c.get("window")}[c["kind"]]


def work(c):
    e = 4 if c.get("dtype") == "f32" else 2
    lens, new = _lengths(c)[:c["seqs"]], _new_tokens(c)
    row = c["n_kv"] * c["d"] * e                    # one token's K (or V) row in one layer
    q_row = c["n_q"] * c["d"] * e
    L, S = c.get("layers", 1), c["seqs"]
    if c["kind"] == "event":
        n = c["window"] - c["buffer"]
        wq = c["queries"] or c["window"]
        moved = new - c["n_windows"] * (n - c["budget"])
        per = (4 * new * row + c["n_windows"] * (wq * q_row + n * row + n * c["n_kv"] * 4)   # append; queries, keys, scores
               + 4 * moved * row)                                                            # compaction
        return {"bytes": S * L * per, "flops": S * L * c["n_windows"] * 2 * n * wq * c["n_q"] * c["d"]}
    if c["kind"] == "decode":
        keys = int((lens + 1).sum())
        return {"bytes": L * (2 * keys * row + S * (4 * row + q_row + c["n_q"] * c["d"] * 4)),
                "flops": L * keys * 4 * c["n_q"] * c["d"]}
    W = c["window"]
    keys = int((lens + W).sum())
    pairs = int((lens * W + W * (W + 1) // 2).sum())
    if c["kind"] == "attention":
        return {"bytes": 2 * keys * row + 2 * S * W * q_row, "flops": pairs * 4 * c["n_q"] * c["d"]}
    params = 2 * c["hidden"] * c["n_q"] * c["d"] + 3 * c["hidden"] * c["ffn"]
    return {"bytes": L * (2 * params + 2 * keys * row + S * W * q_row) + 2 * S * W * c["hidden"] * 4,
            "flops": L * (2 * params * S * W + pairs * 4 * c["n_q"] * c["d"])}


def _gen(seed):
    g = torch.Generator(device=_DEV)
    g.manual_seed(int(seed))
    return g


def _randn(g, shape, dt):
    return torch.randn(shape, generator=g, device=_DEV, dtype=dt)


def _paged(c, seed, reserve):
    """Tables of a fragmented pool: every sequence mapped for its tokens plus `reserve`."""
    lens = _lengths(c)
    bs = c["block"]
    need = [-(-int(n + (reserve if i < c["seqs"] else 0)) // bs) for i, n in enumerate(lens)]
    pages = math.ceil(sum(need) * 1.05) + 1
    order = np.random.default_rng(seed).permutation(pages)
    table = np.full((len(lens), max(max(need), 1)), -1, dtype=np.int32)
    at = 0
    for i, n in enumerate(need):
        table[i, :n] = order[at:at + n]
        at += n
    return lens.astype(np.int32), table, pages


def _params(c, pages, max_blocks):
    ev = c["kind"] == "event"
    w = c.get("window", 64)
    return kara.make_params(dict(
        window=w, buffer=c["buffer"] if ev else 0, budget=c["budget"] if ev else max(1, w // 5),
        chunk_budget=c["alpha"] if ev else 0, max_chunk_len=c["gamma"] if ev else 4, head_dim=c["d"], n_q_heads=c["n_q"],
        n_kv_heads=c["n_kv"], block_size=c["block"], num_pages=pages, max_blocks_per_seq=max_blocks,
        dtype=c.get("dtype", "bf16"), scale=0.0, score_queries=c["queries"] if ev else 0),
        c["seqs"] + c.get("idle", 0))


def prepare(c, seed):
    dt = torch.float32 if c.get("dtype") == "f32" else torch.bfloat16
    g = _gen(seed)
    new = _new_tokens(c)
    lens, table, pages = _paged(c, seed, new)
    L, S, H, d = c.get("layers", 1), c["seqs"], c["n_kv"], c["d"]
    st = dict(case=c, p=_params(c, pages, table.shape[1]))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(_DEV)  # noqa: E731
    shape = (L, pages, H, c["block"], d)
    # earlier context is not read by an event: its rows may hold anything
    fill = (lambda: torch.zeros(shape, dtype=dt, device=_DEV)) if c["kind"] == "event" else (lambda: _randn(g, shape, dt))
    st["k"], st["v"] = fill(), fill()
    st["kp"], st["vp"] = list(st["k"].unbind(0)), list(st["v"].unbind(0))
    st["seqs"] = torch.arange(S, dtype=torch.int32, device=_DEV)
    # the triggered sequences come first in `lens`; the others are idle
    st["bt0"], st["lens0"] = dev(table), dev(lens)
    st["bt"], st["lens"] = st["bt0"].clone(), st["lens0"].clone()
    st["status"] = torch.zeros(S, dtype=torch.int32, device=_DEV)
    i32 = dict(dtype=torch.int32, device=_DEV)
    if c["kind"] in ("event", "decode"):
        st["k_new"], st["v_new"] = (_randn(g, (L, S, new, H, d), dt) for _ in range(2))
        st["app_status"] = torch.zeros(S, **i32)
    if c["kind"] == "event":
        if c["keys"] == "heavy":
            hot = torch.rand((L, S, new, H, 1), generator=g, device=_DEV) < 0.02
            st["k_new"].mul_(torch.where(hot, 4.0, 1.0).to(dt))
        elif c["keys"] == "lowrank":
            for layer in range(L):
                basis = _randn(g, (H, 8, d), torch.float32) / 8 ** 0.5
                coef = _randn(g, (H, S * new, 8), torch.float32)
                low = torch.matmul(coef, basis).view(H, S, new, d).permute(1, 2, 0, 3)
                st["k_new"][layer] = (st["k_new"][layer].float() + low).to(dt)
        wq = c["queries"] or c["window"]
        nw, n = c["n_windows"], c["window"] - c["buffer"]
        st["q"] = _randn(g, (L, S) + ((nw,) if c["entry"] == "prefill" else ()) + (wq, c["n_q"], d), dt)
        st["win_start"] = st["lens0"].clone()
        units = (L, S) + ((nw,) if c["entry"] == "prefill" else ()) + (H,)
        st["scores"] = torch.empty(units + (n,), dtype=torch.float32, device=_DEV)
        st["discrete"] = torch.empty(units + (c["budget"] - c["alpha"],), **i32)
        st["kept"] = torch.empty(units + (c["budget"],), **i32)
        st["freed"], st["n_freed"] = torch.empty((S, table.shape[1]), **i32), torch.empty(S, **i32)
        if c["entry"] != "noalloc":
            st["ws"] = torch.empty(kara.workspace_size(st["p"], S * nw, L), dtype=torch.uint8, device=_DEV)
    elif c["kind"] == "decode":
        st["max_len"] = table.shape[1] * c["block"]
        st["q"] = _randn(g, (L, S, c["n_q"], d), dt)
        st["out"] = torch.empty((L, S, c["n_q"], d), dtype=torch.float32, device=_DEV)
        st["ws"] = torch.empty(kara.decode_workspace_size(st["p"], S, L, st["max_len"]), dtype=torch.uint8, device=_DEV)
    else:
        W = c["window"]
        st["win_start"] = st["lens0"].clone()
        st["lens"] = st["lens0"] + W
        if c["kind"] == "attention":
            st["q"] = _randn(g, (S, W, c["n_q"], d), dt)
            st["out"] = torch.empty_like(st["q"])
        else:
            D, F, HD = c["hidden"], c["ffn"], c["n_q"] * d
            w = lambda a, b: _randn(g, (a, b), dt) / a ** 0.5  # noqa: E731
            st["weights"] = [dict(w_q=w(D, HD), w_o=w(HD, D), w_gate=w(D, F), w_up=w(D, F), w_down=w(F, D),
                                  g_attn=torch.ones(D, dtype=dt, device=_DEV), g_ffn=torch.ones(D, dtype=dt, device=_DEV))
                             for _ in range(L)]
            st["model"] = kara.make_model(D, F, 1e6, 1e-6)
            st["h0"] = _randn(g, (S, W, D), torch.float32)
            st["h1"] = torch.empty_like(st["h0"])
            st["q"] = torch.empty((L, S, W, c["n_q"], d), dtype=dt, device=_DEV)
            st["rope_pos0"] = st["win_start"].clone()
            st["ws"] = torch.empty(kara.recompute_workspace_size(st["p"], st["model"], S), dtype=torch.uint8, device=_DEV)
    return st


def _bits(t):
    return t.view(torch.int16 if t.dtype == torch.bfloat16 else torch.int32)


def run(st):
    c, p = st["case"], st["p"]
    if c["kind"] == "event":
        st["bt"].copy_(st["bt0"])
        st["lens"].copy_(st["lens0"])
        kara.kv_append(p, st["seqs"], st["k_new"], st["v_new"], st["kp"], st["vp"], st["bt"], st["lens"], st["app_status"])
        args = (st["q"], st["kp"], st["vp"], st["bt"], st["lens"], st["win_start"], True, st["status"])
        outs = dict(scores=st["scores"], discrete=st["discrete"], kept=st["kept"], freed=st["freed"], n_freed=st["n_freed"])
        if c["entry"] == "prefill":
            kara.compress_prefill(p, st["seqs"], c["n_windows"], *args, st["ws"], **outs)
        elif c["entry"] == "noalloc":
            kara.compress_window_noalloc(p, st["seqs"], *args, **outs)
        else:
            kara.compress_window(p, st["seqs"], *args, st["ws"], **outs)
        return dict(outs, tables=st["bt"], lens=st["lens"], status=st["status"], k=_bits(st["k"]), v=_bits(st["v"]))
    if c["kind"] == "decode":
        st["lens"].copy_(st["lens0"])
        kara.kv_append(p, st["seqs"], st["k_new"], st["v_new"], st["kp"], st["vp"], st["bt"], st["lens"], st["app_status"])
        kara.decode_attention(p, st["seqs"], st["q"], st["kp"], st["vp"], st["bt"], st["lens"], st["max_len"], st["out"],
                              st["ws"])
        return dict(out=st["out"], lens=st["lens"], status=st["app_status"], k=_bits(st["k"]), v=_bits(st["v"]))
    if c["kind"] == "attention":
        kara.recompute_attention(p, st["seqs"], st["q"], st["kp"][0], st["vp"][0], st["bt"], st["lens"], st["win_start"],
                                 st["out"], st["status"])
        return dict(out=st["out"], status=st["status"])
    kara.recompute_queries(p, st["model"], st["seqs"], st["weights"], st["h0"], st["h1"], st["kp"], st["vp"], st["bt"],
                           st["lens"], st["win_start"], st["rope_pos0"], st["q"], st["status"], st["ws"])
    return dict(hidden=st["h1"], queries=st["q"], status=st["status"])


def tolerance(c):
    """Scores: column sums over `rows` query rows of bf16 inputs, each weight
    held to 11 bits (fp32 inputs: fp32 throughout).  `differ` is for ties in
    the kept sets: two scores closer than their rounding may swap, which
    shifts the positions between them and the rows moved.  Decoding: fp32
    weights and sums.  Recompute: bf16 weights and activations."""
    if c["kind"] == "event":
        rows = c["n_q"] // c["n_kv"] * (c["queries"] or c["window"])
        rel = 1e-6 if c["dtype"] == "f32" else 1e-6 + 1.5e-3 / math.sqrt(rows)
        return {"rel": rel, "max": 20 * rel, "differ": 0.005}
    if c["kind"] == "decode":
        return {"rel": 2e-6, "max": 4e-5}
    return {"rel": 1e-2, "max": 1e-1 if c["kind"] == "attention" else 2e-1}


# ---- the same results in fp64 torch

def _rows(pool, table, lens, s, h, n, bs):
    """Positions [0, n) of sequence s, head h from one layer's pool, fp64."""
    pos = torch.arange(n, device=_DEV)
    pages = table[s].to(torch.int64)[pos // bs]
    return pool[pages, h, pos % bs].double()


def _chunked_attention(q, k, v, first_len, causal_group):
    """softmax(q k^T) v in fp64, row r of q seeing the first first_len + r // causal_group keys."""
    out = torch.empty(q.shape[0], v.shape[1], dtype=torch.float64, device=_DEV)
    kt = k.t().contiguous()
    step = max(1, (1 << 26) // k.shape[0])
    at = torch.arange(k.shape[0], device=_DEV)
    for r0 in range(0, q.shape[0], step):
        x = torch.matmul(q[r0:r0 + step], kt)
        rows = torch.arange(r0, r0 + x.shape[0], device=_DEV)
        x.masked_fill_(at[None, :] >= (first_len + rows // causal_group)[:, None], -math.inf)
        out[r0:r0 + step] = torch.matmul(torch.softmax(x, dim=1), v)
    return out


def _window_attention(q, k, v, st, s, c):
    """Causal attention of one sequence's window queries [W][n_q][d] over its cache, fp64."""
    G, W = c["n_q"] // c["n_kv"], c["window"]
    p0 = int(st["win_start"][s])
    out = torch.empty(q.shape, dtype=torch.float64, device=_DEV)
    for h in range(c["n_kv"]):
        kr, vr = (_rows(t, st["bt"], None, s, h, p0 + W, c["block"]) for t in (k, v))
        rows = (q[:, h * G:(h + 1) * G].double() / math.sqrt(c["d"])).reshape(W * G, c["d"])
        out[:, h * G:(h + 1) * G] = _chunked_attention(rows, kr, vr, p0 + 1, G).view(W, G, c["d"])
    return out


def exact(c, seed):
    st = prepare(c, seed)
    S, G, H, d = c["seqs"], c["n_q"] // c["n_kv"], c["n_kv"], c["d"]
    if c["kind"] == "event":
        n, nw = c["window"] - c["buffer"], c["n_windows"]
        q = st["q"].view(c["layers"], S, nw, -1, H, G, d)
        scores = torch.empty((c["layers"], S, nw, H, n), dtype=torch.float64, device=_DEV)
        for layer in range(c["layers"]):
            for s in range(S):
                for w in range(nw):
                    k = st["k_new"][layer, s, w * n:w * n + n].double().permute(1, 2, 0).contiguous()       # [H][d][n]
                    rows = q[layer, s, w].double().permute(1, 0, 2, 3).reshape(H, -1, d) / math.sqrt(d)
                    x = torch.matmul(rows, k)
                    scores[layer, s, w] = torch.softmax(x, dim=2).sum(dim=1)
        names = ("discrete", "kept", "freed", "n_freed", "tables", "lens", "status", "k", "v")
        return dict({k: None for k in names}, scores=scores.view(st["scores"].shape))
    if c["kind"] == "decode":
        out = torch.empty(st["out"].shape, dtype=torch.float64, device=_DEV)
        lens = st["lens0"].tolist()
        for layer in range(c["layers"]):
            for s in range(S):
                n = lens[s]
                pos = torch.arange(n, device=_DEV)
                pages = st["bt"][s].to(torch.int64)[pos // c["block"]]
                k, v = (torch.cat([pool[layer][pages, :, pos % c["block"]], new[layer, s]]).double()                 # [n+1][H][d]
                        for pool, new in ((st["k"], st["k_new"]), (st["v"], st["v_new"])))
                rows = st["q"][layer, s].double().view(H, G, d) / math.sqrt(d)
                x = torch.softmax(torch.matmul(rows, k.permute(1, 2, 0).contiguous()), dim=2)
                out[layer, s] = torch.matmul(x, v.permute(1, 0, 2).contiguous()).reshape(c["n_q"], d)
        return dict(out=out, lens=None, status=None, k=None, v=None)
    if c["kind"] == "attention":
        out = torch.stack([_window_attention(st["q"][s], st["k"][0], st["v"][0], st, s, c) for s in range(S)])
        return dict(out=out, status=None)
    h = st["h0"].double()
    queries = torch.empty(st["q"].shape, dtype=torch.float64, device=_DEV)
    half = d // 2
    freq = st["model"].rope_theta ** (-torch.arange(half, dtype=torch.float64, device=_DEV) / half)
    pos = st["rope_pos0"].double()[:S, None] + torch.arange(c["window"], dtype=torch.float64, device=_DEV)
    ang = pos[:, :, None, None] * freq
    norm = lambda x: x / torch.sqrt((x * x).mean(dim=-1, keepdim=True) + 1e-6)  # noqa: E731  (unit gains)
    for layer in range(c["layers"]):
        w = {k: t.double() for k, t in st["weights"][layer].items()}
        x = torch.matmul(norm(h), w["w_q"]).view(S, c["window"], c["n_q"], d)
        a, b = x[..., :half], x[..., half:]
        q = torch.cat([a * torch.cos(ang) - b * torch.sin(ang), b * torch.cos(ang) + a * torch.sin(ang)], dim=-1)
        queries[layer] = q
        o = torch.stack([_window_attention(q[s], st["k"][layer], st["v"][layer], st, s, c) for s in range(S)])
        h = h + torch.matmul(o.reshape(S, c["window"], -1), w["w_o"])
        x = norm(h)
        gate = torch.matmul(x, w["w_gate"])
        h = h + torch.matmul(gate * torch.sigmoid(gate) * torch.matmul(x, w["w_up"]), w["w_down"])
    return dict(hidden=h, queries=queries, status=None)
