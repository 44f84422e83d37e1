"""Performance cases of the attention forward: what a program calls it with.

Each case is one `fwd` call: a dtype, a head tuple, a layout (fixed-length
batch or packed variable-length batch), a mask and the score and norm options.
Sequence lengths, segment starts and listed global positions of a case come
from its own `len_seed`, tensor values from the seed given to `prepare`.

`listed()` are twelve representative calls; `draw(rng)` makes further ones of
the same families: fp32 calls, prompts, packed prompts, decode steps against
caches of even and uneven length, chunked prefill, index masks, and the ReLU
and Sigmoid normalisations.
"""
import math
import random

import numpy as np
import torch

import paper_2605_05023_amd as attn

_DEFAULTS = dict(dtype="bf16", layout="fixed", batch=1, hq=32, hkv=8, d=128, sq=0, sk=0,
                 # packed: query lengths in [q_lo, q_hi]; key length = query length plus a
                 # cached part in [c_lo, c_hi]
                 q_lo=0, q_hi=0, c_lo=0, c_hi=0, len_seed=0,
                 mask="causal", window_left=-1, window_right=-1, prefix_len=0, num_global=0,
                 listed_global=False, num_segments=0, query_start=0, alibi=False, softcap=0.0,
                 relpos=False, norm="softmax", sigma=1.0)


def _full(case):
    c = dict(_DEFAULTS)
    c.update(case)
    return c


def listed():
    return [
        # the smallest fp32 call of the benchmark: launch and start-up latency
        dict(name="fp32_small", dtype="fp32", batch=1, hq=2, hkv=2, d=64, sq=128, sk=128,
             mask="none"),
        # an fp32 training-size check run: grouped heads, causal, ragged length
        dict(name="fp32_causal", dtype="fp32", batch=2, hq=16, hkv=4, d=128, sq=1000, sk=1000),
        # one short user prompt
        dict(name="prompt_short", batch=1, hq=32, hkv=8, d=128, sq=333, sk=333),
        # training / prefill batch, multi-head causal
        dict(name="prefill_causal", batch=4, hq=16, hkv=16, d=128, sq=2048, sk=2048),
        # long-context prefill with a sliding window and grouped heads
        dict(name="prefill_window", batch=2, hq=32, hkv=8, d=128, sq=8192, sk=8192,
             mask="sliding_window", window_left=1023, window_right=0),
        # bidirectional encoder, ALiBi and soft-cap, head dim 64
        dict(name="encoder_alibi_softcap", batch=8, hq=16, hkv=16, d=64, sq=4096, sk=4096,
             mask="none", alibi=True, softcap=50.0, sigma=1.5),
        # packed prefill of a serving batch, lengths 256..8192 (the largest case)
        dict(name="packed_prefill", layout="packed", batch=16, hq=32, hkv=8, d=128, q_lo=256,
             q_hi=8192, len_seed=4),
        # one decode step of a serving batch against caches of uneven length
        dict(name="decode_packed", layout="packed", batch=32, hq=32, hkv=8, d=128, q_lo=1, q_hi=1,
             c_lo=256, c_hi=8192, len_seed=5),
        # one decode step of a single long conversation, 128/8/128 heads
        dict(name="decode_single", batch=1, hq=128, hkv=8, d=128, sq=1, sk=8192),
        # chunked prefill: new tokens of four sequences against their caches, 64/8/128 heads
        dict(name="chunk_prefill", layout="packed", batch=4, hq=64, hkv=8, d=128, q_lo=100,
             q_hi=512, c_lo=1024, c_hi=12288, len_seed=6),
        # several answers sharing one question (general mask path), odd length
        dict(name="share_question", batch=2, hq=32, hkv=32, d=128, sq=5001, sk=5001,
             mask="share_question", prefix_len=1250, num_segments=4, len_seed=7),
        # PrefixLM with soft-cap and the Sigmoid normalisation
        dict(name="prefix_softcap_sigmoid", batch=1, hq=32, hkv=32, d=128, sq=3000, sk=3000,
             mask="prefix_lm", prefix_len=700, softcap=50.0, norm="sigmoid"),
    ]


# ---- drawing --------------------------------------------------------------

_MAX_FLOPS = {"bf16": 1.2e12, "fp32": 1.8e10}
_MAX_BYTES = 1.0e9


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _heads(rng, big=True):
    pool = [(32, 32, 128), (32, 8, 128), (16, 16, 128), (16, 16, 64), (12, 4, 64), (8, 8, 64)]
    if big:
        pool += [(64, 8, 128), (128, 8, 128)]
    return rng.choice(pool)


def _score_options(rng, c):
    kind = rng.choice(["plain", "plain", "plain", "alibi", "softcap", "relpos"])
    if kind == "alibi":
        c["alibi"] = True
        if rng.random() < 0.4:
            c["softcap"] = 50.0
    elif kind == "softcap":
        c["softcap"] = rng.choice([30.0, 50.0])
    elif kind == "relpos":
        c["relpos"] = True


def _fit_batch(rng, c, lo, hi):
    """Largest batch within the cost bounds, then a log-uniform one up to it;
    shorter sequences where even `lo` is too much."""
    while True:
        c["batch"] = lo
        w = work(c)
        room = min(_MAX_FLOPS[c.get("dtype", "bf16")] / w["flops"], _MAX_BYTES / w["bytes"])
        if room >= 1:
            break
        for k in ("sq", "sk", "q_hi", "c_hi"):
            if c.get(k, 0) > 1:
                c[k] = max(1, int(c[k] * 0.8))
        if "q_hi" in c:
            c["q_lo"], c["c_lo"] = min(c["q_lo"], c["q_hi"]), min(c["c_lo"], c["c_hi"])
        for k in ("prefix_len", "query_start"):
            if k in c:
                c[k] = int(c[k] * 0.8)
    c["batch"] = _log_int(rng, lo, max(lo, min(hi, int(lo * room))))


def draw(rng):
    fam = rng.choice(["fp32", "prompt", "prompt", "packed", "decode", "decode", "decode_packed",
                      "chunk", "chunk_packed", "index", "norm"])
    c = {"len_seed": rng.randrange(1 << 20)}
    hq, hkv, d = _heads(rng)
    c.update(hq=hq, hkv=hkv, d=d)
    if fam == "fp32":
        hq, hkv, d = rng.choice([(2, 2, 64), (8, 8, 64), (16, 4, 128), (8, 2, 128)])
        s = _log_int(rng, 64, 1500)
        c.update(dtype="fp32", hq=hq, hkv=hkv, d=d, sq=s, sk=s,
                 mask=rng.choice(["none", "causal", "causal", "sliding_window"]))
        if c["mask"] == "sliding_window":
            c.update(window_left=_log_int(rng, 16, 512), window_right=0)
        _fit_batch(rng, c, 1, 4)
    elif fam == "prompt":
        s = _log_int(rng, 100, 8192)
        c.update(sq=s, sk=s, mask=rng.choice(["none", "causal", "causal", "sliding_window",
                                              "prefix_lm"]))
        if c["mask"] == "sliding_window":
            c.update(window_left=_log_int(rng, 64, 2048), window_right=rng.choice([0, 0, 64]))
        if c["mask"] == "prefix_lm":
            c["prefix_len"] = rng.randrange(1, s)
        _score_options(rng, c)
        _fit_batch(rng, c, 1, 16)
    elif fam == "packed":
        hi = _log_int(rng, 256, 8192)
        c.update(layout="packed", q_lo=max(1, hi // 32), q_hi=hi)
        if rng.random() < 0.3:
            c.update(mask="sliding_window", window_left=1023, window_right=0)
        _score_options(rng, c)
        _fit_batch(rng, c, 2, 48)
    elif fam == "decode":
        c.update(sq=rng.choice([1, 1, 1, 2, 4]), sk=_log_int(rng, 200, 16384))
        _score_options(rng, c)
        _fit_batch(rng, c, 1, 64)
    elif fam == "decode_packed":
        hi = _log_int(rng, 512, 16384)
        c.update(layout="packed", q_lo=1, q_hi=rng.choice([1, 1, 4]), c_lo=hi // 32, c_hi=hi)
        if rng.random() < 0.3:
            c.update(mask="sliding_window", window_left=1023, window_right=0)
        _score_options(rng, c)
        _fit_batch(rng, c, 2, 64)
    elif fam == "chunk":
        sq = _log_int(rng, 33, 1024)
        c.update(sq=sq, sk=sq + _log_int(rng, 256, 12288))
        _score_options(rng, c)
        _fit_batch(rng, c, 1, 8)
    elif fam == "chunk_packed":
        hi = _log_int(rng, 64, 1024)
        c.update(layout="packed", q_lo=1, q_hi=hi, c_lo=128, c_hi=_log_int(rng, 512, 12288))
        _score_options(rng, c)
        _fit_batch(rng, c, 2, 16)
    elif fam == "index":
        s = _log_int(rng, 500, 8192)
        c.update(sq=s, sk=s, mask=rng.choice(["global_sliding_window", "share_question",
                                              "causal_blockwise"]))
        if c["mask"] == "global_sliding_window":
            w = _log_int(rng, 64, 512)
            c.update(window_left=w, window_right=w, num_global=_log_int(rng, 1, 64),
                     listed_global=rng.random() < 0.5)
        elif c["mask"] == "share_question":
            c.update(prefix_len=s // 4, num_segments=rng.randrange(2, 9))
        else:
            c.update(query_start=s * 3 // 4, num_segments=rng.randrange(2, 9))
        _fit_batch(rng, c, 1, 8)
    else:
        s = _log_int(rng, 200, 6000)
        c.update(sq=s, sk=s, mask=rng.choice(["causal", "none", "prefix_lm"]),
                 norm=rng.choice(["relu", "sigmoid"]), softcap=rng.choice([0.0, 0.0, 50.0]))
        if c["mask"] == "prefix_lm":
            c["prefix_len"] = s // 4
        _fit_batch(rng, c, 1, 8)
    return c


# ---- layouts --------------------------------------------------------------

def _lengths(c):
    """[(query length, key length)] of the case's sequences."""
    if c["layout"] == "fixed":
        return [(c["sq"], c["sk"])] * c["batch"]
    rng = random.Random(c["len_seed"])
    out = []
    for _ in range(c["batch"]):
        q = rng.randint(c["q_lo"], c["q_hi"])
        out.append((q, q + rng.randint(c["c_lo"], c["c_hi"])))
    return out


def _segments(c):
    """Segment starts (share question: from the prompt's end; causal
    blockwise: documents over [0, query_start))."""
    lo, hi = (c["prefix_len"], c["sk"]) if c["mask"] == "share_question" else (0, c["query_start"])
    rng = random.Random(c["len_seed"] + 1)
    cuts = rng.sample(range(lo + 1, hi), min(c["num_segments"] - 1, max(0, hi - lo - 1)))
    return [lo] + sorted(cuts)


def _globals(c):
    """Listed global positions, scattered over the sequence."""
    rng = random.Random(c["len_seed"] + 2)
    return sorted(rng.sample(range(c["sk"]), min(c["num_global"], c["sk"])))


def _row_ranges(c, lq, lk):
    """Per query row: keys j < pfx and lo <= j <= hi are visible (pfx < lo)."""
    i = np.arange(lq, dtype=np.int64) + (lk - lq)
    pfx = np.zeros(lq, np.int64)
    lo = np.zeros(lq, np.int64)
    hi = np.full(lq, lk - 1, np.int64)
    m = c["mask"]
    if m == "causal":
        hi = np.minimum(hi, i)
    elif m == "prefix_lm":
        hi = np.minimum(hi, np.maximum(i, c["prefix_len"] - 1))
    elif m in ("sliding_window", "global_sliding_window"):
        if c["window_left"] >= 0:
            lo = np.maximum(0, i - c["window_left"])
        if c["window_right"] >= 0:
            hi = np.minimum(hi, i + c["window_right"])
    elif m in ("share_question", "causal_blockwise"):
        seg = np.array(_segments(c), np.int64)
        k = np.searchsorted(seg, i, side="right") - 1
        start = np.where(k >= 0, seg[np.maximum(k, 0)], 0)
        hi = np.minimum(hi, i)
        if m == "share_question":
            lo = start
            pfx = np.where(k >= 0, np.minimum(seg[0], start), 0)
        else:
            lo = np.where(i >= c["query_start"], 0, start)
    return pfx, lo, hi


def _global_set(c):
    return _globals(c) if c["listed_global"] else list(range(min(c["num_global"], c["sk"])))


def _pairs(c, lq, lk):
    pfx, lo, hi = _row_ranges(c, lq, lk)
    n = pfx + np.maximum(0, hi - lo + 1)
    if c["mask"] == "global_sliding_window" and c["num_global"]:
        g = np.array(_global_set(c), np.int64)
        inside = np.searchsorted(g, hi, side="right") - np.searchsorted(g, lo, side="left")
        n = n + len(g) - inside
        pos = np.arange(lq, dtype=np.int64) + (lk - lq)
        n[np.isin(pos, g)] = lk
    return int(n.sum())


def _keys_read(c, lq, lk):
    """Keys that some row of the sequence sees (a closed range in every family here)."""
    pfx, lo, hi = _row_ranges(c, lq, lk)
    if c["mask"] in ("global_sliding_window", "share_question", "causal_blockwise"):
        return lk
    return int(max(0, hi.max() - lo.min() + 1))


def work(case):
    c = _full(case)
    elt = 2 if c["dtype"] == "bf16" else 4
    flops = nbytes = 0
    for lq, lk in _lengths(c):
        flops += 4 * c["d"] * c["hq"] * _pairs(c, lq, lk)
        nbytes += elt * c["d"] * (2 * lq * c["hq"] + 2 * _keys_read(c, lq, lk) * c["hkv"])
        if c["norm"] == "softmax":
            nbytes += 4 * lq * c["hq"]
    return {"bytes": nbytes, "flops": flops}


# ---- inputs and calls -----------------------------------------------------

def _inputs(c, seed):
    dev = torch.device("cuda")
    g = torch.Generator(device=dev).manual_seed(seed)
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    lens = _lengths(c)
    if c["layout"] == "fixed":
        qs = (c["batch"], c["hq"], c["sq"], c["d"])
        ks = (c["batch"], c["hkv"], c["sk"], c["d"])
    else:
        qs = (sum(a for a, _ in lens), c["hq"], c["d"])
        ks = (sum(b for _, b in lens), c["hkv"], c["d"])

    def one(shape):
        return (torch.randn(shape, generator=g, device=dev) * c["sigma"]).to(dt)

    return one(qs), one(ks), one(ks), lens


def _slopes(c):
    return [2.0 ** (-8.0 * h / c["hq"]) for h in range(1, c["hq"] + 1)]


def _i32(values):
    return torch.tensor(values, dtype=torch.int32, device="cuda")


def prepare(case, seed):
    c = _full(case)
    q, k, v, lens = _inputs(c, seed)
    kw = dict(mask=c["mask"], softcap=c["softcap"], relative_position=c["relpos"], norm=c["norm"])
    if c["mask"] in ("sliding_window", "global_sliding_window"):
        kw["window"] = (c["window_left"], c["window_right"])
    if c["mask"] == "prefix_lm":
        kw["prefix_len"] = c["prefix_len"]
    if c["mask"] == "global_sliding_window":
        if c["listed_global"]:
            kw["global_tokens"] = _i32(_globals(c))
        else:
            kw["num_global"] = c["num_global"]
    if c["mask"] in ("share_question", "causal_blockwise"):
        kw["segment_starts"] = _i32(_segments(c))
        kw["query_start"] = c["query_start"]
    if c["alibi"]:
        kw["alibi_slopes"] = torch.tensor(_slopes(c), dtype=torch.float32, device="cuda")
    if c["layout"] == "packed":
        kw["cu_seqlens_q"] = _i32(np.cumsum([0] + [a for a, _ in lens]).tolist())
        kw["cu_seqlens_k"] = _i32(np.cumsum([0] + [b for _, b in lens]).tolist())
        kw["max_seqlen_q"] = max(a for a, _ in lens)
        kw["max_seqlen_k"] = max(b for _, b in lens)
    return {"q": q, "k": k, "v": v, "kw": kw}


def run(state):
    return attn.fwd(state["q"], state["k"], state["v"], **state["kw"])


def tolerance(case):
    # fp32: rounding of the sums. bf16: P and O are rounded to 8 bits (about
    # 2e-3 each over a whole output).
    return {"rel": 1e-5} if _full(case)["dtype"] == "fp32" else {"rel": 1e-2}


# ---- 64-bit reference -----------------------------------------------------

def _exact_one(c, q, k, v, lq, lk, slopes):
    """Attention of one sequence in float64: q [Hq, lq, D], k/v [Hkv, lk, D]."""
    dev = q.device
    group = c["hq"] // c["hkv"]
    out = torch.empty(q.shape, dtype=torch.float64, device=dev)
    lse = torch.empty(q.shape[:2], dtype=torch.float64, device=dev)
    pfx, lo, hi = (torch.from_numpy(x).to(dev) for x in _row_ranges(c, lq, lk))
    j = torch.arange(lk, device=dev)
    ip = torch.arange(lq, device=dev) + (lk - lq)
    gset = torch.zeros(max(lk, 1), dtype=torch.bool, device=dev)
    if c["mask"] == "global_sliding_window" and c["num_global"]:
        gset[torch.tensor(_global_set(c), device=dev)] = True
    rows = max(1, (1 << 26) // max(1, lk))
    for h in range(c["hkv"]):
        kt = k[h].double().t().contiguous()
        vh = v[h].double().contiguous()
        for r0 in range(0, lq, rows):
            r1 = min(lq, r0 + rows)
            dist = (ip[r0:r1, None] - j[None, :])
            vis = (j[None, :] < pfx[r0:r1, None]) | ((j[None, :] >= lo[r0:r1, None]) &
                                                     (j[None, :] <= hi[r0:r1, None]))
            if c["mask"] == "global_sliding_window" and c["num_global"]:
                vis = vis | gset[None, :lk] | gset[ip[r0:r1], None]
            for u in range(group):
                hq = h * group + u
                s = (q[hq, r0:r1].double() @ kt) / math.sqrt(c["d"])
                if c["softcap"]:
                    s = c["softcap"] * torch.tanh(s / c["softcap"])
                if c["alibi"]:
                    s = s - slopes[hq] * dist.abs().double()
                if c["relpos"]:
                    s = s + dist.double()
                s = s.masked_fill(~vis, -math.inf)
                if c["norm"] == "softmax":
                    m = s.amax(dim=1, keepdim=True)
                    m = torch.where(m == -math.inf, torch.zeros_like(m), m)
                    p = torch.exp(s - m)
                    total = p.sum(dim=1, keepdim=True)
                    lse[hq, r0:r1] = (m + torch.log(total))[:, 0]
                    p = p / torch.where(total > 0, total, torch.ones_like(total))
                elif c["norm"] == "relu":
                    p = torch.relu(s) / lk
                else:
                    p = torch.sigmoid(s) / lk
                out[hq, r0:r1] = p @ vh
    return out, lse


def exact(case, seed):
    c = _full(case)
    q, k, v, lens = _inputs(c, seed)
    # the slopes as the call takes them (fp32)
    slopes = torch.tensor(_slopes(c), dtype=torch.float32).double().tolist()
    out = torch.empty(q.shape, dtype=torch.float64, device=q.device)
    if c["layout"] == "fixed":
        lse = torch.empty(q.shape[:3], dtype=torch.float64, device=q.device)
        for b, (lq, lk) in enumerate(lens):
            out[b], lse[b] = _exact_one(c, q[b], k[b], v[b], lq, lk, slopes)
    else:
        lse = torch.empty((c["hq"], q.shape[0]), dtype=torch.float64, device=q.device)
        a = b = 0
        for lq, lk in lens:
            o, l = _exact_one(c, q[a:a + lq].transpose(0, 1), k[b:b + lk].transpose(0, 1),
                              v[b:b + lk].transpose(0, 1), lq, lk, slopes)
            out[a:a + lq] = o.transpose(0, 1)
            lse[:, a:a + lq] = l
            a, b = a + lq, b + lk
    return (out, lse) if c["norm"] == "softmax" else out
