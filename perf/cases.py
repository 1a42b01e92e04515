"""The work a serving program has the segment re-prefill library do, as timed cases.

Each case is a dict of plain values; `kind` names the calls one pass makes:

  attn    sa_segment_prefill_attn over a cache that already holds everything
          (decode steps, one attention call of a layer)
  append  sa_segment_prefill_attn_append: a segment's rows go into the cache,
          then its attention
  alias   sa_kv_splice_alias, sa_kv_append, sa_segment_prefill_attn: a turn of an
          agent on a prefix whose pages stay where they are
  commit  sa_kv_assemble_append, sa_segment_prefill_attn: the commit splice into
          fresh pages with the segment's append, then its attention
  splice  sa_kv_assemble alone, over every layer of the pool

`n` sequences carry a segment of q_lo..q_hi tokens behind a prefix of pre_lo..pre_hi
tokens, `dec` more are decode requests (one query token) with ctx_lo..ctx_hi cached
tokens; lengths are drawn from `lens`, contents from the seed that prepare() is given:
N(0, 1) / 2 rounded to bf16 on a shuffled page pool, the distribution of the named
configurations c1..c5, with 1% of the key rows times 8 where `outliers` is set (c4's
recipe).  `folded` asks for the folded-scale mode, `noalloc` for the allocation-free
entry point.
"""
import math
import random

import numpy as np
import torch

import paper_2607_00151_amd as sa

D = 128


def _case(name, kind, heads, page, n=0, pre=(0, 0), q=(0, 0), dec=0, ctx=(0, 0), lens=1, layers=1, outliers=False,
          folded=False, noalloc=False):
    c = {"kind": kind, "Hq": heads[0], "Hkv": heads[1], "page": page, "layers": layers, "n": n, "pre_lo": pre[0],
         "pre_hi": pre[1], "q_lo": q[0], "q_hi": q[1], "dec": dec, "ctx_lo": ctx[0], "ctx_hi": ctx[1], "lens": lens,
         "outliers": outliers, "folded": folded, "noalloc": noalloc}
    return dict(c, name=name) if name else c


def listed():
    return [
        # a decode step of a few interactive requests with short contexts: the smallest call of a serving loop
        _case("decode_few", "attn", (32, 8), 16, dec=4, ctx=(1024, 4096)),
        # configuration c1: a small model's segment, append and attention in one call
        _case("segment_c1", "append", (8, 2), 16, n=1, pre=(512, 512), q=(256, 256)),
        # one 256-token chunk of a chunked prefill over a 4K prefix, from a loop that must not allocate
        _case("chunk_256", "attn", (32, 8), 16, n=1, pre=(4096, 4096), q=(256, 256), noalloc=True),
        # a decode step of a full batch (c5's 64 decode requests)
        _case("decode_batch", "attn", (32, 8), 16, dec=64, ctx=(4096, 16384)),
        # one decode row on a very long context (c4's layout after its segment)
        _case("decode_long", "attn", (64, 8), 32, dec=1, ctx=(73729, 73729)),
        # short instruction chunks streamed onto 32 sub-agent contexts of ~8K
        _case("short_segments", "alias", (32, 8), 16, n=32, pre=(8000, 8300), q=(16, 64)),
        # one agent turn of 600-650 tokens on its context, folded-scale mode
        _case("turn_folded", "alias", (32, 8), 16, n=1, pre=(12007, 12007), q=(631, 631), folded=True),
        # configuration c2: the commit of an 8K prefix and its 2K segment
        _case("commit_c2", "commit", (32, 8), 16, n=1, pre=(8192, 8192), q=(2048, 2048)),
        # the commit splice of c2's prefix alone, over eight layers in one launch
        _case("splice_layers", "splice", (32, 8), 16, n=1, pre=(8192, 8192), q=(2048, 2048), layers=8),
        # configuration c5: decode requests and prefill segments in one launch
        _case("mixed_c5", "append", (32, 8), 16, n=4, pre=(16384, 16384), q=(2048, 2048), dec=64, ctx=(4096, 16384)),
        # configuration c3: the commit of 16 ragged contexts
        _case("ragged_c3", "commit", (32, 8), 16, n=16, pre=(4096, 32768), q=(512, 4096)),
        # configuration c4: an 8K segment on a 64K context, outlier keys
        _case("long_c4", "attn", (64, 8), 32, n=1, pre=(65536, 65536), q=(8192, 8192), outliers=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _span(rng, lo, hi, ragged):
    """A range of lengths inside [lo, hi], a single length unless ragged."""
    a, b = sorted((_log(rng, lo, hi), _log(rng, lo, hi)))
    return (a, b) if ragged else (b, b)


def draw(rng):
    """One more case of the ranges the listed ones span."""
    while True:
        kind = rng.choice(["attn", "attn", "append", "alias", "commit", "splice"])
        heads, page = rng.choice([((32, 8), 16), ((32, 8), 16), ((64, 8), 32), ((8, 2), 16), ((32, 4), 32)])
        lens = rng.randrange(1 << 20)
        folded = rng.random() < 0.15
        if kind == "attn" and rng.random() < 0.6:                      # a decode step
            dec = _log(rng, 1, 64)
            c = _case(None, "attn", heads, page, dec=dec, ctx=_span(rng, 512, 131072 // max(1, dec // 4), dec > 1),
                      lens=lens, folded=folded, noalloc=rng.random() < 0.2)
        elif kind == "splice":
            c = _case(None, "splice", heads, page, n=rng.randint(1, 4), pre=_span(rng, 1000, 16384, True),
                      q=_span(rng, 16, 2048, True), layers=rng.choice([1, 2, 4, 8]), lens=lens)
        else:
            n = _log(rng, 1, 32)
            mixed = kind == "append" and rng.random() < 0.5
            c = _case(None, kind, heads, page, n=n, pre=_span(rng, 256, 65536, True), q=_span(rng, 16, 8192, True),
                      dec=_log(rng, 1, 64) if mixed else 0, ctx=_span(rng, 1024, 16384, True) if mixed else (0, 0),
                      lens=lens, folded=folded, outliers=rng.random() < 0.2)
        w = work(c)
        if w["flops"] <= 1.2e13 and w["bytes"] <= 3e9:
            return c


# ------------------------------------------------------------------------- shapes

def _lengths(case):
    """(pre, q) of every sequence: segments first, then decode rows (prefix = context - 1)."""
    r = random.Random(case["lens"])
    pre = [r.randint(case["pre_lo"], case["pre_hi"]) for _ in range(case["n"])]
    q = [r.randint(case["q_lo"], case["q_hi"]) for _ in range(case["n"])]
    pre += [r.randint(case["ctx_lo"], case["ctx_hi"]) - 1 for _ in range(case["dec"])]
    return np.array(pre, dtype=np.int64), np.array(q + [1] * case["dec"], dtype=np.int64)


def _dropped(case, pre):
    """Per sequence: (first dropped page, dropped pages) of the source cache, a quarter of it, never page 0."""
    r = random.Random(case["lens"] + 17)
    full = [int(x) // case["page"] for x in pre]
    return [(r.randint(1, max(1, f)), -(-f // 3)) for f in full]


def _pages(x, P):
    return -(-np.asarray(x, dtype=np.int64) // P)


def work(case):
    pre, q = _lengths(case)
    Hq, Hkv, P = case["Hq"], case["Hkv"], case["page"]
    row = Hkv * D * 2 * 2                                    # K and V of one token
    moved = 0
    if case["kind"] in ("commit", "splice"):
        moved += 2 * int(_pages(pre, P).sum()) * P * row * case["layers"]
    if case["kind"] in ("append", "alias", "commit"):
        moved += 2 * int(q.sum()) * row
    flops = 0.0
    if case["kind"] != "splice":
        pairs = int((q * pre + q * (q + 1) // 2).sum())
        flops = 4.0 * D * Hq * pairs
        moved += int((pre + q).sum()) * row + int(q.sum()) * Hq * (2 * D * 2 + 4)
    return {"bytes": float(moved), "flops": flops}


def tolerance(case):
    """Splices move bits.  O is bf16 (one rounding, 2^-9) of sums whose probabilities were rounded to bf16: measured
    against the 64-bit result it is off by 2.0e-3 to 2.4e-3 (2-norm) in every case, folded scale or not, and by up
    to about six times that in single values; four times both."""
    if case["kind"] == "splice":
        return "exact"
    return {"rel": 1e-2, "max": 0.1}


# ------------------------------------------------------------------------- inputs

def _rows(g, shape):
    t = torch.empty(shape, dtype=torch.int16, device="cuda")
    flat = t.view(-1)
    step = 1 << 28
    for i in range(0, flat.numel(), step):
        n = min(step, flat.numel() - i)
        flat[i:i + n] = torch.randn(n, generator=g, device="cuda").mul_(0.5).to(torch.bfloat16).view(torch.int16)
    return t


def _table(lists):
    indptr = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int32)
    flat = torch.cat(lists) if lists else torch.zeros(0, dtype=torch.int32, device="cuda")
    return torch.from_numpy(indptr).cuda(), flat.contiguous()


def _inputs(case, seed):
    """Everything in plain torch and numpy: pools, tables, rows and host lengths."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    pre, q = _lengths(case)
    P, Hkv, Hq, B = case["page"], case["Hkv"], case["Hq"], len(q)
    x = {"pre": pre, "q_len": q.astype(np.int32), "kv_len": (pre + q).astype(np.int32)}
    cut = _dropped(case, pre) if case["kind"] in ("commit", "splice") else [(0, 0)] * B
    n_src = [int(_pages(p, P)) + nd for p, (_, nd) in zip(pre, cut)]
    n_all = _pages(pre + q, P)
    aliased = case["kind"] == "alias"
    if case["kind"] in ("commit", "splice"):
        n_fresh = int(n_all.sum())
    elif aliased:
        n_fresh = int((n_all - _pages(pre, P)).sum())
    else:
        n_src, n_fresh = [int(v) for v in n_all], 0
    need = sum(n_src) + n_fresh
    x["num_slots"] = max(16, need + need // 2)
    shape = (case["layers"], x["num_slots"], Hkv, P, D)
    x["k"], x["v"] = _rows(g, shape), _rows(g, shape)
    if case["outliers"]:
        kf = x["k"].view(-1, D).view(torch.bfloat16)
        hit = torch.randperm(kf.shape[0], generator=g, device="cuda")[:kf.shape[0] // 100]
        kf[hit] = kf[hit] * 8
    perm = torch.randperm(x["num_slots"], generator=g, device="cuda").to(torch.int32)
    at, lists = 0, []
    for n in n_src:
        lists.append(perm[at:at + n])
        at += n
    x["indptr"], x["indices"] = _table(lists)
    x["fresh"] = perm[at:at + n_fresh].contiguous()
    if case["kind"] in ("commit", "splice", "alias"):
        spans, keep = [], [0]
        for b in range(B):
            a, nd = cut[b]
            spans += [s for s in ((0, a), (a + nd, n_src[b])) if s[0] < s[1]] if nd else [(0, n_src[b])]
            keep.append(len(spans))
        x["keep_indptr"], x["keep_spans"] = np.array(keep, dtype=np.int32), np.array(spans, dtype=np.int32)
        x["src_len"] = np.array([p + nd * P for p, (_, nd) in zip(pre, cut)], dtype=np.int32)
        x["dst_indptr"] = torch.zeros(B + 1, dtype=torch.int32, device="cuda")
        x["dst_indices"] = torch.zeros(int(n_all.sum()), dtype=torch.int32, device="cuda")
    if case["kind"] != "splice":
        T = int(q.sum())
        x["q"] = _rows(g, (T, Hq, D))
        x["o"] = torch.empty((T, Hq, D), dtype=torch.bfloat16, device="cuda")
        x["lse"] = torch.empty((T, Hq), dtype=torch.float32, device="cuda")
        if case["kind"] != "attn":
            x["k_new"], x["v_new"] = _rows(g, (T, Hkv, D)), _rows(g, (T, Hkv, D))
    return x


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    s["layout"] = sa.Layout(num_q_heads=case["Hq"], num_kv_heads=case["Hkv"], head_dim=D, page_size=case["page"],
                            num_layers=case["layers"], num_slots=s["num_slots"])
    s["ctx"] = sa.Context(0)
    if case["folded"]:
        sa.sa_set_exact_scale(s["ctx"], False)
    return s


def run(s):
    c, ctx, L, scale = s["case"], s["ctx"], s["layout"], D ** -0.5
    kind = c["kind"]
    if kind == "splice":
        sa.sa_kv_assemble(ctx, L, s["k"], s["v"], s["k"], s["v"], s["src_len"], s["keep_indptr"], s["keep_spans"],
                          s["q_len"], s["indptr"], s["indices"], s["fresh"], s["dst_indptr"], s["dst_indices"])
        return [s["k"], s["v"], s["dst_indptr"], s["dst_indices"]]
    if kind == "append":
        sa.sa_segment_prefill_attn_append(ctx, L, 0, s["q"], s["k"], s["v"], s["k_new"], s["v_new"], s["q_len"],
                                          s["kv_len"], s["indptr"], s["indices"], scale, s["o"], s["lse"])
        return [s["o"], s["lse"], s["k"], s["v"]]
    if kind == "attn":
        call = sa.sa_segment_prefill_attn_noalloc if c["noalloc"] else sa.sa_segment_prefill_attn
        call(ctx, L, 0, s["q"], s["k"], s["v"], s["q_len"], s["kv_len"], s["indptr"], s["indices"], scale, s["o"],
             s["lse"])
        return [s["o"], s["lse"]]
    if kind == "commit":
        kept = sa.sa_kv_assemble_append(ctx, L, s["k"], s["v"], s["k"], s["v"], s["src_len"], s["keep_indptr"],
                                        s["keep_spans"], s["q_len"], s["indptr"], s["indices"], s["fresh"],
                                        s["dst_indptr"], s["dst_indices"], 0, s["k_new"], s["v_new"], s["q_len"])
    else:
        kept = sa.sa_kv_splice_alias(ctx, L, s["src_len"], s["keep_indptr"], s["keep_spans"], s["q_len"], s["indptr"],
                                     s["indices"], s["fresh"], s["dst_indptr"], s["dst_indices"])
        sa.sa_kv_append(ctx, L, 0, s["k"], s["v"], s["k_new"], s["v_new"], kept, s["q_len"], s["dst_indptr"],
                        s["dst_indices"])
    sa.sa_segment_prefill_attn(ctx, L, 0, s["q"], s["k"], s["v"], s["q_len"], kept + s["q_len"], s["dst_indptr"],
                               s["dst_indices"], scale, s["o"], s["lse"])
    return [s["o"], s["lse"], s["k"], s["v"], s["dst_indptr"], s["dst_indices"]]


# ------------------------------------------------------------------------- 64-bit reference

def _attend(q, k, v, G, scale):
    """q [n][Hq][D], k and v [kv][Hkv][D] of one sequence, in float64: (o, lse)."""
    n, kv, Hkv = q.shape[0], k.shape[0], k.shape[1]
    o, lse = torch.empty_like(q), torch.empty(q.shape[:2], dtype=torch.float64, device=q.device)
    key = torch.arange(kv, device=q.device)
    step = max(1, (1 << 26) // (kv * G))
    for h in range(Hkv):
        kt, vh = k[:, h].t().contiguous(), v[:, h].contiguous()
        for i in range(0, n, step):
            j = min(n, i + step)
            s = (q[i:j, h * G:(h + 1) * G].reshape(-1, D) @ kt).mul_(scale)
            last = (kv - n + torch.arange(i, j, device=q.device)).repeat_interleave(G)
            s.masked_fill_(key[None, :] > last[:, None], -math.inf)
            m = s.amax(dim=1, keepdim=True)
            s = s.sub_(m).exp_()
            t = s.sum(dim=1, keepdim=True)
            o[i:j, h * G:(h + 1) * G] = ((s @ vh) / t).view(j - i, G, D)
            lse[i:j, h * G:(h + 1) * G] = (m + t.log()).view(j - i, G)
    return o, lse


def exact(case, seed):
    if case["kind"] == "splice":
        return None
    x = _inputs(case, seed)
    P, Hkv, G = case["page"], case["Hkv"], case["Hq"] // case["Hkv"]

    def f64(t):
        return t.view(torch.bfloat16).double()

    ip = x["indptr"].tolist()
    o = torch.empty(x["o"].shape, dtype=torch.float64, device="cuda")
    lse = torch.empty(x["lse"].shape, dtype=torch.float64, device="cuda")
    t0 = 0
    for b, (p, n) in enumerate(zip(x["pre"].tolist(), x["q_len"].tolist())):
        slots = x["indices"][ip[b]:ip[b + 1]].long()
        if "keep_spans" in x:
            spans = x["keep_spans"][x["keep_indptr"][b]:x["keep_indptr"][b + 1]]
            slots = torch.cat([slots[a:e] for a, e in spans.tolist()])
        kv = []
        for pool in ("k", "v"):
            rows = x[pool][0][slots].transpose(1, 2).reshape(-1, Hkv, D)
            if case["kind"] == "attn":
                kv.append(f64(rows[:p + n]))
            else:
                kv.append(f64(torch.cat([rows[:p], x[pool + "_new"][t0:t0 + n]])))
        o[t0:t0 + n], lse[t0:t0 + n] = _attend(f64(x["q"][t0:t0 + n]), kv[0], kv[1], G, D ** -0.5)
        t0 += n
    tail = {"attn": 0, "append": 2, "alias": 4, "commit": 4}[case["kind"]]
    return [o, lse] + [None] * tail
