"""Performance cases of the decode-step attention: what a serving engine calls this library for.

A case is one batch shape (how many serial requests, how many requests in a parallel phase, how long
their contexts are), one attention shape (heads, head_dim), and the options a caller chooses (format of
the partial rows, log-sum-exp output).  Most cases are the attention of one layer with the step's plan in
hand, as a model's layer loop calls it; one is a whole decode step (KV append, plan, attention of all
layers).  Lengths are fixed by the case; page placement and values are drawn from the seed.

Values are N(0,1) rounded to bf16 everywhere, in every page of the pool, pages of a sequence scattered
over the pool, as an engine that has been running for a while leaves them.
"""
import math

import numpy as np
import torch

from paper_2605_06914_amd import Context, append_slots

PAGE = 16
DEVICE = "cuda:0"

# --------------------------------------------------------------------------- cases
BASE = dict(
    hq=64, hkv=8, d=128,          # the 64-query-head / 8-KV-head shape the benchmark is quoted on
    serial=0, ctx_lo=0, ctx_hi=0,  # serial requests: count, context range
    parallel=0, pre_lo=0, pre_hi=0, width_lo=0, width_hi=0, suf_lo=0, suf_hi=0,  # requests in a parallel phase
    reduce=0,                      # how many of the parallel requests are in their reduce phase
    lens=0,                        # seed of the lengths
    partial="f16_scaled", lse=False,
    layers=0,                      # > 0: a whole decode step of that many layers; 0: one layer's attention
)


def _case(name=None, **kw):
    c = dict(BASE, **kw)
    return c if name is None else dict(name=name, **c)


MIXED = dict(serial=16, ctx_lo=1024, ctx_hi=4096, parallel=8, pre_lo=2048, pre_hi=8192, width_lo=4, width_hi=8,
             suf_lo=0, suf_hi=1024, lens=20260503)


def listed():
    return [
        # the smallest call: five short sequences of a small model (launch and latency)
        _case("tiny", hq=4, hkv=1, d=64, serial=1, ctx_lo=256, ctx_hi=256, parallel=1, pre_lo=192, pre_hi=192,
              width_lo=4, width_hi=4, suf_lo=0, suf_hi=32, lens=20260501),
        # one user, one request: interactive latency
        _case("one_request", serial=1, ctx_lo=2048, ctx_hi=2048, lens=1),
        # a chat server full of short contexts
        _case("short_serial", serial=512, ctx_lo=32, ctx_hi=512, lens=2),
        # branch parallelism off: serial requests only
        _case("irp_off", serial=32, ctx_lo=1024, ctx_hi=4096, lens=20260502),
        # the benchmark's headline batch: serial requests beside requests with 4 to 8 branches
        _case("mixed", **MIXED),
        # the same batch on one rank of a tensor-parallel group of eight: one KV head and its 8 query heads
        _case("mixed_tp8", hq=8, hkv=1, **MIXED),
        # the same batch on a model with head_dim 64 and 4 query heads per KV head, fp32 partial rows, lse wanted
        _case("mixed_d64", hq=32, hkv=8, d=64, partial="f32", lse=True, **MIXED),
        # long shared documents: 8 requests with a 32768-token prefix and 16 branches each
        _case("long_prefix", serial=32, ctx_lo=1024, ctx_hi=8192, parallel=8, pre_lo=32768, pre_hi=32768,
              width_lo=16, width_hi=16, suf_lo=0, suf_hi=2048, lens=20260504),
        # requests wider than one workgroup's query rows: 64 branches
        _case("wide64", serial=16, ctx_lo=1024, ctx_hi=4096, parallel=8, pre_lo=2048, pre_hi=8192,
              width_lo=64, width_hi=64, suf_lo=0, suf_hi=1024, lens=20260506),
        # half of the parallel requests have joined their branches and decode the reduce phase
        _case("reduce", serial=16, ctx_lo=512, ctx_hi=8192, parallel=8, pre_lo=1024, pre_hi=16384, width_lo=17,
              width_hi=17, suf_lo=0, suf_hi=2048, reduce=4, lens=3),
        # the largest batch: 96 serial and 32 parallel requests, all 17 branches of each admitted
        _case("sweep_full", serial=96, ctx_lo=512, ctx_hi=8192, parallel=32, pre_lo=1024, pre_hi=16384, width_lo=17,
              width_hi=17, suf_lo=0, suf_hi=2048, lens=20260505),
        # a whole decode step: append of the new tokens' K and V, the step's plan, the attention of four layers
        _case("decode_step", layers=4, **MIXED),
    ]


# attention shapes of the tests and the benchmark: (query heads, KV heads, head_dim)
SHAPES = [(64, 8, 128), (64, 8, 128), (64, 8, 128), (8, 1, 128), (16, 1, 128), (64, 4, 128), (6, 2, 128), (32, 8, 64),
          (8, 8, 64), (4, 1, 64)]
MOST_BYTES = 3 << 30


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        hq, hkv, d = rng.choice(SHAPES)
        c = _case(hq=hq, hkv=hkv, d=d, lens=rng.randrange(1 << 30), partial=rng.choice(["f16_scaled", "f16_scaled", "f32"]),
                  lse=rng.random() < 0.25)
        kind = rng.choice(["serial", "mixed", "mixed", "wide", "reduce", "step"])
        if kind == "serial" or rng.random() < 0.8:
            lo = log_int(1, 8192)
            c.update(serial=log_int(1, 512), ctx_lo=lo, ctx_hi=min(32768, log_int(lo, 4 * lo)))
        if kind != "serial":
            lo, suf = log_int(16, 32768), log_int(1, 2048)
            w = log_int(2, 17) if kind != "wide" else log_int(18, 64)
            c.update(parallel=log_int(1, 32), pre_lo=lo, pre_hi=min(32768, log_int(lo, 4 * lo)), width_lo=w,
                     width_hi=min(64, w + rng.randrange(0, 5)), suf_lo=rng.choice([0, 0, suf // 2]), suf_hi=suf)
        if kind == "reduce":
            c["reduce"] = rng.randint(1, c["parallel"])
        if kind == "step":
            c.update(layers=rng.randint(1, 4), lse=False)
        if work(c)["bytes"] <= MOST_BYTES:
            return c


# --------------------------------------------------------------------------- integers of a batch
def _requests(case):
    """Lengths: [(prefix, [[private segments of a sequence], ...]), ...]."""
    r = np.random.Generator(np.random.PCG64(case["lens"]))

    def some(lo, hi, n):
        return r.integers(lo, hi, size=n, endpoint=True) if lo < hi else np.full(n, lo)

    ctx = some(case["ctx_lo"], case["ctx_hi"], case["serial"])
    pre = some(case["pre_lo"], case["pre_hi"], case["parallel"])
    wid = some(case["width_lo"], case["width_hi"], case["parallel"])
    suf = [[int(x) for x in some(case["suf_lo"], case["suf_hi"], int(w))] for w in wid]
    grows = case["layers"] > 0  # a context that grows in place is its request's private segment
    reqs = [(0, [[int(c)]]) if grows else (int(c), [[0]]) for c in ctx]
    for i in range(case["parallel"]):
        if i < case["reduce"]:  # one sequence: prefix, every branch's pages, the reduce tokens so far
            reqs.append((int(pre[i]), [suf[i] + [1 + int(pre[i]) % 97]]))
        else:
            reqs.append((int(pre[i]), [[s] for s in suf[i]]))
    return reqs


def _pages(n):
    return (n + PAGE - 1) // PAGE


def _batch(case, seed):
    """Block table and lengths; the pages come from a random permutation of a pool with 10 % to spare."""
    grow = 1 if case["layers"] > 0 else 0  # (room for the token this step appends)
    reqs = _requests(case)
    used = sum(_pages(p) + sum(sum(_pages(x) for x in segs[:-1]) + _pages(segs[-1] + grow) for segs in seqs) for p, seqs in reqs)
    n_pages = max(1, math.ceil(1.1 * used))
    free = np.random.Generator(np.random.PCG64(seed)).permutation(n_pages).astype(np.int32)
    cur, rows, group, prefix, seg_start, seg_len = 0, [], [], [], [0], []
    for g, (p, seqs) in enumerate(reqs):
        shared = free[cur:cur + _pages(p)]
        cur += len(shared)
        for segs in seqs:
            n = sum(_pages(x) for x in segs[:-1]) + _pages(segs[-1] + grow)
            rows.append(np.concatenate([shared, free[cur:cur + n]]))
            cur += n
            group.append(g)
            prefix.append(p)
            seg_len += segs
            seg_start.append(len(seg_len))
    table = np.full((len(rows), max(1, max(len(r) for r in rows))), -1, np.int32)
    for s, row in enumerate(rows):
        table[s, :len(row)] = row
    as_i32 = lambda v: np.array(v, np.int32)  # noqa: E731
    return dict(table=table, group=as_i32(group), prefix=as_i32(prefix), seg_start=as_i32(seg_start), seg_len=as_i32(seg_len),
                n_pages=n_pages)


def _tensors(case, batch, seed):
    hq, hkv, d, S = case["hq"], case["hkv"], case["d"], len(batch["group"])
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed + 1000)

    def normal(*shape):
        return torch.empty(shape, device=DEVICE, dtype=torch.bfloat16).normal_(generator=gen)

    n = max(1, case["layers"])
    q = [normal(S, hq, d) for _ in range(n)]
    kv = [normal(batch["n_pages"], 2, hkv, PAGE * d) for _ in range(n)]
    new = [(normal(S, hkv, d), normal(S, hkv, d)) for _ in range(n)] if case["layers"] > 0 else []
    return q, kv, new


# --------------------------------------------------------------------------- the calls
_contexts = {}


def _context(case):
    """One context per attention shape and partial format for the life of the process, as an engine has it."""
    key = (case["hq"], case["hkv"], case["d"], case["partial"])
    if key not in _contexts:
        _contexts[key] = Context(key[0], key[1], key[2], device=0, partial_format=key[3])
    return _contexts[key]


def _plan(ctx, b, seg_len):
    if len(seg_len) == len(b["group"]):
        return ctx.plan_build(b["table"], b["group"], b["prefix"], seg_len, b["n_pages"])
    return ctx.plan_build_segments(b["table"], b["group"], b["prefix"], b["seg_start"], seg_len, b["n_pages"])


def prepare(case, seed):
    b = _batch(case, seed)
    q, kv, new = _tensors(case, b, seed)
    state = dict(case=case, ctx=_context(case), batch=b, q=q, kv=kv, new=new, out=[torch.empty_like(x) for x in q],
                 lse=torch.empty(len(b["group"]), case["hq"], device=DEVICE) if case["lse"] else None)
    if case["layers"] == 0:  # one plan serves all layers of a step: a layer's call finds it built
        state["plan"] = _plan(state["ctx"], b, b["seg_len"])
    return state


def run(state):
    ctx, b = state["ctx"], state["batch"]
    if state["case"]["layers"] == 0:
        ctx.decode_step_attention(state["plan"], state["q"][0], state["kv"][0], state["out"][0], state["lse"])
        return {"out": state["out"][0], "lse": state["lse"]}
    n = len(b["group"])
    slots, _ = append_slots(b["table"], b["prefix"], b["seg_start"], b["seg_len"], PAGE, b["n_pages"])
    slots = torch.from_numpy(slots).to(DEVICE, non_blocking=True)
    seg_len = b["seg_len"].copy()
    seg_len[b["seg_start"][1:] - 1] += 1
    plan = _plan(ctx, b, seg_len)
    for q, kv, (k_new, v_new), out in zip(state["q"], state["kv"], state["new"], state["out"]):
        ctx.kv_append(k_new, v_new, slots, kv, n)
        ctx.decode_step_attention(plan, q, kv, out)
    plan.free()
    return {"out": state["out"], "kv": state["kv"]}


# --------------------------------------------------------------------------- what a pass cannot do without
def work(case):
    """Every visible K and V element once (a shared prefix once per request), q and out once; two products of
    head_dim per query head and visible token."""
    reqs, layers = _requests(case), max(1, case["layers"])
    grow = 1 if case["layers"] > 0 else 0
    unique = sum(p + sum(sum(segs) + grow for segs in seqs) for p, seqs in reqs)
    logical = sum(sum(p + sum(segs) + grow for segs in seqs) for p, seqs in reqs)
    n = sum(len(seqs) for _, seqs in reqs)
    token = 2 * case["hkv"] * case["d"] * 2
    rows = n * case["hq"]
    return {"bytes": layers * (unique * token + 2 * rows * case["d"] * 2 + (rows * 4 if case["lse"] else 0) + grow * 2 * n * token),
            "flops": layers * 4 * logical * case["hq"] * case["d"]}


def tolerance(case):
    # bf16 products accumulated in 32 bits, probabilities and results rounded to bf16
    return {"rel": 1e-2, "max": 6e-2}


# --------------------------------------------------------------------------- the same in 64 bits
def _rows(kv, pages, n, which, hkv, d):
    """K (which 0) or V (1) of the first n tokens of `pages`, [hkv, n, d]: a K tile is [d/8][token][8], a V tile
    [token/4][d][4]."""
    t = kv[pages, which]
    if which == 0:
        t = t.view(len(pages), hkv, d // 8, PAGE, 8).permute(1, 0, 3, 2, 4)
    else:
        t = t.view(len(pages), hkv, PAGE // 4, d, 4).permute(1, 0, 2, 4, 3)
    return t.reshape(hkv, len(pages) * PAGE, d)[:, :n].double().contiguous()


def _attention(case, b, q, kv):
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    g, grow = hq // hkv, 1 if case["layers"] > 0 else 0
    S = len(b["group"])
    out = torch.empty(S, hq, d, device=DEVICE, dtype=torch.float64)
    lse = torch.empty(S, hq, device=DEVICE, dtype=torch.float64)
    table = torch.from_numpy(b["table"].astype(np.int64)).to(DEVICE)
    shared = (-1, None, None)
    for s in range(S):
        p = int(b["prefix"][s])
        if shared[0] != b["group"][s]:
            pages = table[s, :_pages(p)]
            shared = (b["group"][s], _rows(kv, pages, p, 0, hkv, d), _rows(kv, pages, p, 1, hkv, d))
        k, v, cur = [shared[1]], [shared[2]], _pages(p)
        segs = [int(x) for x in b["seg_len"][b["seg_start"][s]:b["seg_start"][s + 1]]]
        segs[-1] += grow
        for n in segs:
            pages = table[s, cur:cur + _pages(n)]
            cur += _pages(n)
            k.append(_rows(kv, pages, n, 0, hkv, d))
            v.append(_rows(kv, pages, n, 1, hkv, d))
        k, v = torch.cat(k, 1), torch.cat(v, 1)
        score = torch.matmul(q[s].double().view(hkv, g, d), k.transpose(1, 2).contiguous()) * d ** -0.5
        lse[s] = torch.logsumexp(score, -1).view(hq)
        out[s] = torch.matmul(torch.softmax(score, -1), v).view(hq, d)
    return out, lse


def exact(case, seed):
    b = _batch(case, seed)
    q, kv, new = _tensors(case, b, seed)
    if case["layers"] == 0:
        out, lse = _attention(case, b, q[0], kv[0])
        return {"out": out, "lse": lse if case["lse"] else None}
    hkv, d, outs = case["hkv"], case["d"], []
    for l in range(case["layers"]):
        for s in range(len(b["group"])):  # the new token behind the last private token
            segs = b["seg_len"][b["seg_start"][s]:b["seg_start"][s + 1]]
            entry = _pages(int(b["prefix"][s])) + sum(_pages(int(x)) for x in segs[:-1]) + int(segs[-1]) // PAGE
            page, tok = int(b["table"][s, entry]), int(segs[-1]) % PAGE
            kv[l][page, 0].view(hkv, d // 8, PAGE, 8)[:, :, tok] = new[l][0][s].view(hkv, d // 8, 8)
            kv[l][page, 1].view(hkv, PAGE // 4, d, 4)[:, tok // 4, :, tok % 4] = new[l][1][s]
        outs.append(_attention(case, b, q[l], kv[l])[0])
    return {"out": outs, "kv": kv}
