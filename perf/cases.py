"""The work that programs give this library, as timed cases.

Five kinds of call, each through the package's public entry points:

  attn        ``verify_attn``: ragged packed verify attention over the paged KV
              cache, one call (``graph`` false) or the attention of ``layers``
              layers captured once and replayed (``graph`` true)
  accept      ``accept``: greedy acceptance of a step's logits, replayed
  stochastic  ``accept_stochastic``: acceptance at temperature > 0, replayed
  decide      the decision step of one bucket, replayed: the predictor (when
              ``predictor`` is true) and DVL allocation and packing
  step        one whole engine step of a ``BucketSet`` bucket: the decision
              graph, then the verify graph (``layers`` layers and acceptance)

Inputs are drawn on the device from the seed.  Context lengths are evenly
spaced over [ctx_lo, ctx_hi] and verify lengths follow the quantiles of their
distribution, both dealt to the requests in an order of the seed's own, so a
case's work does not depend on the seed.
"""
import functools
import math
import random

import numpy as np
import torch

import paper_2609_37532_amd as dsv
from paper_2609_37532_amd import buckets as dsv_buckets

PAGE = 16   # tokens per KV page
WIDTH = 16  # block width: the anchor and 15 candidates
PRED_IN, PRED_HIDDEN = 1735, 64
LARGEST_BYTES = 1_260_000_000  # of one pass of the largest listed case


# ------------------------------------------------------------------- the cases
def _attn(name, reqs, hkv, group, dim, ctx_lo, ctx_hi, lens, layers, graph):
    return {"name": name, "kind": "attn", "reqs": reqs, "hkv": hkv, "group": group, "dim": dim,
            "ctx_lo": ctx_lo, "ctx_hi": ctx_hi, "lens": lens, "layers": layers, "graph": graph}


def listed():
    return [
        # one interactive request with a full block: latency and launches count
        _attn("attn_b1_ctx700", 1, 8, 4, 128, 700, 700, "full", 4, True),
        # a small server, full blocks, short contexts (B=8, contexts to 2K)
        _attn("attn_b8_ctx2k", 8, 8, 4, 128, 256, 2048, "full", 4, True),
        # the flagship verify step: B=32, 32 query and 8 KV heads, contexts to 8K
        _attn("attn_b32_ctx8k", 32, 8, 4, 128, 1024, 8192, "geom", 1, False),
        # long contexts under 64 query heads, lengths as DVL's budget fills them
        _attn("attn_b32_g8_ctx16k", 32, 8, 8, 128, 2000, 16300, "dvl", 1, False),
        # 16 query heads on each of two KV heads (a tensor-parallel share), full blocks
        _attn("attn_b24_g16_ctx6k", 24, 2, 16, 128, 500, 6007, "full", 2, True),
        # head_dim 64 at the flagship's batch
        _attn("attn_b32_d64_ctx8k", 32, 8, 4, 64, 1024, 8192, "geom", 1, False),
        # greedy acceptance of the flagship step: bf16 logits, 256 packed rows
        {"name": "accept_b32_v151936", "kind": "accept", "reqs": 32, "lens": "geom",
         "vocab": 151936, "dtype": "bf16"},
        # the same from fp32 logits of a vocabulary whose rows are not 16-byte aligned
        {"name": "accept_b32_v50257_f32", "kind": "accept", "reqs": 32, "lens": "dvl",
         "vocab": 50257, "dtype": "f32"},
        # sampling at temperature 0.8 over the flagship step's logits
        {"name": "stochastic_b32_v151936", "kind": "stochastic", "reqs": 32, "lens": "geom",
         "vocab": 151936, "dtype": "bf16", "temperature": 0.8},
        # the decision step of a 32-request bucket: predictor, then DVL
        {"name": "decide_b32", "kind": "decide", "reqs": 32, "live": 29, "predictor": True},
        # DVL for the largest bucket, its logits from elsewhere
        {"name": "decide_b1024_dvl", "kind": "decide", "reqs": 1024, "live": 1000,
         "predictor": False},
        # one engine step of a 16-request bucket with two sentinel slots
        {"name": "step_b16_ctx4k", "kind": "step", "reqs": 16, "live": 14, "hkv": 8, "group": 4,
         "dim": 128, "ctx_lo": 512, "ctx_hi": 4096, "layers": 4, "vocab": 151936},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["attn", "attn", "attn", "attn", "accept", "stochastic", "decide", "step"])
    if kind == "attn":
        hi = _log_int(rng, 200, 16384)
        c = {"kind": kind, "reqs": _log_int(rng, 1, 64), "hkv": rng.choice([1, 2, 4, 8]),
             "group": rng.choice([1, 2, 4, 8, 16]), "dim": rng.choice([64, 128, 128]),
             "ctx_lo": max(1, int(hi * rng.uniform(0.1, 0.9))), "ctx_hi": hi,
             "lens": rng.choice(["full", "geom", "dvl"])}
        c["layers"] = rng.choice([1, 2, 4])
        c["graph"] = c["layers"] > 1 or rng.random() < 0.5
    elif kind in ("accept", "stochastic"):
        c = {"kind": kind, "reqs": _log_int(rng, 1, 64), "lens": rng.choice(["full", "geom", "dvl"]),
             "vocab": rng.choice([32000, 50257, 65537, 151936, 262144, _log_int(rng, 1000, 262144)]),
             "dtype": rng.choice(["bf16", "bf16", "f32"])}
        if kind == "stochastic":
            c["temperature"] = round(rng.uniform(0.6, 1.3), 2)
    elif kind == "decide":
        n = _log_int(rng, 2, 1024)
        c = {"kind": kind, "reqs": n, "live": max(1, n - rng.randrange(1 + n // 4)),
             "predictor": rng.random() < 0.6}
    else:
        n = rng.choice([4, 8, 16, 32])
        hi = _log_int(rng, 512, 8192)
        c = {"kind": kind, "reqs": n, "live": n - rng.randrange(1 + n // 4), "hkv": 8, "group": 4,
             "dim": 128, "ctx_lo": max(1, int(hi * rng.uniform(0.1, 0.9))), "ctx_hi": hi,
             "layers": rng.choice([1, 2, 4]), "vocab": rng.choice([32000, 50257, 151936])}
    while work(c)["bytes"] > LARGEST_BYTES:
        if c.get("layers", 1) > 1:
            c["layers"] //= 2
        else:
            c["reqs"] = max(1, c["reqs"] * 3 // 4)
            c["live"] = min(c.get("live", c["reqs"]), c["reqs"])
    if kind not in ("decide", "step"):
        c.pop("live", None)
    return c


# --------------------------------------------------------------------- lengths
def _lengths(lens, n):
    """Verify lengths of n requests: full blocks, an anchor with a truncated
    geometric prefix (p = 0.25), or lengths that fill DVL's budget of 8 a request."""
    if lens == "full":
        return [WIDTH] * n
    at = [(i + 0.5) / n for i in range(n)]
    if lens == "geom":
        k = [min(WIDTH, 1 + int(math.log(1 - u) / math.log(0.75))) for u in at]
    else:
        k = [1 + int((WIDTH - 1) * u) for u in at]
    while sum(k) > 8 * n:
        k[max(range(n), key=lambda i: k[i])] -= 1
    return k


def _contexts(case, n):
    lo, hi = case["ctx_lo"], case["ctx_hi"]
    return [lo + int((hi - lo) * (i + 0.5) / n) for i in range(n)]


def _capacity(case):
    return (WIDTH if case.get("lens") == "full" else WIDTH // 2) * case["reqs"]


def _dealt(seed, values):
    values = list(values)
    random.Random(seed).shuffle(values)
    return values


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(1_000_003 * int(seed) + 17)
    return g


def _i32(values):
    return torch.tensor(values, dtype=torch.int32, device="cuda")


def _offsets(k):
    cu = [0]
    for x in k:
        cu.append(cu[-1] + x)
    return cu


# ---------------------------------------------------------------------- inputs
def _paged(case, seed, ctx, g):
    """Page table and per-layer KV pools: the requests' pages lie scattered over the pool."""
    n, dim, hkv = case["reqs"], case["dim"], case["hkv"]
    pages = [(c + WIDTH + PAGE - 1) // PAGE for c in ctx]
    pmax = (case["ctx_hi"] + WIDTH + PAGE - 1) // PAGE
    total = sum(pages) + 8
    ids = torch.randperm(total, generator=g, device="cuda", dtype=torch.int32)
    table = torch.zeros((n, pmax), dtype=torch.int32, device="cuda")
    at = 0
    for i, p in enumerate(pages):
        table[i, :p] = ids[at:at + p]
        at += p
    kv = [torch.randn((total, 2, hkv, PAGE * dim), generator=g, device="cuda",
                      dtype=torch.bfloat16) for _ in range(case["layers"])]
    return table, kv


def _attn_inputs(case, seed):
    g = _generator(seed)
    k = _dealt(2 * seed, _lengths(case["lens"], case["reqs"]))
    ctx = _dealt(2 * seed + 1, _contexts(case, case["reqs"]))
    table, kv = _paged(case, seed, ctx, g)
    hq = case["hkv"] * case["group"]
    q = [torch.randn((_capacity(case), hq, case["dim"]), generator=g, device="cuda",
                     dtype=torch.bfloat16) for _ in kv]
    return {"k": k, "ctx": ctx, "table": table, "kv": kv, "q": q}


def _logits_inputs(case, seed):
    """Logits, offsets and drafted ids of one step.  Greedy: the target repeats
    a geometric prefix of each draft.  Stochastic: logits as peaked as a
    language model's, the drafted ids with real probability."""
    g = _generator(seed)
    r = random.Random(seed)
    n, vocab, cap = case["reqs"], case["vocab"], _capacity(case)
    k = _dealt(2 * seed, _lengths(case["lens"], n))
    cu = _offsets(k)
    dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    draft = [r.randrange(vocab) for _ in range(cap)]
    logits = torch.randn((cap, vocab), generator=g, device="cuda", dtype=dtype)
    rows, ids, values = [], [], []
    if case["kind"] == "accept":
        for i in range(n):
            a = min(int(math.log(1 - r.random()) / math.log(0.75)), k[i] - 1)
            for j in range(min(a + 1, k[i])):
                hit = j < a
                rows.append(cu[i] + j)
                ids.append(draft[cu[i] + j + 1] if hit else r.randrange(vocab))
                values.append(14.0)
    else:
        logits *= 4.0
        lse = math.log(vocab) + 8.0  # log of the sum of exp(4 x), x ~ N(0, 1)
        for i in range(n):
            for j in range(k[i] - 1):
                rows.append(cu[i] + j)
                ids.append(draft[cu[i] + j + 1])
                values.append(lse + r.uniform(-2.0, 2.0))
    if rows:
        logits[torch.tensor(rows, device="cuda"), torch.tensor(ids, device="cuda")] = torch.tensor(
            values, device="cuda").to(dtype)
    uniforms = torch.rand((cap, 2), generator=g, device="cuda")
    return {"k": k, "cu": cu, "draft": draft, "logits": logits, "uniforms": uniforms}


def _decide_inputs(case, seed):
    n, g = case["reqs"], _generator(seed)
    rate = 0.85 + 0.145 * torch.rand((n, 1), generator=g, device="cuda", dtype=torch.float64)
    p = rate ** torch.arange(1, WIDTH, device="cuda")
    noise = torch.randn((n, WIDTH - 1), generator=g, device="cuda", dtype=torch.float64)
    s = {"live": case["live"], "pred_logits": (torch.log(p / (1 - p)) + 0.5 * noise).float()}
    for name, top in (("tokens", 151936), ("positions", 16384), ("kv_refs", 1 << 20)):
        s[name] = torch.randint(0, top, (n, WIDTH), generator=g, device="cuda", dtype=torch.int32)
    if case.get("predictor", True):
        rnd = lambda *shape: torch.randn(shape, generator=g, device="cuda")  # noqa: E731
        f = rnd(n, PRED_IN)
        f[:, :WIDTH - 1] = 14 + 3 * f[:, :WIDTH - 1]   # top logits of the 15 positions
        s["features"] = f
        s["w1"], s["b1"] = rnd(PRED_IN, PRED_HIDDEN) * math.sqrt(2 / PRED_IN), 0.3 * rnd(PRED_HIDDEN)
        s["w2"], s["b2"] = rnd(PRED_HIDDEN, WIDTH - 1) / 8, 1 + 0.7 * rnd(WIDTH - 1)
    return s


# --------------------------------------------------------------------- prepare
@functools.lru_cache(maxsize=None)
def _stream():
    """The program's own stream (graphs are captured on one, not on the null stream)."""
    return torch.cuda.Stream()


def _captured(state, call):
    torch.cuda.synchronize()  # the inputs are there
    state["graph"] = dsv.Graph().capture(call, _stream())
    return state


def _prepare_attn(case, seed):
    x = _attn_inputs(case, seed)
    s = {"kind": "attn", "q": x["q"], "kv": x["kv"], "table": x["table"],
         "cu": _i32(_offsets(x["k"])), "ctx": _i32(x["ctx"]),
         "out": [torch.empty_like(q) for q in x["q"]], "stream": _stream()}
    s["dims"] = dsv.attn_dims(s["q"][0], s["kv"][0], s["table"], max_kv_len=case["ctx_hi"] + WIDTH)
    s["ws"] = dsv.alloc_workspace(dsv.verify_attn_workspace_bytes(s["dims"]))
    if case["graph"]:
        return _captured(s, lambda: _attn_layers(s))
    torch.cuda.synchronize()
    return s


def _attn_layers(s):
    for q, kv, out in zip(s["q"], s["kv"], s["out"]):
        dsv.verify_attn(q, s["cu"], kv, s["table"], s["ctx"], out, dims=s["dims"],
                        workspace=s["ws"], stream=s["stream"])


def _prepare_logits(case, seed):
    x = _logits_inputs(case, seed)
    n, cap, vocab = case["reqs"], _capacity(case), case["vocab"]
    logits, cu, draft, uniforms = x["logits"], _i32(x["cu"]), _i32(x["draft"]), x["uniforms"]
    s = {"kind": case["kind"], "keep": (logits, cu, draft, uniforms), "stream": _stream(),
         "accept_len": _i32([0] * n), "next_token": _i32([0] * n)}
    a, t = s["accept_len"], s["next_token"]
    if case["kind"] == "accept":
        ws = s["ws"] = dsv.alloc_workspace(dsv.accept_workspace_bytes(cap, n, vocab))
        return _captured(s, lambda: dsv.accept(logits, cu, draft, a, t, workspace=ws,
                                               stream=s["stream"]))
    ws = s["ws"] = dsv.alloc_workspace(dsv.accept_stochastic_workspace_bytes(cap, n, vocab))
    return _captured(s, lambda: dsv.accept_stochastic(
        logits, cu, draft, uniforms, case["temperature"], a, t, workspace=ws, stream=s["stream"]))


def _prepare_decide(case, seed):
    x, n = _decide_inputs(case, seed), case["reqs"]
    s = {"kind": "decide", "x": x, "live": _i32([x["live"]]), "stream": _stream(),
         "pred_logits": x["pred_logits"], "k": _i32([0] * n), "cu": _i32([0] * (n + 1)),
         "packed": [_i32([0] * (WIDTH * n // 2)) for _ in range(3)]}
    if case["predictor"]:
        s["pred_logits"] = torch.zeros_like(x["pred_logits"])
        s["ws"] = dsv.alloc_workspace(dsv.predictor_workspace_bytes(n, PRED_IN))

    def call():
        if case["predictor"]:
            dsv.predictor_forward(x["features"], s["live"], x["w1"], x["b1"], x["w2"], x["b2"],
                                  s["pred_logits"], workspace=s["ws"], stream=s["stream"])
        dsv.dvl_allocate_pack(s["pred_logits"], s["live"], x["tokens"], x["positions"],
                              x["kv_refs"], s["k"], s["cu"], *s["packed"], stream=s["stream"])

    return _captured(s, call)


def _step_inputs(case, seed):
    x = _decide_inputs(case, seed)
    g = _generator(seed + 7919)
    ctx = _dealt(seed, _contexts(case, case["reqs"]))
    x["ctx"] = ctx
    x["table"], x["kv"] = _paged(case, seed, ctx, g)
    hq, cap = case["hkv"] * case["group"], WIDTH // 2 * case["reqs"]
    x["q"] = torch.randn((case["layers"], cap, hq, case["dim"]), generator=g, device="cuda",
                         dtype=torch.bfloat16)
    x["logits"] = torch.randn((cap, case["vocab"]), generator=g, device="cuda",
                              dtype=torch.bfloat16)
    return x


def _prepare_step(case, seed):
    x, n = _step_inputs(case, seed), case["reqs"]
    hq = case["hkv"] * case["group"]
    bs = dsv_buckets.BucketSet(
        [n], kv_pools=x["kv"], max_pages=x["table"].shape[1], max_kv_len=case["ctx_hi"] + WIDTH,
        num_q_heads=hq, head_dim=case["dim"], vocab=case["vocab"],
        predictor={w: x[w] for w in ("w1", "b1", "w2", "b2")})
    torch.cuda.synchronize()
    bs.capture(_stream())
    b = bs[bs.select(case["live"])]
    live = case["live"]
    b.stage_decision(live, x["features"], x["tokens"], x["positions"], x["kv_refs"])
    b.stage_verify(live, _i32(x["ctx"]), x["table"])
    b.q.copy_(x["q"])
    b.logits.copy_(x["logits"])
    torch.cuda.synchronize()
    return {"kind": "step", "set": bs, "bucket": b, "kv": x["kv"], "stream": _stream(),
            "weights": [x[w] for w in ("w1", "b1", "w2", "b2")]}


def prepare(case, seed):
    make = {"attn": _prepare_attn, "accept": _prepare_logits, "stochastic": _prepare_logits,
            "decide": _prepare_decide, "step": _prepare_step}[case["kind"]]
    return make(case, seed)


# ------------------------------------------------------------------------- run
def run(state):
    kind = state["kind"]
    if kind == "step":
        b = state["bucket"]
        b.replay_decision(state["stream"])
        b.replay_verify(state["stream"])
        return {"pred_logits": b.pred_logits, "k": b.k, "cu": b.cu, "tokens": b.packed_tokens,
                "positions": b.packed_positions, "kv_refs": b.packed_kv_refs, "out": b.out,
                "accept_len": b.accept_len, "next_token": b.next_token}
    if "graph" in state:
        state["graph"].replay(state["stream"])
    else:
        _attn_layers(state)
    if kind == "attn":
        return state["out"]
    if kind == "decide":
        return {"pred_logits": state["pred_logits"], "k": state["k"], "cu": state["cu"],
                "packed": state["packed"]}
    return {"accept_len": state["accept_len"], "next_token": state["next_token"]}


# ------------------------------------------------------------------------ work
def _attn_work(case, k, ctx):
    hq, dim, live = case["hkv"] * case["group"], case["dim"], sum(k)
    keys = sum(c + x for c, x in zip(ctx, k) if x)
    pages = sum((c + x + PAGE - 1) // PAGE for c, x in zip(ctx, k) if x)
    cap = _capacity(case)
    seen = sum(c * x + x * (x + 1) // 2 for c, x in zip(ctx, k))
    per_layer = keys * case["hkv"] * dim * 4 + (live + cap) * hq * dim * 2
    return {"bytes": case["layers"] * (per_layer + 4 * pages + 8 * len(k)),
            "flops": case["layers"] * 4 * dim * hq * seen}


def _decide_work(n, live, predictor):
    dvl = live * (WIDTH - 1) * 4 + 6 * 4 * (WIDTH // 2) * n
    if not predictor:
        return {"bytes": dvl, "flops": live * (WIDTH - 1) * 4}
    weights = PRED_IN * PRED_HIDDEN + PRED_HIDDEN * WIDTH
    return {"bytes": dvl + 4 * (weights + live * PRED_IN + n * (WIDTH - 1)),
            "flops": 2 * live * (PRED_IN * PRED_HIDDEN + PRED_HIDDEN * (WIDTH - 1))}


def work(case):
    n, kind = case["reqs"], case["kind"]
    if kind == "attn":
        return _attn_work(case, _lengths(case["lens"], n), _contexts(case, n))
    if kind == "decide":
        return _decide_work(n, case["live"], case["predictor"])
    if kind == "step":
        live = case["live"]
        d = _decide_work(n, live, True)
        a = _attn_work(case, [WIDTH // 2] * live, _contexts(case, n)[:live])
        rows = WIDTH // 2 * live
        return {"bytes": d["bytes"] + a["bytes"] + rows * case["vocab"] * 2,
                "flops": d["flops"] + a["flops"] + rows * case["vocab"]}
    rows = sum(_lengths(case["lens"], n))
    size = 2 if case["dtype"] == "bf16" else 4
    per = 1 if kind == "accept" else 4
    return {"bytes": rows * case["vocab"] * size + 8 * rows + 8 * n,
            "flops": rows * case["vocab"] * per}


def tolerance(case):
    kind = case["kind"]
    if kind == "accept" or (kind == "decide" and not case["predictor"]):
        return "exact"
    if kind == "stochastic":
        # whole numbers; a draw may move to the next token where its uniform
        # lies within fp32 rounding of the boundary between the two
        return {"rel": 0.0, "differ": 0.01}
    if kind == "decide":
        # fp32 sums of 1,735 products; a length may flip between equal scores
        return {"rel": 5e-6, "max": 5e-5, "differ": 0.01}
    # outputs rounded once to bf16
    return {"rel": 6e-3, "max": 2e-2, "differ": 0.01}


# ----------------------------------------------------------------------- exact
def _exact_attn(case, k, ctx, table, kv, q):
    """Masked softmax attention in 64 bits; rows past the live ones are zero."""
    dim, hkv, grp = case["dim"], case["hkv"], case["group"]
    out = torch.zeros(q.shape, dtype=torch.float64, device="cuda")
    at = 0
    for i, (x, c) in enumerate(zip(k, ctx)):
        if not x:
            continue
        t = c + x
        pages = kv[table[i, :(t + PAGE - 1) // PAGE].long()].double()
        # K tile: element (slot, d) at ((d / 8) * 16 + slot) * 8 + d % 8; V tile: d * 16 + slot
        kk = pages[:, 0].reshape(-1, hkv, dim // 8, PAGE, 8).permute(1, 2, 4, 0, 3)
        kk = kk.reshape(hkv, dim, -1)[:, :, :t].contiguous()
        vv = pages[:, 1].reshape(-1, hkv, dim, PAGE).permute(1, 0, 3, 2)
        vv = vv.reshape(hkv, -1, dim)[:, :t].contiguous()
        rows = q[at:at + x].double().reshape(x, hkv, grp, dim).permute(1, 0, 2, 3)
        s = torch.bmm(rows.reshape(hkv, x * grp, dim).contiguous(), kk) / math.sqrt(dim)
        limit = c + torch.arange(x, device="cuda").repeat_interleave(grp)
        s.masked_fill_(torch.arange(t, device="cuda")[None, None] > limit[None, :, None], -math.inf)
        o = torch.bmm(torch.softmax(s, dim=-1), vv).reshape(hkv, x, grp, dim)
        out[at:at + x] = o.permute(1, 0, 2, 3).reshape(x, hkv * grp, dim)
        at += x
    return out


def _prefix(best, cu, draft):
    accepted, token = [], []
    for o, e in zip(cu[:-1], cu[1:]):
        a = 0
        while o + a + 1 < e and best[o + a] == draft[o + a + 1]:
            a += 1
        accepted.append(a if e > o else 0)
        token.append(best[o + a] if e > o else -1)
    return {"accept_len": _i32(accepted), "next_token": _i32(token)}


def _first_best(logits):
    """Lowest index of each row's largest value."""
    top = logits.max(dim=1, keepdim=True).values
    return (logits == top).int().argmax(dim=1).tolist()


def _exact_stochastic(case, x):
    cu, draft, u = x["cu"], x["draft"], x["uniforms"].double().cpu().numpy()
    accepted, token = [], []
    for o, e in zip(cu[:-1], cu[1:]):
        p = torch.softmax(x["logits"][o:e].double() / case["temperature"], dim=1)
        a = 0
        while o + a + 1 < e and u[o + a, 0] < float(p[a, draft[o + a + 1]]):
            a += 1
        row = p[a].clone()
        if o + a + 1 < e:
            row[draft[o + a + 1]] = 0.0
        cum = torch.cumsum(row, 0)
        accepted.append(a)
        token.append(int(torch.searchsorted(cum, u[o + a, 1] * float(cum[-1]), right=True)))
    return {"accept_len": _i32(accepted), "next_token": _i32(token)}


def _exact_logits(x):
    h = torch.relu(x["features"].double() @ x["w1"].double() + x["b1"].double())
    y = h @ x["w2"].double() + x["b2"].double()
    y[x["live"]:] = 0
    return y


def _allocate(pred_logits, live):
    """DVL's lengths: scores, seeds, then one slot at a time until the budget is met."""
    x = pred_logits[:live].float().double().cpu().numpy()
    with np.errstate(over="ignore"):
        score = np.minimum.accumulate((1 / (1 + np.exp(-x))).astype(np.float32), axis=1)
    k = []
    for row in score:
        s = np.float32(0)
        for v in row:
            s = np.float32(s + v)
        k.append(min(WIDTH, max(1, int(math.floor(np.float32(s + np.float32(0.5)))))))
    q = [[1.0] + [float(v) for v in row] for row in score]
    gap = WIDTH * live // 2 - sum(k)
    while gap:
        if gap > 0:
            i = max((i for i in range(live) if k[i] < WIDTH), key=lambda i: (q[i][k[i]], -i))
        else:
            i = min((i for i in range(live) if k[i] > 1), key=lambda i: (q[i][k[i] - 1], i))
        k[i] += 1 if gap > 0 else -1
        gap += -1 if gap > 0 else 1
    return k


def exact(case, seed):
    kind = case["kind"]
    if kind == "attn":
        x = _attn_inputs(case, seed)
        return [_exact_attn(case, x["k"], x["ctx"], x["table"], kv, q)
                for kv, q in zip(x["kv"], x["q"])]
    if kind == "accept":
        x = _logits_inputs(case, seed)
        return _prefix(_first_best(x["logits"][:x["cu"][-1]]), x["cu"], x["draft"])
    if kind == "stochastic":
        return _exact_stochastic(case, _logits_inputs(case, seed))
    if kind == "decide":
        if not case["predictor"]:
            return None  # whole numbers only
        return {"pred_logits": _exact_logits(_decide_inputs(case, seed)), "k": None, "cu": None,
                "packed": [None, None, None]}
    x = _step_inputs(case, seed)
    y = _exact_logits(x)
    k = _allocate(y, case["live"]) + [0] * (case["reqs"] - case["live"])
    out = torch.stack([_exact_attn(case, k, x["ctx"], x["table"], kv, q)
                       for kv, q in zip(x["kv"], x["q"])])
    return {"pred_logits": y, "k": _i32(k), "cu": None, "tokens": None, "positions": None,
            "kv_refs": None, "out": out, "accept_len": None, "next_token": None}
