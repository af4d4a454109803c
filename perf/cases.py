"""The calls by which this library's speed is judged: decode steps and cache
constructions through the Python binding, over the sizes they are used at.

A case names one entry point and the sizes of its call. Contexts, budgets and
residual counts per (sequence, KV head) follow from the case alone, tensor
values from the seed alone: keys N(0, 1) plus a per-channel bias on four
channels of each KV head, some "heavy" keys three times as large, queries
that mix four heavy keys with noise (the statistics of the workloads in
paper_2607_29591_amd/synth.py).
"""

import math
import random

import torch

from paper_2607_29591_amd import reskv as rk

TAU, ALPHA, G_MIN, BETA = 0.25, 12.0, 0.0, 1.0
DECODE = ("decode", "ragged", "branches")


# ------------------------------------------------------------------- cases

def _decode(name, kind, dtype, B, Hq, Hkv, d, layers, budget, budget_min, res_max, room, tau, mix):
    c = dict(kind=kind, dtype=dtype, B=B, Hq=Hq, Hkv=Hkv, d=d, layers=layers, budget=budget,
             budget_min=budget_min, res_max=res_max, room=room, tau=tau, mix=mix)
    return dict(c, name=name) if name else c


def _build(name, kind, dtype, B, Hq, Hkv, d, ctx, ctx_min, budget, budget_min, res_max, window, mix):
    c = dict(kind=kind, dtype=dtype, B=B, Hq=Hq, Hkv=Hkv, d=d, ctx=ctx, ctx_min=ctx_min, budget=budget,
             budget_min=budget_min, res_max=res_max, window=window, mix=mix)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: one layer of a toy model in fp32, no append
        _decode("decode_toy_f32", "decode", "f32", 1, 8, 2, 64, 1, 128, 128, 32, 0, False, 1),
        # one user's chat: a step of a 32-layer Llama-3.1-8B-shaped model on 512-slot caches
        _decode("decode_llama_b1", "decode", "bf16", 1, 32, 8, 128, 32, 512, 512, 128, 128, False, 2),
        # four long documents: eight layers of 1024-slot caches, still fewer heads than CUs
        _decode("decode_long_b4", "decode", "bf16", 4, 32, 8, 128, 8, 1024, 1024, 256, 64, False, 3),
        # a full serving batch: four layers, per-query thresholds, one block per head
        _decode("decode_batch_b32", "decode", "bf16", 32, 32, 8, 128, 4, 2048, 2048, 512, 256, True, 4),
        # a batch of uneven budgets (28 query heads over 4 KV heads) through the ragged schedule
        _decode("decode_ragged_gqa7", "ragged", "bf16", 64, 28, 4, 128, 4, 1024, 256, 512, 128, False, 5),
        # the two-branch form and its log-sum-exp merge
        _decode("branches_b8", "branches", "bf16", 8, 32, 8, 128, 4, 1024, 1024, 256, 0, False, 6),
        # the smallest construction: a toy layer in fp32
        _build("build_toy_f32", "build", "f32", 1, 8, 2, 64, 1024, 1024, 128, 128, 32, 16, 7),
        # one user's prompt: a 32K-token Llama-3.1-8B-shaped layer
        _build("build_llama_b1", "build", "bf16", 1, 32, 8, 128, 32768, 32768, 512, 512, 128, 32, 8),
        # a serving batch's prompts, the largest call
        _build("build_batch_b32", "build", "bf16", 32, 32, 8, 128, 32768, 32768, 2048, 2048, 512, 32, 9),
        # long documents: 128K tokens, 64-row window
        _build("build_long_b4", "build", "bf16", 4, 32, 8, 128, 131072, 131072, 1024, 1024, 256, 64, 10),
        # uneven prompts with the budget shared across KV heads
        _build("adakv_ragged_gqa7", "adakv", "bf16", 16, 28, 4, 128, 65536, 4096, 1024, 256, 256, 32, 11),
        # residual counts chosen by the validation proxy (five candidates)
        _build("proxy_b2", "proxy", "bf16", 2, 32, 8, 128, 32768, 32768, 2048, 2048, 0, 32, 12),
    ]


def draw(rng):
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["decode", "decode", "ragged", "branches", "build", "build", "adakv", "proxy"])
    dtype, d = rng.choice([("bf16", 128), ("bf16", 128), ("bf16", 128), ("bf16", 64), ("f32", 64), ("f32", 128)])
    if kind == "ragged" and dtype == "f32":
        d = 64  # the widest fp32 rows that schedule takes
    G, Hkv = rng.choice([1, 2, 4, 4, 7, 8]), rng.choice([1, 2, 4, 8])
    mix = rng.randrange(1 << 20)
    if kind in DECODE:
        layers = rng.choice([1, 2, 4, 8])
        B = logint(8 if kind == "ragged" else 1, 64)
        budget = logint(100, 2100)
        while B * Hkv * budget * d * layers > 32 * 8 * 2048 * 128 * 4:
            budget = max(64, budget // 2)
            B = max(1, B // 2)
        lo = rng.randint(max(2, budget // 4), budget) if kind == "ragged" else budget
        return _decode("", kind, dtype, B, G * Hkv, Hkv, d, layers, budget, lo, int(lo * rng.uniform(0, 0.5)),
                       0 if kind == "branches" else rng.choice([16, 64, 100]), rng.random() < 0.5, mix)
    ctx = logint(1000, 131072)
    B = logint(1, 32)
    window = rng.choice([8, 16, 32, 32, 64])
    most = {"build": 1 << 22, "adakv": 1 << 21, "proxy": 1 << 19}[kind] // (4 if dtype == "f32" else 1)
    while B * Hkv * ctx > most:
        if B > 1:
            B //= 2
        else:
            ctx //= 2
    budget = min(logint(100, 2048), max(64, ctx // 2))
    ragged = kind == "adakv" or rng.random() < 0.3
    ctx_min = max(window, ctx // 3) if ragged else ctx
    budget_min = max(2, budget // 2) if ragged else budget
    res_max = 0 if kind == "proxy" else int(budget_min * rng.uniform(0, 0.4))
    return _build("", kind, dtype, B, G * Hkv, Hkv, d, ctx, ctx_min, budget, budget_min, res_max, window, mix)


def _sizes(case):
    """Per-sequence contexts and budgets, per-head residual counts and, for decode, main lengths."""
    r = random.Random(case["mix"])
    B, H = case["B"], case["Hkv"]
    budget = [r.randint(case["budget_min"], case["budget"]) for _ in range(B)]
    res = [[0 if case["res_max"] == 0 else r.choice([0, case["res_max"] // 4, case["res_max"] // 2, case["res_max"]])
            for _ in range(H)] for _ in range(B)]
    ctx = [r.randint(case["ctx_min"], case["ctx"]) for _ in range(B)] if "ctx" in case else None
    res = [[min(x, b - 1) for x in row] for row, b in zip(res, budget)]
    return ctx, budget, res


def _dt(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _capacity(case):
    if case["kind"] in DECODE:
        return case["budget"] + case["room"]
    return case["budget"] + (64 if case["kind"] == "adakv" else 0)


GRID = (0.0, 0.05, 0.10, 0.15, 0.20)   # candidate fractions of the validation proxy


def _proxy_rows(case):
    return max(1, case["window"] // 4)   # a quarter of the window validates


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)


def _bias(g, H, d):
    """Key bias on four channels of each head."""
    ch = torch.rand((H, d), generator=g, device="cuda").argsort(dim=-1)[:, :4]
    return torch.zeros((H, d), device="cuda").scatter_(1, ch, 3.0 * _randn(g, H, 4))


def _queries(g, heavy, n):
    """[.., n, d] queries from heavy keys [.., nh, d]: 0.7 * mean of four + 0.3 * N(0, 1)."""
    lead, (nh, d) = heavy.shape[:-2], heavy.shape[-2:]
    pick = torch.randint(nh, (*lead, n * 4), generator=g, device="cuda")
    k = torch.gather(heavy, -2, pick[..., None].expand(*pick.shape, d)).reshape(*lead, n, 4, d)
    return 0.7 * k.mean(dim=-2) + 0.3 * _randn(g, *lead, n, d)


def _inputs_decode(case, seed):
    g, dt = _gen(seed), _dt(case)
    L, B, Hq, H, d = (case[x] for x in ("layers", "B", "Hq", "Hkv", "d"))
    G, C = Hq // H, _capacity(case)
    _, budget, res = _sizes(case)
    Rcap = max(1, max(max(row) for row in res))
    r = torch.tensor(res, device="cuda")                                   # [B, H]
    n = torch.tensor(budget, device="cuda")[:, None] - r
    kc = torch.empty((L, B, H, C, d), dtype=dt, device="cuda")
    vc = torch.empty_like(kc)
    logc = torch.full((L, B, H, Rcap), -math.inf, device="cuda")
    q = torch.empty((L, B, Hq, d), dtype=dt, device="cuda")
    k_new = torch.empty((L, B, H, d), dtype=dt, device="cuda")
    v_new = torch.empty_like(k_new)
    slot = torch.arange(C, device="cuda")
    for l in range(L):
        bias = _bias(g, B * H, d).reshape(B, H, 1, d)
        # residual slots are means of `count` tokens: noise shrinks with the count, a few are empty
        count = torch.exp(4.0 + _randn(g, B, H, Rcap)).floor() + 1.0
        empty = torch.rand((B, H, Rcap), generator=g, device="cuda") < 0.02
        live = (slot[:Rcap] < r[..., None]) & ~empty
        logc[l] = torch.where(live, torch.log(count), logc[l])
        shrink = torch.ones((B, H, C), device="cuda")
        is_res = slot < r[..., None]
        shrink[..., :Rcap] = torch.where(is_res[..., :Rcap], count.rsqrt(), shrink[..., :Rcap])
        K = _randn(g, B, H, C, d) * shrink[..., None] + bias
        nh = max(4, case["budget"] // 32)
        at = r[..., None] + (torch.rand((B, H, nh), generator=g, device="cuda") * n[..., None]).long()
        at = at[..., None].expand(B, H, nh, d)
        heavy = 3.0 * K.gather(2, at)
        kc[l] = K.scatter_(2, at, heavy).to(dt)
        vc[l] = (_randn(g, B, H, C, d) * shrink[..., None]).to(dt)
        q[l] = _queries(g, heavy, G).reshape(B, Hq, d).to(dt)
        k_new[l] = (_randn(g, B, H, d) + bias[:, :, 0]).to(dt)
        v_new[l] = _randn(g, B, H, d).to(dt)
    tau = 0.5 * _randn(g, L, B, Hq) if case["tau"] else None
    return dict(q=q, kc=kc, vc=vc, logc=logc, k_new=k_new, v_new=v_new, tau=tau, r=r, n=n, Rcap=Rcap, C=C)


def _inputs_build(case, seed):
    g, dt = _gen(seed), _dt(case)
    B, Hq, H, d, w, S = (case[x] for x in ("B", "Hq", "Hkv", "d", "window", "ctx"))
    ctx, _, _ = _sizes(case)
    # with sharp queries the heavy keys hold all attention and every candidate of the proxy loses nothing: its heads
    # are diffuse ones, where residual entries matter
    scale = 0.15 if case["kind"] == "proxy" else 1.0
    k = torch.zeros((B, H, S, d), dtype=dt, device="cuda")
    v = torch.zeros_like(k)
    q = torch.empty((B, Hq, w, d), dtype=dt, device="cuda")
    for b, s in enumerate(ctx):
        K = _randn(g, H, s, d) + _bias(g, H, d)[:, None]
        nh = max(4, s // 100 if s > 65536 else s // 512)
        at = torch.randint(s, (H, nh), generator=g, device="cuda")[..., None].expand(H, nh, d)
        heavy = 3.0 * K.gather(1, at)
        k[b, :, :s] = K.scatter_(1, at, heavy).to(dt)
        v[b, :, :s] = _randn(g, H, s, d).to(dt)
        q[b] = _queries(g, heavy, Hq // H * w).reshape(Hq, w, d).mul(scale).to(dt)
    return dict(k=k, v=v, q=q)


def prepare(case, seed):
    L, B, Hq, H, d = (case.get(x, 1) for x in ("layers", "B", "Hq", "Hkv", "d"))
    dev = "cuda"
    if case["kind"] in DECODE:
        x = _inputs_decode(case, seed)
        shape = rk.make_shape(B, Hq, H, d, case["dtype"], x["C"], x["Rcap"])
        res_len = x["r"].to(torch.int32).reshape(-1).contiguous()
        main_len0 = x["n"].to(torch.int32).reshape(1, -1).repeat(L, 1).contiguous()
        size = rk.reskv_decode_ragged_workspace_size if case["kind"] == "ragged" else rk.reskv_decode_workspace_size
        st = dict(x, case=case, shape=shape, res_len=res_len, main_len0=main_len0, main_len=main_len0.clone(),
                  ws=torch.empty(size(shape), dtype=torch.uint8, device=dev),
                  out=torch.empty((L, B, Hq, d), dtype=torch.float32, device=dev))
        tau = x["tau"]
        st["gates"] = [rk.make_gate(tau=None if tau is None else tau[l], tau_scalar=TAU, alpha=ALPHA, g_min=G_MIN,
                                    beta=BETA) for l in range(L)]
        if case["kind"] == "branches":
            def rows():
                return torch.empty((L, B, Hq), dtype=torch.float32, device=dev)
            st.update(o_main=torch.empty_like(st["out"]), o_res=torch.empty_like(st["out"]), lse_main=rows(),
                      lse_res=rows(), gate=rows())
            return st
        # the step's calls, marshalled once as a serving loop keeps them
        prep = rk.prepare_decode_attn_ragged if case["kind"] == "ragged" else rk.prepare_decode_attn
        new = [(x["k_new"][l], x["v_new"][l]) if case["room"] else (None, None) for l in range(L)]
        st["calls"] = [prep(shape, st["gates"][l], x["q"][l], x["kc"][l], x["vc"][l], x["logc"][l], res_len,
                            st["main_len"][l], st["out"][l], st["ws"], k_new=new[l][0], v_new=new[l][1])
                       for l in range(L)]
        return st
    x = _inputs_build(case, seed)
    ctx, budget, res = _sizes(case)
    if case["kind"] == "proxy":
        Rcap = max(1, max(int(math.floor(max(GRID) * b + 0.5)) for b in budget))
    else:
        Rcap = max(1, max(max(row) for row in res))
    C = _capacity(case)
    shape = rk.make_shape(B, Hq, H, d, case["dtype"], C, Rcap)
    params = rk.BuildParams(case["ctx"], case["window"], case["window"], 4, 0, 0)
    flat = [r for row in res for r in row]
    st = dict(x, case=case, shape=shape, params=params, ctx=ctx, budget=budget, res=flat,
              kc=torch.zeros((B, H, C, d), dtype=_dt(case), device=dev),
              vc=torch.zeros((B, H, C, d), dtype=_dt(case), device=dev),
              logc=torch.zeros((B, H, Rcap), dtype=torch.float32, device=dev),
              main_idx=torch.zeros((B, H, C), dtype=torch.int32, device=dev),
              res_len=torch.zeros(B * H, dtype=torch.int32, device=dev),
              main_len=torch.zeros(B * H, dtype=torch.int32, device=dev))
    if case["kind"] == "proxy":
        st["proxy"] = rk.make_proxy(GRID, val_rows=_proxy_rows(case), delta=0.01)
        st["gate"] = rk.make_gate(tau_scalar=TAU, alpha=ALPHA, g_min=G_MIN, beta=BETA)
        st["loss"] = torch.zeros((B * H, len(GRID)), dtype=torch.float32, device=dev)
        size = rk.reskv_build_proxy_workspace_size(shape, params, st["proxy"], ctx, budget)
    elif case["kind"] == "adakv":
        size = rk.reskv_build_adakv_workspace_size(shape, params, 0.2, 64, ctx, budget, flat)
    else:
        size = rk.reskv_build_workspace_size(shape, params, ctx, budget, flat)
    st["ws"] = torch.empty(size, dtype=torch.uint8, device=dev)
    return st


# --------------------------------------------------------------------- run

def run(st):
    kind = st["case"]["kind"]
    if kind == "branches":
        for l in range(st["case"]["layers"]):
            rk.reskv_decode_branches(st["shape"], st["gates"][l], st["q"][l], st["kc"][l], st["vc"][l], st["logc"][l],
                                     st["res_len"], st["main_len"][l], st["o_main"][l], st["lse_main"][l],
                                     st["o_res"][l], st["lse_res"][l], st["gate"][l], st["ws"])
            rk.reskv_merge_branches(st["shape"], rk.RESKV_MERGE_SHARED, st["o_main"][l], st["lse_main"][l],
                                    st["o_res"][l], st["lse_res"][l], st["gate"][l], st["out"][l])
        return {k: st[k] for k in ("out", "o_main", "o_res", "lse_main", "lse_res", "gate")}
    if kind in DECODE:
        if not st["case"]["room"]:
            for call in st["calls"]:
                call()
            return {"out": st["out"]}
        st["main_len"].copy_(st["main_len0"])   # the step appends the same token again
        for call in st["calls"]:
            call()
        return {k: st[k] for k in ("out", "main_len", "kc", "vc")}
    outs = (st["kc"], st["vc"], st["logc"], st["main_idx"], st["res_len"], st["main_len"], st["ws"])
    got = {k: st[k] for k in ("kc", "vc", "logc", "main_idx", "res_len", "main_len")}
    if kind == "proxy":
        rk.reskv_build_cache_proxy(st["shape"], st["params"], st["proxy"], st["gate"], st["k"], st["v"], st["ctx"],
                                   st["q"], st["budget"], *outs, val_loss=st["loss"])
        got["loss"] = st["loss"]
    elif kind == "adakv":
        rk.reskv_build_cache_adakv(st["shape"], st["params"], 0.2, 64, st["k"], st["v"], st["ctx"], st["q"],
                                   st["budget"], st["res"], *outs)
    else:
        rk.reskv_build_cache(st["shape"], st["params"], st["k"], st["v"], st["ctx"], st["q"], st["budget"], st["res"],
                             *outs)
    return got


# -------------------------------------------------------- work, tolerances

def _build_sizes(case):
    """(s, budget, [candidate counts]) of every (sequence, KV head)."""
    ctx, budget, res = _sizes(case)
    for b in range(case["B"]):
        for h in range(case["Hkv"]):
            if case["kind"] == "proxy":
                yield ctx[b], budget[b], [int(math.floor(f * budget[b] + 0.5)) for f in GRID]
            else:
                yield ctx[b], budget[b], [res[b][h]]


def work(case):
    e = 2 if case["dtype"] == "bf16" else 4
    B, Hq, H, d = (case[x] for x in ("B", "Hq", "Hkv", "d"))
    G = Hq // H
    _, budget, res = _sizes(case)
    if case["kind"] in DECODE:
        new = 1 if case["room"] else 0
        slots = sum(b + new for b in budget) * H
        nbytes = slots * 2 * d * e + 4 * sum(map(sum, res)) + B * Hq * d * (e + 4) + 2 * new * B * H * d * e
        if case["kind"] == "branches":
            nbytes += 2 * B * Hq * d * 4
        return {"bytes": case["layers"] * nbytes, "flops": case["layers"] * 4 * G * d * slots}
    w, nbytes, flops = case["window"], B * Hq * case["window"] * d * e, 0
    rows = w - _proxy_rows(case) if case["kind"] == "proxy" else w
    for s, b, counts in _build_sizes(case):
        nbytes += 2 * s * d * e + 2 * min(b, s) * d * e + 4 * b
        flops += 2 * G * rows * s * d
        for r in counts:
            m = b - r
            if s > m:
                flops += 4 * 2 * (s - m) * r * d
        if case["kind"] == "proxy":
            flops += 4 * G * _proxy_rows(case) * d * (s + len(counts) * b)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # decode: fp32 sums in another order (1e-6 off 64 bits; the gate and the residual branch, whose bf16 entries are
    # few, 9e-6). Constructions: a token at a near-tie of two centres joins another group and moves two means
    # (0.001 - 0.005 off 64 bits in 2-norm where no kept token changes)
    if case["kind"] == "branches":
        return {"rel": 4e-5}
    if case["kind"] in DECODE:
        return {"rel": 1e-5}
    return {"rel": 0.02, "max": 0.9, "differ": 0.005}


# ------------------------------------------------------- 64-bit references

def _decode64(q, kc, vc, logc, r, n, tau):
    """Shared-softmax decode of q [B, H, G, d] over caches [B, H, C, d]; tau [B, H, G]. Returns the output, the two
    branches' outputs and log-sum-exps, and the gate."""
    C, d = kc.shape[-2:]
    slot = torch.arange(C, device=q.device)
    a = torch.matmul(q, kc.transpose(-1, -2).contiguous()) / math.sqrt(d)             # [B, H, G, C]
    is_res = (slot < r[..., None])[..., None, :]
    is_main = ((slot >= r[..., None]) & (slot < (r + n)[..., None]))[..., None, :]
    bias = torch.full_like(kc[..., 0], -math.inf)
    R = min(C, logc.shape[-1])
    bias[..., :R] = BETA * logc[..., :R]
    am = a.masked_fill(~is_main, -math.inf)
    ar = (a + bias[..., None, :]).masked_fill(~is_res, -math.inf)
    lm, lr = torch.logsumexp(am, -1), torch.logsumexp(ar, -1)
    g = torch.clamp(torch.sigmoid((tau - torch.exp(am.max(-1).values - lm)) * ALPHA), min=G_MIN)
    has = torch.isfinite(lr)
    pm = torch.exp(am - lm[..., None])
    pr = torch.where(has[..., None], torch.exp(ar - torch.where(has, lr, 0.0)[..., None]), 0.0)
    om, orr = torch.matmul(pm, vc), torch.matmul(pr, vc)
    share = torch.where(has, torch.sigmoid(torch.where(has, lr, 0.0) + torch.log(g) - lm), 0.0)[..., None]
    return om * (1 - share) + orr * share, om, orr, lm, lr, g


def _exact_decode(case, seed):
    x = _inputs_decode(case, seed)
    L, B, Hq, H, d = (case[k] for k in ("layers", "B", "Hq", "Hkv", "d"))
    r, n, kc, vc = x["r"], x["n"].clone(), x["kc"], x["vc"]
    if case["room"]:
        at = (r + n)[None, ..., None, None].expand(L, B, H, 1, d)
        kc.scatter_(3, at, x["k_new"][..., None, :])
        vc.scatter_(3, at, x["v_new"][..., None, :])
        n += 1
    got = []
    for l in range(L):
        tau = torch.full((B, Hq), TAU, device="cuda") if x["tau"] is None else x["tau"][l]
        o, om, orr, lm, lr, g = _decode64(x["q"][l].double().reshape(B, H, -1, d), kc[l].double(), vc[l].double(),
                                          x["logc"][l].double(), r, n, tau.double().reshape(B, H, -1))
        got.append([y.reshape(B, Hq, d) for y in (o, om, orr)] + [y.reshape(B, Hq) for y in (lm, lr, g)])
    got = dict(zip(("out", "o_main", "o_res", "lse_main", "lse_res", "gate"), map(torch.stack, zip(*got))))
    if case["kind"] == "branches":
        return got
    if not case["room"]:
        return {"out": got["out"]}
    return {"out": got["out"], "main_len": n.to(torch.int32).reshape(1, -1).repeat(L, 1), "kc": kc, "vc": vc}


def _scores64(q, K, rows):
    """Pooled window scores of one head: q [G, w, d] at positions s-w.., K [s, d]; the leading `rows` rows score."""
    G, w, d = q.shape
    s = K.shape[0]
    pos = torch.arange(s - w, s - w + rows, device=K.device)
    raw = torch.zeros(s, dtype=torch.float64, device=K.device)
    for h in range(G):
        a = q[h, :rows] @ K.t().contiguous() / math.sqrt(d)
        a.masked_fill_(torch.arange(s, device=K.device)[None] > pos[:, None], -math.inf)
        raw += torch.softmax(a, -1).sum(0)
    return raw


def _pool64(raw, n):
    x = torch.nn.functional.pad(raw[:n], (2, 2))
    return sum(x[i:i + n] for i in range(5))


def _construct64(K, V, score, k_top, r, C, Rcap):
    """Cache of one head: its k_top best-scored tokens, the unscored last ones and r groups of the rest."""
    s, d = K.shape
    n = score.numel()
    kc = torch.zeros((C, d), dtype=torch.float64, device=K.device)
    vc, idx = torch.zeros_like(kc), torch.zeros(C, dtype=torch.int32, device=K.device)
    logc = torch.full((Rcap,), -math.inf, dtype=torch.float64, device=K.device)
    order = torch.sort(score, descending=True, stable=True).indices
    top = torch.sort(order[:k_top]).values
    main = torch.cat([top, torch.arange(n, s, device=K.device)])
    keep = torch.ones(n, dtype=torch.bool, device=K.device)
    keep[top] = False
    E = torch.nonzero(keep).flatten()
    r_eff = min(r, E.numel())
    kc[r:r + main.numel()], vc[r:r + main.numel()], idx[:main.numel()] = K[main], V[main], main.to(torch.int32)
    if r_eff:
        KE, mu = K[E], K[torch.sort(order[k_top:k_top + r_eff]).values]
        for _ in range(4):
            a = torch.argmin((mu * mu).sum(-1)[None] - 2.0 * (KE @ mu.t().contiguous()), dim=1)
            cnt = torch.bincount(a, minlength=r_eff).double()
            full = cnt[:, None] > 0
            mean = torch.zeros_like(mu).index_add_(0, a, KE) / cnt.clamp(min=1)[:, None]
            mu = torch.where(full, mean, mu)
        kc[:r_eff] = mu
        vc[:r_eff] = torch.zeros_like(mu).index_add_(0, a, V[E]) / cnt.clamp(min=1)[:, None]
        logc[:r_eff] = torch.log(cnt)
    return kc, vc, logc, idx, main.numel()


def _adakv64(scores, k_tops, caps, safeguard):
    """Top-k counts of one sequence's heads: a floor each, the rest down one ranking of all heads."""
    take = [int(math.floor(safeguard * k)) for k in k_tops]
    left = sum(k_tops) - sum(take)
    sc, hd = [], []
    for h, x in enumerate(scores):
        rest = torch.sort(x, descending=True, stable=True).values[take[h]:]
        sc.append(rest[:caps[h] - take[h]])   # a head's tokens past its cap are passed over
        hd.append(torch.full((sc[-1].numel(),), h, device=x.device))
    order = torch.sort(torch.cat(sc), descending=True, stable=True).indices[:left]
    more = torch.bincount(torch.cat(hd)[order], minlength=len(take)).tolist()
    return [t + m for t, m in zip(take, more)]


def _exact_build(case, seed):
    x = _inputs_build(case, seed)
    B, Hq, H, d, w = (case[k] for k in ("B", "Hq", "Hkv", "d", "window"))
    G, C, kind = Hq // H, _capacity(case), case["kind"]
    ctx, budget, res = _sizes(case)
    val = _proxy_rows(case)
    if kind == "proxy":
        Rcap = max(1, max(int(math.floor(max(GRID) * b + 0.5)) for b in budget))
    else:
        Rcap = max(1, max(max(row) for row in res))
    got = dict(kc=[], vc=[], logc=[], main_idx=[], res_len=[], main_len=[], loss=[])

    def put(r, built):
        for k, y in zip(("kc", "vc", "logc", "main_idx", "main_len"), built):
            got[k].append(y)
        got["res_len"].append(r)

    for b in range(B):
        s, bud = ctx[b], budget[b]
        K = [x["k"][b, h, :s].double() for h in range(H)]
        V = [x["v"][b, h, :s].double() for h in range(H)]
        q = [x["q"][b, h * G:(h + 1) * G].double() for h in range(H)]
        raw = [_scores64(q[h], K[h], w - val if kind == "proxy" else w) for h in range(H)]

        def head(h, r, k_top=None):
            m = bud - r
            if s <= m:
                return _construct64(K[h], V[h], raw[h][:0], 0, 0, C, Rcap)
            P = min(w, m)
            return _construct64(K[h], V[h], _pool64(raw[h], s - P), m - P if k_top is None else k_top, r, C, Rcap)

        if kind == "adakv":
            part = [h for h in range(H) if s > bud - res[b][h]]
            P = {h: min(w, bud - res[b][h]) for h in part}
            k = dict(zip(part, _adakv64([_pool64(raw[h], s - P[h]) for h in part],
                                        [bud - res[b][h] - P[h] for h in part],
                                        [min(s - P[h], C - 64 - res[b][h] - P[h]) for h in part], 0.2)))
        for h in range(H):
            if kind != "proxy":
                put(res[b][h], head(h, res[b][h], k.get(h) if kind == "adakv" else None))
                continue
            qv = q[h][:, w - val:].reshape(1, 1, -1, d)
            tau = torch.full(qv.shape[:3], TAU, dtype=torch.float64, device="cuda")

            def attend(kc, vc, logc, r, n):
                t = [torch.tensor([[y]], device="cuda") for y in (r, n)]
                return _decode64(qv, kc[None, None], vc[None, None], logc[None, None], *t, tau)[0]

            none = torch.full((1,), -math.inf, dtype=torch.float64, device="cuda")
            whole = attend(K[h], V[h], none, 0, s)
            loss, cands = [], [int(math.floor(f * bud + 0.5)) for f in GRID]
            built = [head(h, r) for r in cands]
            for r, y in zip(cands, built):  # decoded from the cache as stored
                o = attend(y[0].to(_dt(case)).double(), y[1].to(_dt(case)).double(), y[2], r, y[4])
                loss.append(float(((o - whole) ** 2).sum() / qv.shape[2]))
            best = min((i for i, r in enumerate(cands) if r > 0), key=lambda i: (loss[i], cands[i]))
            pick = best if loss[best] < 0.99 * loss[0] else 0
            got["loss"].append(torch.tensor(loss, dtype=torch.float64))
            put(cands[pick], built[pick])
    out = {k: torch.stack(got[k]).reshape(B, H, *got[k][0].shape) for k in ("kc", "vc", "logc", "main_idx")}
    for k in ("res_len", "main_len"):
        out[k] = torch.tensor(got[k], dtype=torch.int32)
    if kind == "proxy":
        out["loss"] = torch.stack(got["loss"])
    return out


def exact(case, seed):
    return _exact_decode(case, seed) if case["kind"] in DECODE else _exact_build(case, seed)
