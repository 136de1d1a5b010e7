"""Performance cases of the selective KV-cache transfer path on one GPU.

Every case is one call (or one short chain of calls) that a serving program
makes through ``paper_2607_28150_amd``: the prefill side's scoring and
selection, the push of the chosen rows or blocks, and the decode side's index
split, on-demand gather, decode-time selection and attention.  Shapes are the
attention shapes of the synthetic workloads (8B- and 70B-shaped GQA heads of
128, the small 8-head model of 64), prompts 2K to 32K tokens, one request or a
varlen batch.  ``listed()`` gives the fixed cases, ``draw()`` others of the
same ranges; ``exact()`` recomputes the numbers in 64 bits with plain torch.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2607_28150_amd import smartgen as sg
from paper_2607_28150_amd.lanes import StepBuffers, TwoLane

DEV = "cuda"
DT = {"f32": torch.float32, "bf16": torch.bfloat16}
SINKS = 4                       # leading tokens that every query attends to
HEAVY = 100                     # one token in HEAVY is a heavy hitter


def listed():
    b8 = dict(dtype="bf16", Hq=32, Hkv=8, d=128)      # Llama-3-8B-shaped attention
    b70 = dict(dtype="bf16", Hq=64, Hkv=8, d=128)     # 70B-shaped attention
    return [
        # one layer of a small fp32 model scored at the end of its prefill: a call of two short launches
        dict(name="score_layer_f32", kind="score", dtype="f32", B=1, L=1, Hq=8, Hkv=8, d=64, W=32, lo=2048, hi=2048,
             lse=False),
        # one 8K prompt, all layers scored after its prefill, without the prefill's row normalisers
        dict(name="score_8k", kind="score", B=1, L=32, W=64, lo=8192, hi=8192, lse=False, **b8),
        # a varlen prefill batch whose attention kernel handed over the window rows' log-sum-exp
        dict(name="score_batch_lse", kind="score", B=8, L=16, W=64, lo=2048, hi=32768, lse=True, **b8),
        # selection counts under the alpha threshold, 8 query heads per KV head (a stage of a 70B-shaped model)
        dict(name="count_16k_g8", kind="count", B=1, L=20, W=64, lo=16384, hi=16384, alpha=5.0, **b70),
        # selection counts when every row picks the top 20% of its keys
        dict(name="topshare_8k", kind="topshare", B=1, L=32, W=64, lo=8192, hi=8192, ratio=2000, **b8),
        # top 10% of one prompt's rows, packed for the transfer
        dict(name="select_8k", kind="select", B=1, L=32, lo=8192, hi=8192, budget=1000, **b8),
        # the same for a varlen batch on one stage's layers
        dict(name="select_batch", kind="select", B=16, L=8, lo=2048, hi=32768, budget=1000, **b8),
        # block-granular proactive transfer of a long prompt: importance, the global top blocks, the push
        dict(name="blocks_32k", kind="blocks", L=32, N=32768, M=1024, share=1500, **b8),
        # one decode step with on-demand transfer from the prefill side's copy in pinned host memory
        dict(name="step_32k", kind="step", L=8, N=32768, budget=500, extra=200, page=16, host=True, **b8),
        # decode-time dynamic selection (alpha rule, capped at 20%) of one request, every layer
        dict(name="dselect_8k", kind="dselect", B=1, L=32, lo=8192, hi=8192, alpha=5.0, cap=2000, **b8),
        # attention of one layer for one request over its 10%: the smallest decode call
        dict(name="decode_one", kind="decode", B=1, lo=819, hi=819, page=16, **b8),
        # attention of one layer for 64 requests of different lengths (12% of 2K to 32K tokens)
        dict(name="decode_batch", kind="decode", B=64, lo=245, hi=3932, page=16, **b8),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["score", "score", "count", "topshare", "select", "blocks", "step", "dselect", "decode",
                       "decode"])
    dtype = "f32" if rng.random() < 0.2 else "bf16"
    d = 64 if rng.random() < 0.25 else 128
    Hkv = rng.choice([4, 8])
    G = rng.choice([1, 2, 4, 4, 8])
    c = dict(kind=kind, dtype=dtype, Hq=G * Hkv, Hkv=Hkv, d=d)
    if kind in ("score", "count", "topshare"):
        c["W"] = min(512 // G, rng.choice([16, 32, 48, 64, 64]) + rng.choice([0, 0, 1]))
    if kind in ("score", "count", "topshare", "select", "dselect"):
        c["B"] = _log(rng, 1, 16)
        c["L"] = _log(rng, 1, 32)
        c["hi"] = _log(rng, 2048, 32768)
        c["lo"] = rng.randint(max(1024, c["hi"] // 4), c["hi"])
    if kind == "score":
        c["lse"] = rng.random() < 0.5
    elif kind == "count":
        c["alpha"] = rng.choice([4.0, 5.0, 6.0])
    elif kind == "topshare":
        c["ratio"] = rng.randint(500, 4000)
    elif kind == "select":
        c["budget"] = rng.randint(300, 2000)
    elif kind == "dselect":
        c["alpha"] = 5.0
        c["cap"] = rng.randint(500, 2500)
        c["d"] = rng.choice([40, 64, 128, 128])
    elif kind == "blocks":
        c.update(L=_log(rng, 4, 32), N=_log(rng, 4096, 32768), M=rng.choice([256, 512, 1024]),
                 share=rng.randint(700, 3000))
    elif kind == "step":
        c.update(L=_log(rng, 1, 8), N=_log(rng, 2048, 32768), budget=rng.randint(300, 1500),
                 extra=rng.randint(30, 200), page=rng.choice([1, 16, 16, 24, 64]), host=rng.random() < 0.5)
    elif kind == "decode":
        c["B"] = _log(rng, 1, 64)
        c["hi"] = _log(rng, 100, 4000)
        c["lo"] = rng.randint(max(1, c["hi"] // 8), c["hi"])
        c["page"] = rng.choice([1, 16, 16, 24, 64])
        if rng.random() < 0.2:
            c["Hq"], c["Hkv"] = 64, 4          # 16 query heads per KV head
    top = {m: max(work(x)[m] for x in listed()) for m in ("bytes", "flops")}
    while any(work(c)[m] > top[m] for m in top):       # no drawn case is larger than the largest listed one
        if c.get("L", 1) > 1:
            c["L"] = c["L"] // 2
        else:
            c["B"] = c["B"] // 2
    return c


# ------------------------------------------------------------------ sizes

def _lens(c):
    """The requests' lengths: a fixed spread over [lo, hi] (the same in every run of the case)."""
    r = random.Random("%d %d %d" % (c["B"], c["lo"], c["hi"]))
    return [r.randint(c["lo"], c["hi"]) for _ in range(c["B"])] if c["B"] > 1 else [c["hi"]]


def _cu(lens):
    out = [0]
    for n in lens:
        out.append(out[-1] + n)
    return out


def _share(n, bp):
    return max(1, n * bp // 10000)


def work(c):
    """Bytes: every input row read once, every output written once.  Flops: one contraction of the window (or
    decode) queries with the keys they see, and for attention the weighted sum of the values."""
    es, d, Hq, Hkv = (4 if c["dtype"] == "f32" else 2), c["d"], c["Hq"], c["Hkv"]
    kind, row = c["kind"], c["d"] * (4 if c["dtype"] == "f32" else 2)
    if kind in ("score", "count", "topshare"):
        lens, L, W = _lens(c), c["L"], c["W"]
        keys = sum(W * n - W * (W - 1) // 2 for n in lens)
        by = L * Hkv * sum(lens) * (row + 4) + c["B"] * L * Hq * W * (row + (4 if c.get("lse") else 0))
        return {"bytes": by, "flops": 2 * d * Hq * L * keys}
    if kind == "select":
        lens, L = _lens(c), c["L"]
        K = sum(_share(n, c["budget"]) for n in lens)
        return {"bytes": L * Hkv * (4 * sum(lens) + K * (4 * row + 8)), "flops": 0}
    if kind == "blocks":
        L, N, M = c["L"], c["N"], c["M"]
        Kr = sg.block_budget(M, L, c["share"] / 10000, 1.0)
        Nb = -(-N // M)
        return {"bytes": 4 * L * Hkv * N + 4 * L * M + 8 * Kr + Kr * Hkv * Nb * 4 * row, "flops": L * Hkv * N}
    if kind == "step":
        L, N = c["L"], c["N"]
        n = _share(N, c["budget"]) + _share(N, c["extra"])
        # the split, the gathered rows moved once into the pool, the pool read once by the attention
        return {"bytes": L * Hkv * n * (4 * 4 + 1 + 2 * 2 * row + 2 * row) + L * Hq * d * (es + 4),
                "flops": 4 * L * Hq * n * d}
    if kind == "dselect":
        lens, L = _lens(c), c["L"]
        return {"bytes": L * Hkv * (sum(lens) * row + 4 * sum(_share(n, c["cap"]) for n in lens)),
                "flops": 2 * d * Hq * L * sum(lens)}
    rows = sum(_lens(c))
    return {"bytes": Hkv * rows * 2 * row + c["B"] * Hq * d * (es + 4), "flops": 4 * Hq * d * rows}


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _i32(x):
    return torch.tensor(x, dtype=torch.int32, device=DEV)


def _means(c, g, B, L):
    """A mean query per (layer, request, KV head): what a head's window and decode queries have in common."""
    return torch.randn((L, B, c["Hkv"], c["d"]), generator=g, device=DEV)


def _queries(c, g, mu, *shape):
    """Queries around their unit's mean: [B][L][Hq]`shape`[d]."""
    L, B, Hkv, d = mu.shape
    G = c["Hq"] // Hkv
    m = mu.permute(1, 0, 2, 3).repeat_interleave(G, dim=2).reshape(B, L, c["Hq"], *([1] * len(shape)), d)
    return (m + torch.randn((B, L, c["Hq"], *shape, d), generator=g, device=DEV)).to(DT[c["dtype"]])


def _keys(c, g, mu, lens):
    """Keys [L][Hkv][T][d] ~ N(0, 1); the first tokens of a request and one token in a hundred lean towards
    their unit's mean query (component 4 along it)."""
    L, B, Hkv, d = mu.shape
    cu, T = _cu(lens), sum(lens)
    k = torch.randn((L, Hkv, T, d), generator=g, device=DEV, dtype=DT[c["dtype"]])
    unit = mu / mu.norm(dim=-1, keepdim=True)
    req = torch.repeat_interleave(torch.arange(B, device=DEV), torch.tensor(lens, device=DEV))
    sinks = torch.cat([torch.arange(s, min(s + SINKS, e), device=DEV) for s, e in zip(cu, cu[1:])])
    head = torch.arange(Hkv, device=DEV)[:, None]
    for l in range(L):
        pos = torch.randperm(T, generator=g, device=DEV)[:max(1, T // HEAVY)]
        pos = torch.unique(torch.cat([sinks, pos])).expand(Hkv, -1)
        u = unit[l, req[pos], head]
        rows = k[l, head, pos].float()
        k[l, head, pos] = (rows + (4.0 - (rows * u).sum(-1, keepdim=True)) * u).to(k.dtype)
    return k


def _window_logits(c, q, k, b, l, s0, n, dtype):
    """Raw products and the causal limit of one request and layer: [Hkv][G * W][n]."""
    Hkv, W = c["Hkv"], c["W"]
    qq = q[b, l].reshape(Hkv, -1, c["d"]).to(dtype)
    z = qq @ k[l, :, s0:s0 + n].to(dtype).transpose(1, 2).contiguous()
    last = n - W + torch.arange(qq.shape[1], device=DEV) % W
    return z.masked_fill_(torch.arange(n, device=DEV)[None, None, :] > last[None, :, None], -math.inf)


def _row_lse(c, q, k, lens):
    """The log-sum-exp of each window row's scaled causal logits, as the prefill attention has it."""
    out = torch.empty((c["B"], c["L"], c["Hq"], c["W"]), device=DEV)
    for b, (s0, n) in enumerate(zip(_cu(lens), lens)):
        for l in range(c["L"]):
            z = _window_logits(c, q, k, b, l, s0, n, torch.float32)
            out[b, l] = torch.logsumexp(z * c["d"] ** -0.5, dim=-1).reshape(c["Hq"], c["W"])
    return out


def _bytes(n):
    return torch.empty(max(16, int(n)), dtype=torch.uint8, device=DEV)


def _pages(g, units, rows, page):
    """A page table whose pages lie at random places of the pool, and the pool's rows."""
    per = -(-rows // page)
    order = torch.randperm(units * per, generator=g, device=DEV)
    return (order * page).to(torch.int32).reshape(units, per), units * per * page


def prepare(c, seed):
    g, dt, Hq, Hkv, d = _gen(seed), DT[c["dtype"]], c["Hq"], c["Hkv"], c["d"]
    return globals()["_prepare_" + {"count": "score", "topshare": "score"}.get(c["kind"], c["kind"])](
        c, g, dt, Hq, Hkv, d)


def _prepare_score(c, g, dt, Hq, Hkv, d):
    B, L, W, lens = c["B"], c["L"], c["W"], _lens(c)
    T, top = sum(lens), max(lens)
    mu = _means(c, g, B, L)
    q = _queries(c, g, mu, W)
    k = _keys(c, g, mu, lens)
    size = sg.score_topshare_workspace_size if c["kind"] == "topshare" else sg.score_workspace_size
    return dict(c=c, q=q, k=k, cu=_i32(_cu(lens)), T=T, top=top, ws=_bytes(size(B, L, Hq, Hkv, d, W, top)),
                out=torch.empty((L, Hkv, T), device=DEV), lse=_row_lse(c, q, k, lens) if c.get("lse") else None)


def _prepare_select(c, g, dt, Hq, Hkv, d):
    L, lens = c["L"], _lens(c)
    T = sum(lens)
    ks = [_share(n, c["budget"]) for n in lens]
    K = sum(ks)
    # window scores: sums of softmax probabilities, spread over several powers of two
    scores = torch.exp(2.0 * torch.randn((L, Hkv, T), generator=g, device=DEV)) * (32.0 / T)
    k = torch.randn((L, Hkv, T, d), generator=g, device=DEV, dtype=dt)
    v = torch.randn((L, Hkv, T, d), generator=g, device=DEV, dtype=dt)
    return dict(c=c, scores=scores, k=k, v=v, cu=_i32(_cu(lens)), cuk=_i32(_cu(ks)), T=T, K=K, top=max(lens),
                max_k=max(ks), idx=torch.empty((L, Hkv, K), dtype=torch.int32, device=DEV),
                dst=_bytes(sg.pack_bytes(dt, L, Hkv, d, K)))


def _prepare_blocks(c, g, dt, Hq, Hkv, d):
    L, N, M = c["L"], c["N"], c["M"]
    Kr = sg.block_budget(M, L, c["share"] / 10000, 1.0)
    Nb = -(-N // M)
    level = torch.exp(torch.randn((L, 1, M), generator=g, device=DEV)).repeat_interleave(Nb, dim=2)[:, :, :N]
    scores = level * torch.rand((L, Hkv, N), generator=g, device=DEV) * (64.0 / N)
    k = torch.randn((L, Hkv, N, d), generator=g, device=DEV, dtype=dt)
    v = torch.randn((L, Hkv, N, d), generator=g, device=DEV, dtype=dt)
    return dict(c=c, scores=scores, k=k, v=v, cu=_i32([0, N]), row=_i32([0, L * M]), cuk=_i32([0, Kr]), Kr=Kr,
                imp=torch.empty((1, L, M), device=DEV), ids=torch.empty(Kr, dtype=torch.int32, device=DEV),
                dst=_bytes(sg.pack_blocks_bytes(dt, Hkv, d, N, M, Kr)))


def _prepare_dselect(c, g, dt, Hq, Hkv, d):
    B, L, lens = c["B"], c["L"], _lens(c)
    T, caps = sum(lens), [_share(n, c["cap"]) for n in lens]
    mu = _means(c, g, B, L)
    i32 = dict(dtype=torch.int32, device=DEV)
    return dict(c=c, q=_queries(c, g, mu), k=_keys(c, g, mu, lens), cu=_i32(_cu(lens)), cap=_i32(_cu(caps)), T=T,
                top=max(lens), K=sum(caps), idx=torch.empty((L, Hkv, sum(caps)), **i32),
                n_sel=torch.empty((B, L, Hkv), **i32),
                ws=_bytes(sg.decode_select_workspace_size(B, L, Hq, max(lens))))


def _attention(c, g, dt, B, Hq, Hkv, d, rows, page):
    """Queries, page table, output and workspace of a decode call over `rows` rows at most per unit."""
    table, pool_rows = _pages(g, B * Hkv, rows, page)
    return dict(q=torch.randn((B, Hq, d), generator=g, device=DEV).to(dt), table=table.reshape(B, Hkv, -1),
                pool_rows=pool_rows, o=torch.empty((B, Hq, d), device=DEV),
                ws=_bytes(sg.decode_workspace_size(B, Hq, Hkv, d, table.shape[1], page)))


def _prepare_decode(c, g, dt, Hq, Hkv, d):
    B, page, lens = c["B"], c["page"], _lens(c)
    s = _attention(c, g, dt, B, Hq, Hkv, d, max(lens), page)
    # only the pages that a request has rows for lie in its pool: the others point at its first page
    per = s["table"].shape[2]
    need = [-(-n // page) for n in lens]
    order = torch.randperm(sum(need) * Hkv, generator=g, device=DEV).to(torch.int32) * page
    table, at = torch.empty((B, Hkv, per), dtype=torch.int32, device=DEV), 0
    for b, m in enumerate(need):
        own = order[at:at + m * Hkv].reshape(Hkv, m)
        table[b, :, :m], table[b, :, m:] = own, own[:, :1]
        at += m * Hkv
    rows = sum(need) * Hkv * page
    s.update(c=c, table=table, pool_rows=rows, n=_i32(lens)[:, None].expand(B, Hkv).contiguous(),
             k=torch.randn((rows, d), generator=g, device=DEV, dtype=dt),
             v=torch.randn((rows, d), generator=g, device=DEV, dtype=dt))
    s["call"] = sg.DecodeCall(s["q"], s["k"], s["v"], table, s["n"], page, s["o"], ws=s["ws"])
    return s


def _prepare_step(c, g, dt, Hq, Hkv, d):
    L, N, page = c["L"], c["N"], c["page"]
    units, ks, ke = L * Hkv, _share(N, c["budget"]), _share(N, c["extra"])
    n = ks + ke
    # a decode side that holds the budget's rows; the step asks for all of them and `ke` others, in any order
    pick = torch.rand((units, N), generator=g, device=DEV).argsort(dim=1)[:, :n]
    mask = torch.full((units, N), 2, dtype=torch.int8, device=DEV).scatter_(1, pick[:, :ks], 1)
    mix = torch.rand((units, n), generator=g, device=DEV).argsort(dim=1)
    store_k = torch.randn((L, Hkv, N, d), generator=g, device=DEV, dtype=dt)
    store_v = torch.randn((L, Hkv, N, d), generator=g, device=DEV, dtype=dt)
    src = [store_k.cpu().pin_memory(), store_v.cpu().pin_memory()] if c["host"] else [store_k.clone(), store_v.clone()]
    far = mask.reshape(L, Hkv, N) == 2                  # what the decode side does not hold is not in its store
    store_k[far], store_v[far] = 0, 0
    s = _attention(c, g, dt, L, Hq, Hkv, d, n, page)
    base = torch.arange(units, dtype=torch.int64, device=DEV) * N
    s.update(c=c, lanes=TwoLane(), buf=StepBuffers.alloc(units, units * n),
             row_off=torch.arange(units + 1, dtype=torch.int32, device=DEV) * n,
             index=pick.gather(1, mix).to(torch.int32).reshape(-1).contiguous(), mask=mask.reshape(-1), base=base,
             mask_len=torch.full((units,), N, dtype=torch.int32, device=DEV), store_k=store_k, store_v=store_v,
             src_k=src[0], src_v=src[1], k=torch.zeros((s["pool_rows"], d), dtype=dt, device=DEV),
             v=torch.zeros((s["pool_rows"], d), dtype=dt, device=DEV))
    return s


# ------------------------------------------------------------------ one pass

def run(s):
    c = s["c"]
    kind, Hkv = c["kind"], c["Hkv"]
    if kind == "score":
        return sg.sg_score(s["q"], s["k"], s["cu"], s["T"], s["top"], Hkv, s["out"], ws=s["ws"], lse_in=s["lse"],
                           k_layer_rows=Hkv * s["T"])
    if kind == "count":
        return sg.sg_score_count(s["q"], s["k"], s["cu"], s["T"], s["top"], Hkv, s["out"], c["alpha"], s["ws"],
                                 k_layer_rows=Hkv * s["T"])
    if kind == "topshare":
        return sg.sg_score_topshare(s["q"], s["k"], s["cu"], s["T"], s["top"], Hkv, s["out"], c["ratio"], s["ws"],
                                    k_layer_rows=Hkv * s["T"])
    if kind == "select":
        sg.sg_topk(s["scores"], s["cu"], s["T"], s["top"], s["cuk"], s["K"], s["idx"])
        sg.sg_pack(s["k"], s["v"], s["idx"], s["cu"], s["T"], s["cuk"], s["K"], s["max_k"], s["dst"])
        return s["idx"], s["dst"]
    if kind == "blocks":
        L, M, N = c["L"], c["M"], c["N"]
        sg.sg_block_importance(s["scores"], s["cu"], N, M, s["imp"])
        sg.sg_topk(s["imp"].view(1, 1, L * M), s["row"], L * M, L * M, s["cuk"], s["Kr"], s["ids"].view(1, 1, -1))
        sg.sg_pack_blocks(s["k"], s["v"], s["ids"], 0, N, M, s["dst"])
        return s["imp"], s["ids"], s["dst"]
    if kind == "dselect":
        sg.sg_decode_select(s["q"], s["k"], s["cu"], s["T"], s["top"], Hkv, s["cap"], s["K"], s["idx"], s["n_sel"],
                            c["alpha"], s["ws"], k_layer_rows=Hkv * s["T"])
        return s["idx"], s["n_sel"]
    if kind == "decode":
        s["call"](s["q"], s["k"], s["v"], s["o"])
        return s["o"]
    # one decode step: split the index, fill the pool on two lanes, attend
    b = s["buf"]
    kept = s["lanes"].gather(row_off=s["row_off"], kv_index=s["index"], mask=s["mask"], mask_off=s["base"],
                             mask_len=s["mask_len"], store_k=s["store_k"], store_v=s["store_v"],
                             store_base=s["base"], src_k=s["src_k"], src_v=s["src_v"], src_base=s["base"],
                             page_table=s["table"].view(c["L"] * Hkv, -1), page_size=c["page"], k_pool=s["k"],
                             v_pool=s["v"], buf=b, reuse=False)
    sg.sg_decode_attn(s["q"], s["k"], s["v"], s["table"], kept.view(c["L"], Hkv), c["page"], s["o"], ws=s["ws"])
    return s["o"], b.order, b.local, b.remote, b.n_local, b.n_remote, b.n_kept


# ------------------------------------------------------------------ what is right

def tolerance(c):
    kind = c["kind"]
    if kind == "select":
        return "exact"                        # ids and copied bytes
    if kind == "score":
        return {"rel": 4e-6, "max": 4e-5}     # fp32 sums of fp32 exponentials of fp32 logits
    if kind in ("count", "topshare"):
        # whole picks as floats: a logit within a rounding of its row's threshold may fall on either side
        return {"rel": 2e-4, "max": 0.99}
    if kind == "blocks":
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.01}
    if kind == "dselect":
        return {"rel": 0.0, "differ": 0.01}   # an id on the rule's edge shifts its unit's later ids
    return {"rel": 2e-6, "max": 4e-5, "differ": 0.0}


def _exact_window(c, s):
    lens, W = _lens(c), c["W"]
    out = torch.zeros((c["L"], c["Hkv"], s["T"]), dtype=torch.float64, device=DEV)
    for b, (s0, n) in enumerate(zip(_cu(lens), lens)):
        if n < W:
            continue
        for l in range(c["L"]):
            z = _window_logits(c, s["q"], s["k"], b, l, s0, n, torch.float64)
            if c["kind"] == "score":
                z *= c["d"] ** -0.5
                lse = (torch.logsumexp(z, dim=-1) if s["lse"] is None
                       else s["lse"][b, l].reshape(c["Hkv"], -1).double())
                r = torch.exp(z - lse[..., None])
            elif c["kind"] == "count":
                r = z >= z.amax(dim=-1, keepdim=True) - c["alpha"] * c["d"] ** 0.5
            else:
                seen = n - W + 1 + torch.arange(z.shape[1], device=DEV) % W
                kth = (seen * c["ratio"] // 10000).clamp(min=1)
                order = torch.sort(z, dim=-1, descending=True).values
                r = z >= order.gather(2, (kth - 1)[None, :, None].expand(z.shape[0], -1, 1))
            out[l, :, s0:s0 + n] = r.double().sum(dim=1)
    return out


def _softmax_rows(q, k, v):
    """q [Hkv][G][d], k and v [Hkv][n][d] in 64 bits."""
    p = torch.softmax((q @ k.transpose(1, 2).contiguous()) * q.shape[-1] ** -0.5, dim=-1)
    return (p @ v).reshape(-1, q.shape[-1])


def exact(c, seed):
    kind, Hkv, d = c["kind"], c["Hkv"], c["d"]
    if kind in ("select", "dselect"):
        return None                           # whole numbers and bytes
    s = prepare(c, seed)
    if kind in ("score", "count", "topshare"):
        return _exact_window(c, s)
    if kind == "blocks":
        L, M, N = c["L"], c["M"], c["N"]
        Nb = -(-N // M)
        x = torch.zeros((L, Hkv, M * Nb), dtype=torch.float64, device=DEV)
        x[:, :, :N] = s["scores"].double()
        left = (N - torch.arange(M, device=DEV) * Nb).clamp(0, Nb)
        imp = x.reshape(L, Hkv, M, Nb).sum(dim=(1, 3)) / (left * Hkv)
        imp[:, left == 0] = -math.inf
        imp[:2] = math.inf
        return imp[None], None, None
    out = []
    if kind == "decode":
        page = c["page"]
        for b, n in enumerate(_lens(c)):
            rows = (s["table"][b].long()[:, :, None] + torch.arange(page, device=DEV)).reshape(Hkv, -1)[:, :n]
            out.append(_softmax_rows(s["q"][b].reshape(Hkv, -1, d).double(), s["k"][rows].double(),
                                     s["v"][rows].double()))
        return torch.stack(out)
    idx = s["index"].long().reshape(c["L"], Hkv, -1)
    head = torch.arange(Hkv)[:, None]
    for l in range(c["L"]):
        at = idx[l].to(s["src_k"].device)
        k, v = (x[l][head.to(at.device), at].to(DEV).double() for x in (s["src_k"], s["src_v"]))
        out.append(_softmax_rows(s["q"][l].reshape(Hkv, -1, d).double(), k, v))
    return (torch.stack(out),) + (None,) * 6
