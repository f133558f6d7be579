"""Timed cases of the CompKV decode-step attention library, through its public Python calls.

A case is one pass of the work a decoder gives this library, in one of five calls:

  step     one token through `layers` attention layers, each one compkv_decode_step (append when `append`,
           scoring, selection, compensated sparse attention);
  split    the same layers as compkv_score_select followed by compkv_sparse_decode;
  prefill  compkv_build_stats over a whole cache;
  append   compkv_append_stats of one token per sequence;
  dense    compkv_dense_decode, the full-attention baseline.

With `graph` the calls of a pass are captured once into a HIP graph (a decoder captures its step and replays
it for every token, which is what the calls' allocation-free interface is for) and a pass replays it; without
it a pass makes the calls themselves. Each layer has its own cache and summaries, so a pass reads memory
like consecutive layers of a model. All inputs are drawn on the GPU from the seed, by the recipe of
workloads/gqa_decode.py: block centroids N(0, I), a spread per block, values N(0, I), queries
N(0, I) / sqrt(128).
"""
from __future__ import annotations

import math

import torch

import paper_2609_26300_amd as P

DEV = "cuda"
N_SINK, N_RECENT = 1, 2


def _case(name, call, batch, hq, hkv, d, ctx, B, K=0, r=4, layout=0, ragged=False, page=0, layers=1, append=False,
          graph=False, sigma="loguniform"):
    return dict(name=name, call=call, batch=batch, hq=hq, hkv=hkv, d=d, ctx=ctx, B=B, K=K, r=r, layout=layout,
                ragged=ragged, page=page, layers=layers, append=append, graph=graph, sigma=sigma)


def listed():
    return [
        # the smallest call: one layer of a short chat on a small model, called directly (launch latency)
        _case("step_4k_direct", "step", 1, 8, 2, 128, 4096, 16, K=16, append=True),
        # one user's token through eight layers at 32K, the Llama-3-8B-shaped layer
        _case("step_32k", "step", 1, 32, 8, 128, 32768, 32, K=65, layers=8, append=True, graph=True),
        # four long documents: the benchmark's default layer
        _case("step_128k", "step", 4, 32, 8, 128, 131072, 32, K=64, layers=2, append=True, graph=True,
              sigma="lognormal"),
        # wide GQA (64 query heads on 8 KV heads) with 64-token blocks
        _case("step_wide_64k", "step", 8, 64, 8, 128, 65536, 64, K=32, layers=2, append=True, graph=True),
        # batched serving: 32 sequences of different lengths in a paged cache
        _case("step_batch_8k", "step", 32, 32, 8, 128, 8192, 16, K=64, ragged=True, page=64, layers=2, append=True,
              graph=True),
        # an attention layer without grouped queries, 64-wide heads, odd sizes, interleaved RoPE pairs
        _case("step_mha_d64", "step", 3, 12, 12, 64, 20011, 48, K=24, r=8, layout=1, ragged=True, layers=4,
              append=True, graph=True),
        # the finest summary (a variance per coordinate) at the 512-token budget, as the separate calls
        _case("split_16k_rd", "split", 2, 32, 8, 128, 16384, 16, K=32, r=128, layers=4, graph=True,
              sigma="lognormal"),
        # prompt processing: the summaries of one layer's cache
        _case("prefill_32k", "prefill", 1, 32, 8, 128, 32768, 32),
        _case("prefill_128k", "prefill", 4, 32, 8, 128, 131072, 32, sigma="lognormal"),
        _case("prefill_wide_64k", "prefill", 8, 64, 8, 128, 65536, 64),
        # the full-attention baseline on the 32K layer
        _case("dense_32k", "dense", 1, 32, 8, 128, 32768, 32),
        # one appended token per sequence as its own call (scoring left to a later call)
        _case("append_64k_direct", "append", 4, 32, 8, 128, 65500, 32, append=True),
    ]


# the largest drawn cache, in tokens x KV heads x layers x head_dim / 128 (the 128K layer twice is 8 Mi)
_MOST_ROWS = 4 << 20


def draw(rng):
    call = rng.choice(["step"] * 5 + ["split"] * 2 + ["prefill"] * 3 + ["dense"] * 2 + ["append"])
    G = rng.choice([1, 2, 4, 4, 8])
    hkv = rng.choice([1, 2, 4, 5, 8, 8])
    d = rng.choice([64, 128, 128, 128])
    B = rng.choice([16, 16, 32, 32, 64, 24, 48, 100, 128])
    ctx = int(round(math.exp(rng.uniform(math.log(1024), math.log(131072)))))
    layers = rng.choice([1, 2, 4]) if call in ("step", "split") else 1
    most = max(1, min(48, _MOST_ROWS // (ctx * hkv * layers)))
    batch = int(round(math.exp(rng.uniform(0.0, math.log(most)))))
    budget = int(round(math.exp(rng.uniform(math.log(256), math.log(4096)))))
    K = max(N_SINK + N_RECENT + 1, min(budget // B, -(-ctx // B)))
    page = rng.choice([0, 0, 0, 4 * B]) if call != "append" else 0
    c = _case("", call, batch, G * hkv, hkv, d, ctx, B, K=K if call in ("step", "split") else 0,
              r=rng.choice([4, 4, 4, 4, 1, 8, 16, d]), layout=rng.choice([0, 0, 1]), ragged=rng.random() < 0.5,
              page=page, layers=layers, append=call == "append" or (call == "step" and rng.random() < 0.8),
              graph=call in ("step", "split"), sigma=rng.choice(["loguniform", "lognormal"]))
    del c["name"]
    return c


# ------------------------------------------------------------------------------------------- inputs

def _lengths(c):
    """Tokens per sequence once the pass is done: `ctx`, or spread over [ctx / 8, ctx]."""
    if not c["ragged"]:
        return [c["ctx"]] * c["batch"]
    return [c["ctx"]] + [max(1, int(c["ctx"] * (0.125 + 0.875 * ((i * 0.6180339887498949) % 1.0))))
                         for i in range(1, c["batch"])]


def _capacity(c):
    unit = c["page"] or 1
    return -(-c["ctx"] // unit) * unit


def _inputs(c, seed):
    """Keys and values [layers][batch][hkv][capacity][d], queries, new rows (bf16) and the page permutation."""
    g = torch.Generator(device=DEV).manual_seed(int(seed))
    b, h, d, cap, L, B = c["batch"], c["hkv"], c["d"], _capacity(c), c["layers"], c["B"]
    X = -(-cap // B)

    def normal(*shape):
        return torch.randn(*shape, generator=g, device=DEV, dtype=torch.float32)

    k = torch.empty(L, b, h, cap, d, dtype=torch.bfloat16, device=DEV)
    v = torch.empty_like(k)
    for layer in range(L):
        for i in range(b):
            if c["sigma"] == "lognormal":
                spread = torch.exp(math.log(0.2) + normal(h, X, 1, 1))
            else:
                spread = torch.exp(math.log(0.05) + (math.log(1.0) - math.log(0.05)) *
                                   torch.rand(h, X, 1, 1, generator=g, device=DEV))
            x = (normal(h, X, 1, d) + spread * normal(h, X, B, d)).reshape(h, X * B, d)
            k[layer, i] = x[:, :cap]
            v[layer, i] = normal(h, cap, d)
    q = (normal(L, b, c["hq"], d) / math.sqrt(128.0)).to(torch.bfloat16)
    k_new = normal(L, b, h, d).to(torch.bfloat16)
    v_new = normal(L, b, h, d).to(torch.bfloat16)
    perm = torch.randperm(b * cap // c["page"], generator=g, device=DEV) if c["page"] else None
    return k, v, q, k_new, v_new, perm


def _paged(c, x, perm):
    """[layers][batch][hkv][capacity][d] -> [layers][pages][hkv][page][d], logical page p at physical perm[p]."""
    L, b, h, cap, d = x.shape
    pages = x.view(L, b, h, cap // c["page"], c["page"], d).permute(0, 1, 3, 2, 4, 5).reshape(L, -1, h, c["page"], d)
    out = torch.empty_like(pages)
    out[:, perm] = pages
    return out


class _State:
    pass


def prepare(case, seed):
    c = case
    s = _State()
    s.case = c
    b, h, d, L = c["batch"], c["hkv"], c["d"], c["layers"]
    cap = _capacity(c)
    k, v, s.q, s.k_new, s.v_new, perm = _inputs(c, seed)
    if perm is not None:
        s.table = perm.view(b, cap // c["page"]).to(torch.int32).contiguous()
        k, v = _paged(c, k, perm), _paged(c, v, perm)
        s.dims = P.make_dims(b, c["hq"], h, d, c["B"], c["r"], cap, max_seq_len=c["ctx"], group_layout=c["layout"],
                             block_table=s.table, page_tokens=c["page"], num_pages=perm.numel())
    else:
        s.dims = P.make_dims(b, c["hq"], h, d, c["B"], c["r"], cap, max_seq_len=c["ctx"], group_layout=c["layout"])
    s.k, s.v = k, v
    s.after = torch.tensor(_lengths(c), dtype=torch.int32, device=DEV)
    s.before = s.after - 1 if c["append"] else s.after
    K = max(1, c["K"])
    s.scale = 1.0 / math.sqrt(d)
    s.params = P.CompkvSelectParams(K, N_SINK, N_RECENT, s.scale)
    X = s.dims.xcap

    def zeros(*shape, dtype=torch.float32):
        return torch.zeros(L, b, *shape, dtype=dtype, device=DEV)

    s.kmean, s.vmean, s.dvar = zeros(h, X, d), zeros(h, X, d), zeros(h, X, c["r"])
    s.sel, s.n_sel = zeros(h, K, dtype=torch.int32), zeros(h, dtype=torch.int32)
    s.blk_logit = zeros(h, c["hq"] // h, X)
    s.scores = zeros(h, X) if c["call"] == "split" else None
    s.out, s.lse = zeros(c["hq"], d), zeros(c["hq"])
    s.ws = P.alloc_workspace(s.dims, K, DEV)
    if c["call"] in ("step", "split", "append"):  # the summaries the prompt left
        for i in range(L):
            P.compkv_build_stats(s.dims, s.k[i], s.v[i], s.before, s.kmean[i], s.dvar[i], s.vmean[i])
    s.graph = None
    if c["graph"]:
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _layer(s, 0)
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        s.graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s.graph):
            for i in range(L):
                _layer(s, i)
    return s


def _layer(s, i):
    c, call = s.case, s.case["call"]
    if call == "step":
        new = (s.k_new[i], s.v_new[i]) if c["append"] else (None, None)
        P.compkv_decode_step(s.dims, s.params, s.q[i], s.k[i], s.v[i], *new, s.after, s.kmean[i], s.dvar[i],
                             s.vmean[i], s.sel[i], s.n_sel[i], s.blk_logit[i], None, s.out[i], s.lse[i], s.ws)
    elif call == "split":
        P.compkv_score_select(s.dims, s.params, s.q[i], s.kmean[i], s.dvar[i], s.after, s.sel[i], s.n_sel[i],
                              s.blk_logit[i], s.scores[i], s.ws)
        P.compkv_sparse_decode(s.dims, s.scale, s.q[i], s.k[i], s.v[i], s.vmean[i], s.blk_logit[i], s.after, s.sel[i],
                               s.n_sel[i], s.out[i], s.lse[i], s.ws)
    elif call == "prefill":
        P.compkv_build_stats(s.dims, s.k[i], s.v[i], s.after, s.kmean[i], s.dvar[i], s.vmean[i])
    elif call == "append":
        P.compkv_append_stats(s.dims, s.k[i], s.v[i], s.k_new[i], s.v_new[i], s.before, s.kmean[i], s.dvar[i],
                              s.vmean[i])
    else:
        P.compkv_dense_decode(s.dims, s.scale, s.q[i], s.k[i], s.v[i], s.after, s.out[i], s.lse[i], s.ws)


def run(state):
    s = state
    if s.graph is not None:
        s.graph.replay()
    else:
        for i in range(s.case["layers"]):
            _layer(s, i)
    call = s.case["call"]
    r = {}
    if call in ("prefill", "append", "step"):
        r.update(kmean=s.kmean, dvar=s.dvar, vmean=s.vmean)
    if call in ("step", "split"):
        r.update(sel=s.sel, n_sel=s.n_sel, blk_logit=s.blk_logit)
    if call == "split":
        r["scores"] = s.scores
    if call in ("step", "split", "dense"):
        r.update(out=s.out, lse=s.lse)
    if s.case["append"]:
        r.update(k_cache=s.k, v_cache=s.v)
    return r


# ------------------------------------------------------------------------- work, tolerance, reference

def work(case):
    """Bytes and operations of one pass. Scoring reads each block's mean key and variances, the attention the
    selected tokens' keys and values and the other blocks' mean values; an append writes a row, reads its
    block and rewrites that block's summary."""
    c = case
    d, r, B, h, G = c["d"], c["r"], c["B"], c["hkv"], c["hq"] // c["hkv"]
    nbytes = flops = 0
    for n in _lengths(c):
        X = -(-n // B)
        K = min(c["K"], X)
        tokens = min(K * B, n)
        if c["append"]:
            rows = n - (X - 1) * B
            nbytes += h * (4 * d * (rows + 1) + 8 * d + 4 * r)
            flops += h * rows * 6 * d
        if c["call"] in ("step", "split"):
            nbytes += h * (X * (4 * d + 4 * r) + (X - K) * 4 * d + tokens * 4 * d + 4 * X * G + 4 * K)
            flops += h * G * (X * 2 * (d + r) + (X - K) * 2 * d + tokens * 4 * d)
            nbytes += c["hq"] * 6 * d
        elif c["call"] == "prefill":
            nbytes += h * (n * 4 * d + X * (8 * d + 4 * r))
            flops += h * n * 5 * d
        elif c["call"] == "dense":
            nbytes += h * n * 4 * d + c["hq"] * 6 * d
            flops += h * G * n * 4 * d
    return {"bytes": float(nbytes * c["layers"]), "flops": float(flops * c["layers"])}


def tolerance(case):
    """About four times what the 32-bit sums measure against 64 bits: summaries 4e-8, dense attention 1.7e-7, a
    step's outputs 2e-7 and its scores 4.5e-7. Ids may differ where scores tie within that rounding."""
    if case["call"] in ("prefill", "append"):
        return {"rel": 2e-7, "max": 1e-5}
    if case["call"] == "dense":
        return {"rel": 1e-6, "max": 1e-4}
    return {"rel": 2e-6, "max": 2e-4, "differ": 0.01}


def _groups(c):
    """Variance group of every coordinate."""
    d, r = c["d"], c["r"]
    if r == d:
        return torch.arange(d, device=DEV)
    f = torch.arange(d, device=DEV)
    pair = f % (d // 2) if c["layout"] == 0 else f // 2
    return pair // (d // 2 // r)


def _block_sums(x, n, B):
    """Sums over the blocks of the first n rows of x [h][n][d] -> [h][X][d]."""
    X = -(-n // B)
    pad = X * B - n
    if pad:
        x = torch.cat([x, x.new_zeros(x.shape[0], pad, x.shape[2])], 1)
    return x.view(x.shape[0], X, B, x.shape[2]).sum(2)


def exact(case, seed):
    c = case
    b, h, d, B, L = c["batch"], c["hkv"], c["d"], c["B"], c["layers"]
    G, call = c["hq"] // h, c["call"]
    k, v, q, k_new, v_new, _ = _inputs(c, seed)
    lens = _lengths(c)
    X_cap = -(-_capacity(c) // B)
    f64 = torch.float64
    scale = float(torch.tensor(1.0 / math.sqrt(d), dtype=torch.float32))
    group = _groups(c)
    member = (group[:, None] == torch.arange(c["r"], device=DEV)[None, :]).to(f64)  # [d][r]

    def zeros(*shape):
        return torch.zeros(L, b, *shape, dtype=f64, device=DEV)

    kmean, vmean, dvar = zeros(h, X_cap, d), zeros(h, X_cap, d), zeros(h, X_cap, c["r"])
    logits, scores = zeros(h, G, X_cap), zeros(h, X_cap)
    out, lse = zeros(c["hq"], d), zeros(c["hq"])
    for layer in range(L):
        for i, n in enumerate(lens):
            kd, vd = k[layer, i, :, :n].to(f64), v[layer, i, :, :n].to(f64)
            if c["append"]:
                kd[:, n - 1], vd[:, n - 1] = k_new[layer, i].to(f64), v_new[layer, i].to(f64)
            qd = q[layer, i].to(f64).view(h, G, d)
            if call == "dense":
                z = torch.stack([(kd * qd[:, g, None]).sum(-1) for g in range(G)], 1) * scale
                out[layer, i] = torch.stack([(torch.softmax(z[:, g], -1)[..., None] * vd).sum(1)
                                             for g in range(G)], 1).view(c["hq"], d)
                lse[layer, i] = torch.logsumexp(z, -1).view(-1)
                continue
            X = -(-n // B)
            count = torch.full((X, 1), float(B), dtype=f64, device=DEV)
            count[-1] = n - (X - 1) * B
            km, vm = _block_sums(kd, n, B) / count, _block_sums(vd, n, B) / count
            dev = kd - km.repeat_interleave(B, 1)[:, :n]
            dv = ((_block_sums(dev * dev, n, B) / count)[..., None] * (member / member.sum(0))).sum(-2)
            del dev
            kmean[layer, i, :, :X], vmean[layer, i, :, :X], dvar[layer, i, :, :X] = km, vm, dv
            if call in ("prefill", "append"):
                continue
            qg = ((scale * qd) ** 2)[..., None] * member
            qg = qg.sum(-2)  # [h][G][r]
            z = torch.stack([(km * qd[:, g, None]).sum(-1) for g in range(G)], 1) * scale
            sig = torch.stack([(dv * qg[:, g, None]).sum(-1) for g in range(G)], 1)
            logits[layer, i, :, :, :X] = z
            lnb = torch.log(count[:, 0])
            score = (torch.softmax(lnb + z + 0.5 * sig, -1) * sig).sum(1)
            scores[layer, i, :, :X] = score
            K = min(c["K"], X)
            rank = score.clone()
            rank[:, :N_SINK] = math.inf
            rank[:, max(0, X - N_RECENT):] = math.inf
            order = torch.sort(rank, dim=-1, descending=True, stable=True).indices[:, :K]
            chosen = torch.zeros(h, X, dtype=torch.bool, device=DEV)
            chosen.scatter_(1, order, True)
            for u in range(h):
                tok = chosen[u].repeat_interleave(B)[:n]
                kt, vt = kd[u][tok], vd[u][tok]
                zt = scale * torch.stack([(kt * qd[u, g]).sum(-1) for g in range(G)])
                zm = (lnb + z[u])[:, ~chosen[u]]
                w = torch.cat([zt, zm], 1)
                vals = torch.cat([vt, vm[u][~chosen[u]]], 0)
                lse[layer, i, u * G:(u + 1) * G] = torch.logsumexp(w, -1)
                p = torch.softmax(w, -1)
                out[layer, i, u * G:(u + 1) * G] = torch.stack([(p[g][:, None] * vals).sum(0) for g in range(G)])
    r = {}
    if call in ("prefill", "append", "step"):
        r.update(kmean=kmean, dvar=dvar, vmean=vmean)
    if call in ("step", "split"):
        r.update(sel=None, n_sel=None, blk_logit=logits)
    if call == "split":
        r["scores"] = scores
    if call in ("step", "split", "dense"):
        r.update(out=out, lse=lse)
    if c["append"]:
        r.update(k_cache=None, v_cache=None)
    return r
