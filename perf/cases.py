"""Timed workloads of the sparse-verification path: what a serving program asks of the library.

Every case is one kind of call (`op`) at one shape:

  verify    one target layer of a verification step: draft scores -> index sets -> sparse attention
  select    mask generation alone
  sparse    sparse attention alone, over index sets that are already there
  dense     the dense attention of the same family (the layers that are not pruned)
  paged     block granularity: page selection, then sparse attention over a paged cache
  draft     a draft layer that hands its scores on: dense attention that sums its attention weights
            over the query block, or dumps its scaled logits, then the selection
  prefill   chunked prefill with an index set per query row: per-row selection, union, attention
  headmap   the offline head mapping (Algorithm 1) over two attention-weight traces

Calls that a serving loop repeats on fixed buffers go through prepared calls, as such a loop would
make them; the others are plain calls. All inputs live on the GPU.
"""
from __future__ import annotations

import math

import torch

import paper_2605_15508_amd as sts

DEV = "cuda"

# target layer shapes (query heads, KV heads, head size, draft heads): the 8B- and the 70B-shaped one
SHAPES = {"8b": (32, 8, 128, 16), "70b": (64, 8, 128, 32)}
# bytes that a drawn case may ask for at most: those of the largest listed case, rounded down
MOST_BYTES = 1.15e9


def listed():
    return [
        # The smallest call: one 8B-shaped layer at 4K of context, one sequence. Launches and latency.
        {"name": "verify-4k", "op": "verify", "shape": "8b", "B": 1, "N": 4096, "Tq": 5, "k": 410, "bf16": False, "tail": False},
        # An ordinary verification step: one sequence whose context has an arbitrary length (33001),
        # 10% kept, the block's own candidates appended causally.
        {"name": "verify-33k-odd", "op": "verify", "shape": "8b", "B": 1, "N": 33001, "Tq": 5, "k": 3301, "bf16": False, "tail": True},
        # Long context, one sequence of a million tokens, 2% kept.
        {"name": "verify-1m", "op": "verify", "shape": "8b", "B": 1, "N": 1048576, "Tq": 5, "k": 20972, "bf16": False, "tail": False},
        # The benchmark's mask generation: 128K of context, batch 4, 10%; sequences of different lengths.
        {"name": "select-128k-b4", "op": "select", "shape": "8b", "B": 4, "N": 131072, "Tq": 5, "k": 13108, "bf16": False, "ragged": True},
        # The benchmark's headline: sparse attention at 128K, batch 4, 10%.
        {"name": "sparse-128k-b4", "op": "sparse", "shape": "8b", "B": 4, "N": 131072, "Tq": 5, "k": 13108, "tail": False},
        # The same layer at the fixed budget of 512 tokens, own candidates appended: a short-list call.
        {"name": "sparse-128k-512", "op": "sparse", "shape": "8b", "B": 4, "N": 131072, "Tq": 5, "k": 512, "tail": True},
        # A layer that is not pruned: dense verification of three sequences of different lengths.
        {"name": "dense-100k-b3", "op": "dense", "shape": "8b", "B": 3, "N": 100003, "Tq": 5},
        # Block granularity over a paged cache: 820 pages of 16 tokens (10% of 128K), batch 4.
        {"name": "paged16-128k-b4", "op": "paged", "shape": "8b", "B": 4, "N": 131072, "Tq": 5, "k": 820, "page": 16},
        # 70B-shaped: the draft layer (head size 64) sums its attention weights for the selection.
        {"name": "draft-sum-128k-b4", "op": "draft", "shape": "70b", "B": 4, "N": 131072, "Tq": 8, "k": 13108, "dump": False},
        # The same hand-over by a bf16 dump of the scaled logits, at a shorter context.
        {"name": "draft-dump-50k-b4", "op": "draft", "shape": "70b", "B": 4, "N": 50000, "Tq": 8, "k": 5000, "dump": True},
        # Chunked prefill: 16 blocks of 16 query rows over one 64K cache, an index set per query row.
        {"name": "prefill-rows-64k", "op": "prefill", "shape": "8b", "B": 16, "N": 65536, "k": 6554},
        # Offline head mapping over traces of 128 query rows.
        {"name": "headmap-16k", "op": "headmap", "S": 2, "R": 64, "Hd": 16, "Ht": 32, "N": 16384, "k": 512},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _budget(rng, N):
    """A fraction of the context (2% to 20%) or one of the fixed budgets of short lists."""
    k = rng.choice([256, 512, 1024, 4096]) if rng.random() < 0.3 else math.ceil(N * rng.uniform(0.02, 0.2))
    return max(16, min(k, N))


def draw(rng):
    while True:
        op = rng.choice(["verify", "verify", "verify", "select", "select", "sparse", "sparse", "dense", "paged", "draft", "prefill", "headmap"])
        shape = rng.choice(["8b", "8b", "70b"])
        Tq = rng.randint(2, 9)
        B = rng.choice([1, 1, 2, 3, 4, 6, 8])
        N = _log(rng, 3000, 1000000)
        if rng.random() < 0.5:          # contexts of whole pages, and of any length
            N = max(4096, N // 64 * 64)
        c = {"op": op, "shape": shape, "B": B, "N": N, "Tq": Tq}
        if op == "verify":
            c.update(k=_budget(rng, N), bf16=rng.random() < 0.3, tail=rng.random() < 0.5)
        elif op == "select":
            c.update(k=_budget(rng, N), bf16=rng.random() < 0.3, ragged=rng.random() < 0.5)
        elif op == "sparse":
            c.update(k=_budget(rng, N), tail=rng.random() < 0.5)
        elif op == "paged":
            page = rng.choice([8, 16, 32])
            c.update(page=page, k=max(4, _budget(rng, N) // page))
        elif op == "draft":
            c.update(shape="70b", k=_budget(rng, N), dump=rng.random() < 0.5)
        elif op == "prefill":
            N = _log(rng, 8192, 131072)
            N = N // 64 * 64 if rng.random() < 0.5 else N
            c = {"op": op, "shape": "8b", "B": rng.randint(2, 24), "N": N, "k": max(256, math.ceil(N * rng.uniform(0.02, 0.12)))}
        elif op == "headmap":
            c = {"op": op, "S": rng.randint(1, 3), "R": rng.randint(16, 64), "Hd": rng.choice([8, 16, 32]), "Ht": 32,
                 "N": _log(rng, 2000, 24000), "k": rng.choice([64, 256, 512, 1000])}
        if work(c)["bytes"] <= MOST_BYTES:
            return c


# ------------------------------------------------------------------------------------ inputs

def _head_map(Hq, Hd):
    return (torch.arange(Hq) * Hd // Hq).to(torch.int32)


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV, dtype=torch.float32)


def _bf16(g, *shape, std=1.0):
    """Normal bf16 values, made slice by slice along the first dimension."""
    out = torch.empty(*shape, device=DEV, dtype=torch.bfloat16)
    for i in range(shape[0]):
        out[i] = _randn(g, *shape[1:]) * std
    return out


def _heavy_logits(g, rows, N):
    """Shared part of the rows' logits: unit normal, a percent of heavy tokens, sinks, a recent window."""
    lg = _randn(g, rows, N)
    heavy = torch.rand(rows, N, generator=g, device=DEV) < 0.01
    lg += heavy * (2.0 + _randn(g, rows, N).abs())
    lg[:, :4] += 4.0
    lg[:, -min(64, N):] += 1.5
    return lg


def _scores(g, B, Hd, Tq, N, noise=0.7, bf16=False, lens=None):
    """Draft attention weights [B,Hd,Tq,N]: the rows of a block share the heavy tokens up to noise."""
    out = torch.empty(B, Hd, Tq, N, device=DEV, dtype=torch.bfloat16 if bf16 else torch.float32)
    for b in range(B):
        lg = _heavy_logits(g, Hd, N)[:, None, :] + noise * _randn(g, Hd, Tq, N)
        if lens is not None:
            lg[:, :, int(lens[b]):] = float("-inf")
        out[b] = torch.softmax(lg, dim=-1)
    return out


def _cache(g, B, Hkv, N, d, q):
    """K, V [B,Hkv,N,d] bf16: normal, with a percent of the keys leaning towards the queries."""
    k = torch.empty(B, Hkv, N, d, device=DEV, dtype=torch.bfloat16)
    v = torch.empty(B, Hkv, N, d, device=DEV, dtype=torch.bfloat16)
    Tq, Hq = q.shape[1], q.shape[2]
    for b in range(B):
        qs = q[b if q.shape[0] == B else 0].float().reshape(Tq, Hkv, Hq // Hkv, d).sum(dim=(0, 2))
        qs = qs / qs.norm(dim=-1, keepdim=True)
        for h in range(Hkv):
            kh = _randn(g, N, d) * 0.5
            pos = torch.randint(0, N, (max(1, N // 100),), generator=g, device=DEV)
            kh[pos] += 3.0 * qs[h]
            k[b, h] = kh
            v[b, h] = _randn(g, N, d) * 0.5
    return k, v


def _index_lists(g, B, Hd, N, k, head_map):
    """Ascending random index lists [B,Hq,k], equal for the target heads of one draft head."""
    lists = torch.empty(B, Hd, k, device=DEV, dtype=torch.int64)
    for b in range(B):
        for j in range(Hd):
            lists[b, j] = torch.randperm(N, generator=g, device=DEV)[:k].sort().values
    return lists[:, head_map.to(DEV).long()].to(torch.int32).contiguous()


def _lens(g, B, N):
    """Valid lengths between half and all of N; one sequence is full."""
    lens = N - torch.randint(0, N // 2 + 1, (B,), generator=g, device=DEV)
    lens[0] = N
    return lens.to(torch.int32)


def prepare(case, seed):
    c, g = dict(case), _gen(seed)
    if c["op"] == "headmap":
        a_d = torch.softmax(_randn(g, c["S"], c["Hd"], c["R"], c["N"]) * 2, dim=-1)
        planted = torch.randint(0, c["Hd"], (c["Ht"],), generator=g, device=DEV)
        a_t = torch.softmax(torch.log(a_d[:, planted]) + _randn(g, c["S"], c["Ht"], c["R"], c["N"]), dim=-1)
        return {"op": "headmap", "a_d": a_d, "a_t": a_t, "k": c["k"]}
    op, B, N, k = c["op"], c["B"], c["N"], c.get("k")
    Hq, Hkv, d, Hd = SHAPES[c["shape"]]
    Tq = 16 if op == "prefill" else c["Tq"]
    hm = _head_map(Hq, Hd)
    st = {"op": op, "hm": hm, "scale": 1.0 / math.sqrt(d)}

    if op in ("verify", "select", "paged"):
        lens = _lens(g, B, N) if c.get("ragged") else None
        st["lens"] = lens
        st["scores"] = _scores(g, B, Hd, Tq, N, bf16=c.get("bf16", False), lens=None if lens is None else lens.tolist())
        pages = c.get("page", 1)
        st["idx"] = torch.empty(B, Hq, k, device=DEV, dtype=torch.int32)
        st["cnt"] = torch.empty(B, Hq, device=DEV, dtype=torch.int32)
        st["select"] = sts.sts_select(st["scores"], hm, k, seq_lens=lens, page_size=pages, out=(st["idx"], st["cnt"]), prepare=True)
        if op == "select":
            return st
    if op == "sparse":
        st["idx"], st["cnt"] = _index_lists(g, B, Hd, N, k, hm), None

    if op == "draft":
        # the draft layer's own shape: head size 64, as many query heads as the target has draft heads
        st["q"] = _bf16(g, B, Tq, Hd, 64)
        st["k"], st["v"] = _cache(g, B, Hkv, N, 64, st["q"])
        st["scale"] = 1.0 / math.sqrt(64)
        out, lse = torch.empty_like(st["q"]), torch.empty(B, Hd, Tq, device=DEV, dtype=torch.float32)
        st["idx"] = torch.empty(B, Hq, k, device=DEV, dtype=torch.int32)
        st["cnt"] = torch.empty(B, Hq, device=DEV, dtype=torch.int32)
        if c["dump"]:
            st["scores"] = torch.empty(B, Hd, Tq, N, device=DEV, dtype=torch.bfloat16)
            st["attn"] = sts.sts_dense_attn(st["q"], st["k"], st["v"], st["scale"], out=out, lse_out=lse, logits_out=st["scores"], prepare=True)
            st["select"] = sts.sts_select(st["scores"], hm, k, lse=lse, kind=sts.STS_SCORES_LOGITS_LSE, out=(st["idx"], st["cnt"]), prepare=True)
        else:
            st["scores"] = torch.empty(B, Hd, N, device=DEV, dtype=torch.float32)
            st["attn"] = sts.sts_dense_attn(st["q"], st["k"], st["v"], st["scale"], out=out, lse_out=lse, weights_sum_out=st["scores"], prepare=True)
            st["select"] = sts.sts_select(st["scores"].view(B, Hd, 1, N), hm, k, out=(st["idx"], st["cnt"]), prepare=True)
        return st

    st["q"] = _bf16(g, B, Tq, Hq, d)
    if op == "prefill":
        # B query blocks over ONE cache; block i sees the tokens before it and adds its own causally
        st["k"], st["v"] = (x.expand(B, Hkv, N, d) for x in _cache(g, 1, Hkv, N, d, st["q"]))
        lens = (N - Tq * (B - 1 - torch.arange(B, device=DEV))).to(torch.int32)
        st["lens"], st["N"], st["budget"] = lens, N, k
        st["scores"] = _scores(g, B, Hd, Tq, N, bf16=True, lens=lens.tolist())
        st["pitch"] = min(6 * k, N)          # neighbouring rows keep much the same tokens: their union is a few lists long
        st["rows"] = (torch.empty(B, Hd, Tq, k, device=DEV, dtype=torch.int32), torch.empty(B, Hd, Tq, device=DEV, dtype=torch.int32))
        st["union"] = (torch.empty(B, Hq, st["pitch"], device=DEV, dtype=torch.int32),
                       torch.empty(B, Hq, st["pitch"], device=DEV, dtype=torch.int16), torch.empty(B, Hq, device=DEV, dtype=torch.int32))
        st["kn"], st["vn"] = (_bf16(g, B, Tq, Hkv, d, std=0.5) for _ in range(2))
        st["out"] = torch.empty_like(st["q"])
        return st

    kc, vc = _cache(g, B, Hkv, N, d, st["q"])
    st["k"], st["v"] = kc, vc
    out = torch.empty_like(st["q"])
    lse = torch.empty(B, Hq, Tq, device=DEV, dtype=torch.float32)
    if op == "dense":
        st["lens"] = _lens(g, B, N)
        st["attn"] = sts.sts_dense_attn(st["q"], kc, vc, st["scale"], seq_lens=st["lens"], out=out, lse_out=lse, prepare=True)
    elif op == "paged":
        p = c["page"]
        nblk = (N + p - 1) // p
        perm = torch.randperm(B * nblk, generator=g, device=DEV)
        pools = []
        for x in (kc, vc):      # the pages of all sequences scattered over one pool [pages,Hkv,p,d]
            padded = torch.zeros(B, Hkv, nblk * p, d, device=DEV, dtype=torch.bfloat16)
            padded[:, :, :N] = x
            pool = torch.empty(B * nblk, Hkv, p, d, device=DEV, dtype=torch.bfloat16)
            pool[perm] = padded.view(B, Hkv, nblk, p, d).permute(0, 2, 1, 3, 4).reshape(B * nblk, Hkv, p, d)
            pools.append(pool)
        st["table"] = perm.view(B, nblk).to(torch.int32).contiguous()
        st["pools"] = pools
        st["attn"] = sts.sts_sparse_attn(st["q"], pools[0], pools[1], st["idx"], st["scale"], counts=st["cnt"], head_map=hm, out=out,
                                         lse_out=lse, page_size=p, block_table=st["table"], N=N, prepare=True)
    else:
        kn = vn = None
        if c["tail"]:
            kn, vn = (_bf16(g, B, Tq, Hkv, d, std=0.5) for _ in range(2))
        st["kn"], st["vn"] = kn, vn
        st["attn"] = sts.sts_sparse_attn(st["q"], kc, vc, st["idx"], st["scale"], counts=st["cnt"], head_map=hm, out=out, lse_out=lse,
                                         k_new=kn, v_new=vn, prepare=True)
    return st


# ------------------------------------------------------------------------------------ the pass

def run(state):
    s = state
    op = s["op"]
    if op == "headmap":
        mapping, overlap = sts.sts_head_map(s["a_d"], s["a_t"], s["k"])
        return {"map": mapping, "overlap": overlap}
    if op == "prefill":
        ridx, rcnt = sts.sts_select_rows(s["scores"], s["budget"], seq_lens=s["lens"], out=s["rows"])
        uidx, umask, ucnt = sts.sts_union_rows(ridx, rcnt, s["hm"], s["N"], pitch=s["pitch"], out=s["union"])
        out, lse = sts.sts_sparse_attn(s["q"], s["k"], s["v"], uidx, s["scale"], counts=ucnt, head_map=s["hm"], out=s["out"],
                                       k_new=s["kn"], v_new=s["vn"], causal=True, row_mask=umask)
        return {"rows": ridx, "row_counts": rcnt, "union": uidx, "bits": umask, "counts": ucnt, "out": out, "lse": lse}
    if op == "select":
        idx, cnt, _ = s["select"]()
        return {"indices": idx, "counts": cnt}
    if op == "draft":
        out, lse, _ = s["attn"]()
        idx, cnt, _ = s["select"]()
        return {"out": out, "lse": lse, "scores": s["scores"], "indices": idx, "counts": cnt}
    if op in ("verify", "paged"):
        idx, cnt, _ = s["select"]()
        out, lse, _ = s["attn"]()
        return {"indices": idx, "counts": cnt, "out": out, "lse": lse}
    out, lse, _ = s["attn"]()
    return {"out": out, "lse": lse}


# ------------------------------------------------------------------------------------ cost

def work(case):
    """Each input once, each output once. Attention reads a K and a V row per entry of a list (per
    set of heads that share it), at most the whole cache."""
    c = case
    op = c["op"]
    if op == "headmap":
        rows = c["S"] * c["R"] * (c["Hd"] + c["Ht"])
        return {"bytes": 4.0 * rows * c["N"], "flops": 0.0}
    Hq, Hkv, d, Hd = SHAPES[c["shape"]]
    B, N, k = c["B"], c["N"], c.get("k", 0)
    Tq = 16 if op == "prefill" else c["Tq"]
    nbytes = flops = 0.0
    mean = 0.75 if c.get("ragged") or op == "dense" else 1.0      # mean share of the tokens that are valid
    if B == 1:
        mean = 1.0
    if op in ("verify", "select", "paged", "prefill"):
        nbytes += B * Hd * Tq * N * mean * (2 if c.get("bf16") or op == "prefill" else 4)
    if op in ("verify", "select", "paged"):
        nbytes += 4.0 * B * Hq * (k + 1)
    if op in ("verify", "sparse", "paged"):
        keys = min(k * c.get("page", 1), N)
        sets = max(Hd, Hkv)
        nbytes += min(B * sets * keys, B * Hkv * N) * 4.0 * d + 2 * 2.0 * B * Tq * Hq * d
        flops += 4.0 * B * Hq * Tq * keys * d
        if op == "sparse":
            nbytes += 4.0 * B * Hq * k
    if op == "dense":
        nbytes += B * Hkv * N * mean * 4.0 * d + 2 * 2.0 * B * Tq * Hq * d
        flops += 4.0 * B * Hq * Tq * N * mean * d
    if op == "draft":
        nbytes += B * Hkv * N * 4.0 * 64 + B * Hd * N * (2.0 * Tq if c["dump"] else 4.0) + 4.0 * B * Hq * k
        flops += 4.0 * B * Hd * Tq * N * 64
    if op == "prefill":
        # the union of a block's 16 lists is about four times a list here (neighbouring rows keep much the same tokens)
        u = min(4 * k, N)
        nbytes += 4.0 * B * Hd * Tq * k + 6.0 * B * Hq * u + 2 * 2.0 * B * Tq * Hq * d + Hkv * N * 4.0 * d
        flops += 4.0 * B * Hq * Tq * k * d
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Index sets, counts and row bits are whole numbers and stay the same. Attention outputs are
    bf16 with bf16 attention weights inside: against 64 bits they are 2e-3 to 3e-3 off (2-norm), and
    two orders of merging differ by as much."""
    if case["op"] in ("select", "headmap"):
        return "exact"
    return {"rel": 1e-2, "max": 0.1, "differ": 0.0}


# ------------------------------------------------------------------------------------ 64 bits

def _attend(q, k, v, scale, idx, kn=None, vn=None, keep=None):
    """q [T,d], k, v [N,d] (any type), idx [k] or None -> (out, lse) in 64 bits; own tokens causally;
    keep [T,k]: which entries each row sees."""
    q = q.double()
    kk, vv = (k, v) if idx is None else (k[idx], v[idx])
    s = q @ kk.double().t() * scale
    if keep is not None:
        s = s.masked_fill(~keep, float("-inf"))
    vv = vv.double()
    if kn is not None:
        T = q.shape[0]
        own = q @ kn.double().t() * scale
        own = own.masked_fill(~torch.ones(T, T, dtype=torch.bool, device=q.device).tril(), float("-inf"))
        s, vv = torch.cat([s, own], dim=1), torch.cat([vv, vn.double()])
    return torch.softmax(s, dim=-1) @ vv, torch.logsumexp(s, dim=-1)


def _top(scores, k, n):
    """Ascending positions of the k largest of scores[:n], ties to the lower position."""
    return torch.sort(scores[:n], descending=True, stable=True).indices[:k].sort().values


def _lists(scores, k, lens, page):
    """[B,Hd] lists of kept tokens: rows added in order in the scores' own 32 bits, as is defined."""
    B, Hd, Tq, N = scores.shape
    agg = scores[:, :, 0].float()
    for i in range(1, Tq):
        agg = agg + scores[:, :, i].float()
    res = []
    for b in range(B):
        n = N if lens is None else lens[b]
        for j in range(Hd):
            a = agg[b, j, :n]
            if page > 1:
                nblk = (n + page - 1) // page
                pad = torch.zeros(nblk * page, device=a.device)
                pad[:n] = a
                blk = pad.view(nblk, page)
                tot = blk[:, 0]
                for e in range(1, page):
                    tot = tot + blk[:, e]
                m = _top(tot, min(k, nblk), nblk)
                t = (m[:, None] * page + torch.arange(page, device=a.device)).reshape(-1)
                res.append(t[t < n])
            else:
                res.append(_top(a, min(k, n), n))
    return [res[b * Hd:(b + 1) * Hd] for b in range(B)]


def exact(case, seed):
    op = case["op"]
    if op in ("select", "headmap"):
        return None
    s = prepare(case, seed)
    Hq, Hkv, _, Hd = SHAPES[case["shape"]]
    B, Tq, H, d = s["q"].shape
    N = case["N"]
    hm = s["hm"].tolist()
    out = torch.empty(B, Tq, H, d, device=DEV, dtype=torch.float64)
    lse = torch.empty(B, H, Tq, device=DEV, dtype=torch.float64)
    G = H // Hkv
    if op == "draft":
        sums = None if case["dump"] else torch.empty(B, Hd, N, device=DEV, dtype=torch.float64)
        logits = torch.empty(B, Hd, Tq, N, device=DEV, dtype=torch.float64) if case["dump"] else None
        for b in range(B):
            for t in range(H):
                sc = s["q"][b, :, t].double() @ s["k"][b, t // G].double().t() * s["scale"]
                lse[b, t] = torch.logsumexp(sc, dim=-1)
                p = torch.exp(sc - lse[b, t][:, None])
                out[b, :, t] = p @ s["v"][b, t // G].double()
                if case["dump"]:
                    logits[b, t] = sc
                else:
                    sums[b, t] = p.sum(dim=0)
        return {"out": out, "lse": lse, "scores": logits if case["dump"] else sums, "indices": None, "counts": None}
    if op == "prefill":
        k = case["k"]
        lens = s["lens"].tolist()
        if B * Hd * N > 16 * 16 * 70000:
            return None
        for b in range(B):
            for j in range(Hd):
                rows = [_top(s["scores"][b, j, i].float(), min(k, lens[b]), lens[b]) for i in range(Tq)]
                uni = torch.unique(torch.cat(rows))
                keep = torch.stack([torch.isin(uni, r) for r in rows])
                for t in range(H):
                    if hm[t] == j:
                        h = t // G
                        out[b, :, t], lse[b, t] = _attend(s["q"][b, :, t], s["k"][b, h], s["v"][b, h], s["scale"], uni,
                                                          s["kn"][b, :, h], s["vn"][b, :, h], keep)
        return {"rows": None, "row_counts": None, "union": None, "bits": None, "counts": None, "out": out, "lse": lse}
    if op in ("verify", "paged"):
        lists = _lists(s["scores"], case["k"], None, case.get("page", 1))
    kn, vn = s.get("kn"), s.get("vn")
    for b in range(B):
        for t in range(H):
            h = t // G
            kk, vv = s["k"][b, h], s["v"][b, h]
            if op == "dense":
                n = int(s["lens"][b])
                kk, vv, idx = kk[:n], vv[:n], None
            else:
                idx = s["idx"][b, t].long() if op == "sparse" else lists[b][hm[t]]
            out[b, :, t], lse[b, t] = _attend(s["q"][b, :, t], kk, vv, s["scale"], idx,
                                              None if kn is None else kn[b, :, h], None if vn is None else vn[b, :, h])
    res = {"out": out, "lse": lse}
    if op in ("verify", "paged"):
        res.update(indices=None, counts=None)
    return res
