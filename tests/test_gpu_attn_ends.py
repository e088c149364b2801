"""What lies past the end of a list, a sequence or a page is not attended to and does not reach the result, whatever it
holds: index entries from a list's count on, the page table's entries and the rows of the last page from a sequence's
length on. Rows of NaN there, in K and in V, against the same call without any: the same result bit for bit."""
import math

import numpy as np
import pytest
import torch

import paper_2605_15508_amd as sts
from test_gpu_attn import DEV, make_indices, make_qkv

pytestmark = pytest.mark.gpu
NAN = float("nan")


def same(make):
    """make(row): the call with that value in the rows that are nobody's."""
    out, lse = make(0.0)[:2]
    assert torch.isfinite(out).all()
    for x in (NAN, float("inf")):
        bad, bad_lse = make(x)[:2]
        assert torch.equal(out, bad) and torch.equal(lse, bad_lse)


SHAPES = [
    (5, 8, 2, 128, 3000, 700, 2),         # one query tile; several tiles per wave, split
    (3, 4, 2, 128, 2000, 257, 2),         # ... and not split
    (16, 8, 2, 128, 3000, 1500, 2),       # two query tiles
    (16, 8, 2, 128, 3000, 450, 2),        # ... which eight waves share
    (16, 8, 2, 128, 3000, 900, 4),        # four
    (8, 8, 2, 64, 3000, 900, 4),
]


@pytest.mark.parametrize("form,shape", [(f, s) for f in ("own caches", "row bits", "shared cache", "shared cache, row bits") for s in SHAPES]
                         + [("heads of 4 GB", SHAPES[0])])
def test_entries_past_a_lists_count(form, shape):
    Tq, Hq, Hkv, d, N, kk, sets = shape
    B = 4
    shared = "shared" in form
    q, k, v = make_qkv(kk, 1 if shared else B, Tq if not shared else B * Tq, Hq, Hkv, d, N)
    q = q.view(B, Tq, Hq, d)
    hm = [t // sets for t in range(Hq)]
    idx = make_indices(N, B, Hq, N - 50, kk, hm)
    cnt = torch.tensor([kk, kk - 1, 33, 0], dtype=torch.int32).view(B, 1).repeat(1, Hq)
    cnt[0, sets:] = kk // 2 + 3
    cnt[2, sets:] = 1
    past = torch.arange(kk).view(1, 1, kk) >= cnt[:, :, None]
    idx = torch.where(past.to(DEV), N - 1 - torch.arange(kk, device=DEV, dtype=torch.int32) % 50, idx)
    kw = {}
    if "bits" in form:
        kw["row_mask"] = torch.randint(-30000, 30000, (B, Hq // sets, kk), generator=torch.Generator().manual_seed(1), dtype=torch.int16).repeat_interleave(
            sets, dim=1).to(DEV)

    def make(x):
        kx, vx = k.clone(), v.clone()
        kx[:, :, N - 50:], vx[:, :, N - 50:] = x, x
        if shared:
            kx, vx = (y.expand(B, -1, -1, -1) for y in (kx, vx))
        if form == "heads of 4 GB":       # the stride alone: one head's rows span more than 32-bit offsets reach
            pitch = (1 << 31) // (N - 4) // 64 * 64 + 64
            base = torch.empty(N * pitch, dtype=torch.bfloat16, device=DEV)
            places = []
            for i, y in enumerate((kx, vx)):
                at = base.as_strided((B, Hkv, N, d), (Hkv * 2 * d, 2 * d, pitch, 1), i * d)
                at.copy_(y)
                places.append(at)
            kx, vx = places
        return sts.sts_sparse_attn(q, kx, vx, idx, 1 / math.sqrt(d), counts=cnt.to(DEV), head_map=hm, out_dtype=torch.float32, **kw)

    same(make)


@pytest.mark.parametrize("page", [2, 8, 32])
@pytest.mark.parametrize("Tq,d,N", [(5, 128, 2000), (16, 128, 1201), (3, 64, 999)])
@pytest.mark.parametrize("logits", [False, True])
def test_pages_past_a_sequences_length(page, Tq, d, N, logits):
    B, Hq, Hkv = 3, 8, 2
    q, _, _ = make_qkv(N, B, Tq, Hq, Hkv, d, 8)
    nblk = -(-N // page)
    P = B * nblk + 2
    g = torch.Generator().manual_seed(page)
    pools = [(torch.randn(P, Hkv, page, d, generator=g) * 0.5).to(torch.bfloat16).to(DEV) for _ in range(2)]
    table = torch.randperm(P, generator=g)[:B * nblk].view(B, nblk).to(torch.int32)
    lens = [N, N // 2 + 1, 3 * page + 1]

    def make(x):
        pk, pv = pools[0].clone(), pools[1].clone()
        for b, n in enumerate(lens):
            used = -(-n // page)
            for y in (pk, pv):
                y[table[b, used:].long()] = x                                    # nobody's pages
                y[int(table[b, used - 1]), :, n - (used - 1) * page:] = x        # the last page's rows that are not filled yet
        return sts.sts_dense_attn(q, pk, pv, 1 / math.sqrt(d), seq_lens=torch.tensor(lens, dtype=torch.int32, device=DEV), page_size=page,
                                  block_table=table.to(DEV), N=N, out_dtype=torch.float32, want_logits=logits)

    same(make)


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("page,N,kb", [(8, 1003, 90), (32, 2017, 40), (2, 777, 300)])
def test_blocks_that_the_caches_end_cuts(page, N, kb, paged):
    """Lists of blocks whose last one is cut, and whose entries past the count name rows of NaN."""
    B, Tq, Hq, Hkv, d = 2, 5, 8, 2, 128
    nblk = -(-N // page)
    q, _, _ = make_qkv(page, B, Tq, Hq, Hkv, d, 8)
    g = torch.Generator().manual_seed(N)
    kc, vc = ((torch.randn(B, Hkv, nblk * page, d, generator=g) * 0.5).to(torch.bfloat16) for _ in range(2))
    rng = np.random.default_rng(kb)
    idx = torch.zeros(B, Hq, kb, dtype=torch.int32)
    cnt = torch.zeros(B, Hq, dtype=torch.int32)
    for b in range(B):
        mine = np.sort(np.append(rng.choice(nblk - 4, kb - 7 - b, replace=False), nblk - 1))
        idx[b, :, :len(mine)] = torch.from_numpy(mine.astype(np.int32))
        idx[b, :, len(mine):] = nblk - 2
        cnt[b] = len(mine)
    table = torch.randperm(B * nblk, generator=g).view(B, nblk).to(torch.int32)

    def make(x):
        kx, vx = kc.clone(), vc.clone()
        for y in (kx, vx):
            y[:, :, N:] = x
            y[:, :, (nblk - 2) * page:(nblk - 1) * page] = x
        kw = dict(counts=cnt.to(DEV), head_map=[0] * 4 + [1] * 4, page_size=page, out_dtype=torch.float32)
        if not paged:
            return sts.sts_sparse_attn(q, kx.to(DEV)[:, :, :N], vx.to(DEV)[:, :, :N], idx.to(DEV), 0.09, **kw)
        pools = []
        for y in (kx, vx):
            pool = torch.zeros(B * nblk, Hkv, page, d, dtype=torch.bfloat16)
            pool[table.view(-1).long()] = y.view(B, Hkv, nblk, page, d).permute(0, 2, 1, 3, 4).reshape(B * nblk, Hkv, page, d)
            pools.append(pool.to(DEV))
        return sts.sts_sparse_attn(q, pools[0], pools[1], idx.to(DEV), 0.09, block_table=table.to(DEV), N=N, **kw)

    same(make)
