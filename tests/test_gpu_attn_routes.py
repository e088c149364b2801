"""GPU parity of the attention kernels' routes that depend on strides, sizes and the scale: batch
elements over one shared cache, heads of more than 4 GB, more batch elements than a grid's last
dimension, head sets with gaps, scales of any sign, and running maxima that grow within a list.
All against the CPU oracle, with the tolerances of the other attention tests."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2605_15508_amd as sts
from gpu_util import bits, check_attn, check_logits, oracle_attn
from test_gpu_attn import DEV, make_indices, make_qkv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Tq,Hq,Hkv,d,N,kk,shared", [
    (2, 16, 4, 2, 128, 700, 31, 1),       # one query tile, less than a key tile
    (3, 5, 8, 2, 128, 2000, 513, 2),      # one tile more than a list that is not split
    (3, 16, 4, 2, 128, 3000, 1, 2),       # two query tiles (eight waves): a single key, seven waves without tiles
    (2, 16, 8, 2, 128, 3000, 255, 2),     # eight waves, one tile each, the last one short
    (5, 13, 8, 4, 128, 9000, 2049, 2),    # an odd number of workgroups; lists that are split; padding rows
    (2, 9, 8, 1, 128, 1500, 300, 8),      # more than 64 rows in a head set: several units
    (2, 16, 8, 2, 128, 1500, 300, 4),     # four query tiles
    (3, 8, 8, 2, 64, 1500, 333, 4),       # head size 64
])
@pytest.mark.parametrize("row_bits", [False, True])
def test_blocks_over_one_shared_cache(B, Tq, Hq, Hkv, d, N, kk, shared, row_bits):
    q, k, v = make_qkv(Tq + N, 1, B * Tq, Hq, Hkv, d, N)
    q = q.view(B, Tq, Hq, d).contiguous()
    ke, ve = (x.expand(B, -1, -1, -1) for x in (k, v))
    hm = [t // shared for t in range(Hq)]
    idx = make_indices(kk, B, Hq, N, kk, hm)
    rng = np.random.default_rng(kk)
    cnt_d = rng.integers(1, kk + 1, size=(B, Hq // shared)).astype(np.int32)
    cnt_d[0] = kk
    cnt_d[-1, -1] = 0                     # an empty list
    cnt = torch.from_numpy(np.repeat(cnt_d, shared, axis=1)).to(DEV)
    scale = 1.0 / math.sqrt(d)
    if not row_bits:
        out, lse = sts.sts_sparse_attn(q, ke, ve, idx, scale, counts=cnt, head_map=hm, out_dtype=torch.float32)
        ref = oracle_attn(q, ke.contiguous(), ve.contiguous(), scale, idx, cnt)
        check_attn(out, lse, ref, what="shared cache")
        return
    mask_d = rng.integers(0, 1 << Tq, size=(B, Hq // shared, kk), dtype=np.int64).astype(np.uint16)
    mask = torch.from_numpy(np.repeat(mask_d, shared, axis=1).view(np.int16)).to(DEV)
    out, lse = sts.sts_sparse_attn(q, ke, ve, idx, scale, counts=cnt, head_map=hm, row_mask=mask, out_dtype=torch.float32)
    rows = np.full((B, Hq, Tq, kk), -1, np.int32)
    rcnt = np.zeros((B, Hq, Tq), np.int32)
    ih, ch, mh = idx.cpu().numpy(), cnt.cpu().numpy(), mask.cpu().numpy().view(np.uint16)
    for b in range(B):
        for t in range(Hq):
            for i in range(Tq):
                mine = ih[b, t, :ch[b, t]][(mh[b, t, :ch[b, t]] >> i) & 1 == 1]
                rows[b, t, i, :len(mine)] = mine
                rcnt[b, t, i] = len(mine)
    ref = oracle.attn_rows(bits(q), bits(ke.contiguous()), bits(ve.contiguous()), scale, rows, rcnt)
    check_attn(out, lse, ref, what="shared cache, row bits")


# eight waves: two query tiles at head size 128, more than eight key tiles a workgroup
@pytest.mark.parametrize("B,Tq,Hq,Hkv,N,kk,shared", [
    (3, 16, 4, 2, 3000, 289, 2),          # ten key tiles, the last one a single key
    (2, 16, 8, 2, 1500, 500, 2),          # sixteen
    (32, 13, 8, 4, 2500, 1033, 2),        # lists in two parts; padding rows
])
@pytest.mark.parametrize("row_bits", [False, True])
def test_blocks_over_one_shared_cache_by_eight_waves(B, Tq, Hq, Hkv, N, kk, shared, row_bits):
    test_blocks_over_one_shared_cache(B, Tq, Hq, Hkv, 128, N, kk, shared, row_bits)


@pytest.mark.parametrize("scale", [-0.11, 0.0, 0.3])
@pytest.mark.parametrize("Tq,d", [(3, 128), (5, 64), (16, 128)])
def test_scales_of_any_sign(scale, Tq, d):
    q, k, v = make_qkv(7, 2, Tq, 4, 2, d, 333)
    out, lse, lg = sts.sts_dense_attn(q, k, v, scale, out_dtype=torch.float32, want_logits=True)
    ref = oracle_attn(q, k, v, scale, want_logits=True)
    check_attn(out, lse, ref, what="dense")
    check_logits(lg.cpu().numpy(), ref["logits"], what="dense")
    idx = make_indices(5, 2, 4, 333, 77, [0, 0, 1, 1])
    out, lse = sts.sts_sparse_attn(q, k, v, idx, scale, head_map=[0, 0, 1, 1], out_dtype=torch.float32)
    check_attn(out, lse, oracle_attn(q, k, v, scale, idx), what="sparse")


@pytest.mark.parametrize("step", [0.5, 3.0, 40.0])
def test_running_maxima_that_grow_along_the_list(step):
    """Logits (log2) that rise by `step` per key tile, so that the accumulators are rescaled in every
    tile of the first half, and fall again in the second, where they are not."""
    N, d = 1500, 128
    g = torch.Generator().manual_seed(3)
    q = torch.zeros(1, 2, 2, d)
    q[..., 0] = 1.0
    k = torch.randn(1, 1, N, d, generator=g) * 0.1
    up = torch.arange(N) // 32
    k[0, 0, :, 0] = torch.minimum(up, N // 32 - up).float() * step * math.log(2.0)
    v = torch.randn(1, 1, N, d, generator=g)
    q, k, v = (x.to(torch.bfloat16).to(DEV) for x in (q, k, v))
    out, lse, _ = sts.sts_dense_attn(q, k, v, 1.0, out_dtype=torch.float32)
    check_attn(out, lse, oracle_attn(q, k, v, 1.0), what="dense")
    idx = make_indices(1, 1, 2, N, 1400, [0, 0])
    out, lse = sts.sts_sparse_attn(q, k, v, idx, 1.0, head_map=[0, 0], out_dtype=torch.float32)
    check_attn(out, lse, oracle_attn(q, k, v, 1.0, idx), what="sparse")


@pytest.mark.parametrize("hm", [[0, 1, 0, 1, 2, 2, 3, 2], [0, 0, 1, 0, 1, 1, 0, 1]])
def test_head_sets_with_gaps(hm):
    q, k, v = make_qkv(2, 2, 5, 8, 2, 128, 900)
    idx = make_indices(9, 2, 8, 900, 130, hm)
    out, lse = sts.sts_sparse_attn(q, k, v, idx, 0.09, head_map=hm, out_dtype=torch.float32)
    check_attn(out, lse, oracle_attn(q, k, v, 0.09, idx), what="gaps")


def test_heads_of_more_than_4_gb():
    """An interleaved cache whose heads span 4.4 GB: rows at 64-bit offsets, on either side of the
    4 GB mark, with and without row bits (all set: the same result bit for bit)."""
    N, H, d, Tq = 1_080_000, 8, 128, 4
    base = torch.zeros(1, N, 2, H, d, dtype=torch.bfloat16, device=DEV)
    g = torch.Generator().manual_seed(1)
    pos = torch.unique(torch.cat([torch.randint(0, N, (500,), generator=g), torch.tensor([0, 1048575, 1048576, 1048577, N - 1])]))
    rows = torch.randn(1, len(pos), 2, H, d, generator=g).to(torch.bfloat16)
    base[:, pos.to(DEV)] = rows.to(DEV)
    k, v = base[:, :, 0].permute(0, 2, 1, 3), base[:, :, 1].permute(0, 2, 1, 3)
    q = torch.randn(1, Tq, 2 * H, d, generator=g).to(torch.bfloat16).to(DEV)
    hm = [t // 2 for t in range(2 * H)]
    idx = pos.to(torch.int32).expand(1, 2 * H, -1).contiguous().to(DEV)
    out, lse = sts.sts_sparse_attn(q, k, v, idx, 0.09, head_map=hm, out_dtype=torch.float32)
    small = [rows[:, :, i].permute(0, 2, 1, 3).contiguous() for i in range(2)]
    own = torch.arange(len(pos), dtype=torch.int32).expand(1, 2 * H, -1).contiguous()
    check_attn(out, lse, oracle_attn(q, small[0], small[1], 0.09, own), what="far rows")
    full = torch.full(idx.shape, -1, dtype=torch.int16, device=DEV)
    out2, lse2 = sts.sts_sparse_attn(q, k, v, idx, 0.09, head_map=hm, row_mask=full, out_dtype=torch.float32)
    assert torch.equal(out, out2) and torch.equal(lse, lse2)


def test_more_batch_elements_than_a_grid_dimension():
    B, N, d = 70000, 40, 64
    q, k, v = make_qkv(4, 1, 1, 1, 1, d, N)
    g = torch.Generator().manual_seed(5)
    q = torch.randn(B, 1, 1, d, generator=g).to(torch.bfloat16).to(DEV)
    idx = torch.stack([torch.randperm(N, generator=g)[:5].sort().values for _ in range(64)]).to(torch.int32)
    idx = idx.repeat(B // 64 + 1, 1)[:B].view(B, 1, 5).contiguous().to(DEV)
    ke, ve = (x.expand(B, -1, -1, -1) for x in (k, v))
    out, lse = sts.sts_sparse_attn(q, ke, ve, idx, 0.125, out_dtype=torch.float32)
    sel = [0, 1, 32767, 32768, 65535, 65536, B - 1]
    ref = oracle_attn(q[sel], ke[sel].contiguous(), ve[sel].contiguous(), 0.125, idx[sel])
    check_attn(out[sel], lse[sel], ref, what="many batch elements")
    out2, lse2, _ = sts.sts_dense_attn(q, ke, ve, 0.125, out_dtype=torch.float32)
    ref2 = oracle_attn(q[sel], ke[sel].contiguous(), ve[sel].contiguous(), 0.125)
    check_attn(out2[sel], lse2[sel], ref2, what="many batch elements, dense")
