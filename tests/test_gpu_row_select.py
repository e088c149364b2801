"""Short rows ranked in one workgroup's registers (csrc/select_row.hip) and the overlap counts of the head
mapping (csrc/headmap.hip) at the edges of their tiles, against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_15508_amd as sts
from gpu_util import stored_agg
from test_gpu_select_sampled import make

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("B,Hd,Tq,N,k,bf16,what", [
    (2, 3, 5, 4, 2, False, "softmax"),               # one quad
    (2, 3, 2, 5, 9, True, "softmax"),                # k > N, an odd row length
    (1, 2, 9, 4095, 400, False, "softmax"),          # 1024 threads, one quad each
    (1, 2, 3, 8191, 8000, False, "signed"),          # two quads each, the threshold among the negative scores
    (1, 3, 2, 8192, 700, True, "constant"),
    (9, 64, 2, 4090, 300, False, "softmax"),         # many rows: 256 threads, four quads each
    (9, 64, 1, 8189, 512, False, "softmax"),         # ... eight quads, a sixteenth of the keys sampled
    (9, 64, 1, 6000, 5000, True, "softmax"),         # ... a budget whose band cannot fit: all keys counted
    (4, 64, 1, 16384, 512, False, "softmax"),        # 256 rows: 1024 threads, four quads each
    (9, 64, 1, 16384, 512, False, "softmax"),        # more rows: 256 threads, sixteen quads
    (9, 64, 1, 30001, 900, True, "softmax"),         # ... 512 threads
    (4, 64, 1, 12345, 512, False, "zeros"),          # the sample's band is one value that most tokens share
    (4, 64, 2, 16001, 800, True, "passages"),
    (4, 64, 1, 32768, 1000, False, "stretch"),       # 1024 threads, eight quads
    (4, 64, 3, 20002, 300, False, "levels"),
])
def test_rows_in_registers(B, Hd, Tq, N, k, bf16, what):
    scores = make(what, B, Hd, Tq, N, N + k)
    scores = scores.to(torch.bfloat16) if bf16 else scores
    flat = torch.zeros(scores.numel() + 8, dtype=scores.dtype, device=DEV)
    off = 1 if N % 2 else 0                          # an odd row length also starts at an odd element
    sd = flat[off:off + scores.numel()].view(B, Hd, Tq, N)
    sd.copy_(scores)
    hm = [t // 2 for t in range(Hd)] + [Hd - 1]
    kh = [max(1, k - j) for j in range(Hd)]
    lens = torch.full((B,), N, dtype=torch.int32)
    lens[-1] = max(1, N - 3)
    if B > 2:
        lens[1], lens[2] = N // 5, 0
    idx, cnt, agg = sts.sts_select(sd, hm, k, seq_lens=lens.to(DEV), k_head=kh, want_agg=True)
    idx2, _, _ = sts.sts_select(sd, hm, k, seq_lens=lens.to(DEV), k_head=kh)
    torch.cuda.synchronize()
    o_idx, o_cnt, o_agg = oracle.select_indices(scores.float().numpy(), np.asarray(hm, np.int32), k, k_head=kh, seq_lens=lens.numpy())
    np.testing.assert_array_equal(cnt.cpu().numpy(), o_cnt)
    np.testing.assert_array_equal(idx.cpu().numpy(), o_idx)
    np.testing.assert_array_equal(agg.cpu().numpy().view(np.uint32), stored_agg(o_agg, lens).view(np.uint32))
    assert torch.equal(idx2, idx)


@pytest.mark.parametrize("S,Hd,Ht,R,N,k", [
    (1, 33, 17, 2, 700, 65),                         # two groups of draft heads, more target heads than waves
    (2, 3, 2, 2, 40000, 300),                        # tokens in two chunks
    (1, 2, 3, 2, 32768, 257),                        # a chunk to the last token
])
def test_overlap_counts(S, Hd, Ht, R, N, k):
    rng = np.random.default_rng(N + k)
    a_d = rng.random((S, Hd, R, N), dtype=np.float32)
    a_t = rng.random((S, Ht, R, N), dtype=np.float32)
    mp, ov = sts.sts_head_map(torch.from_numpy(a_d).to(DEV), torch.from_numpy(a_t).to(DEV), k)
    torch.cuda.synchronize()
    o_mp, o_ov = oracle.head_mapping(a_d, a_t, k)
    np.testing.assert_array_equal(ov.cpu().numpy(), o_ov)
    np.testing.assert_array_equal(mp.cpu().numpy(), o_mp)
