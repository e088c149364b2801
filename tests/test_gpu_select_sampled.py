"""The sampled selection (csrc/select_sampled.hip) where it can go wrong: row lengths that are no multiple
of a quad, a group or a part, scores at any alignment, rows whose sample misleads or whose band is
one key, and rows cut into more than eight parts. Bit for bit against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_15508_amd as sts
from gpu_util import stored_agg
from test_select_emulated import between_samples

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def make(what, B, Hd, Tq, N, seed):
    g = torch.Generator().manual_seed(seed)
    s = torch.softmax(torch.randn(B, Hd, Tq, N, generator=g) * 2, dim=-1)
    if what == "zeros":                       # the threshold is one value that most tokens share
        return s * (torch.rand(B, Hd, 1, N, generator=g) < 0.05)
    if what == "constant":
        return torch.full((B, Hd, Tq, N), 0.25)
    if what == "levels":                      # two neighbouring levels can fill the band: bitmaps hold them
        return torch.randint(0, 5, (B, Hd, 1, N), generator=g).float().expand(B, Hd, Tq, N).contiguous() / 8
    if what == "signed":                      # negative scores, -0 and +0
        s = torch.randn(B, Hd, Tq, N, generator=g)
        s[..., ::7] = 0.0
        s[..., 3::14] = -0.0
        return s
    if what == "stretch":                     # all heavy tokens next to each other
        s[..., N // 3:N // 3 + N // 8] += 1e-3
        return s
    if what == "passages":                    # heavy passages of 200 tokens
        m = (torch.rand(B, Hd, 1, N // 200 + 1, generator=g) < 0.1).float().repeat_interleave(200, -1)[..., :N]
        return s * (1 + 20 * m)
    if what == "recent":                      # the last tokens are heavy
        s[..., -N // 20:] *= 50
        return s
    if what == "edge":
        return s * (torch.rand(B, Hd, 1, N, generator=g) < 0.1)
    if what == "inf":                         # infinite scores are kept before all others
        s[..., N // 2::1000] = float("inf")
        return s
    return s


@pytest.mark.parametrize("B,Hd,Tq,N,k,bf16,what", [
    (2, 3, 5, 8193, 819, False, "softmax"),          # one token past the shortest row; two parts
    (2, 3, 5, 33001, 3301, False, "softmax"),
    (1, 2, 1, 65537, 6554, True, "softmax"),         # bf16 rows at any even address, ties at the threshold
    (1, 2, 9, 100003, 700, False, "softmax"),        # more score rows than are in flight
    (2, 2, 3, 8447, 8447, False, "softmax"),         # everything kept, a group that ends one token short
    (2, 2, 2, 40961, 1, False, "softmax"),
    (2, 2, 2, 40002, 9000, False, "zeros"),
    (2, 2, 2, 40002, 9000, True, "constant"),
    (2, 2, 2, 40002, 9000, False, "levels"),
    (2, 2, 1, 40002, 30000, False, "signed"),        # the threshold among the negative scores
    (2, 2, 3, 70001, 7000, False, "stretch"),
    (2, 2, 3, 70001, 7000, False, "passages"),
    (2, 2, 2, 40002, 100, False, "inf"),
    (1, 16, 1, 262147, 9000, True, "softmax"),       # more than eight parts per row
    (3, 48, 1, 33000, 1500, False, "softmax"),       # one part per row: 144 rows
    (1, 128, 2, 16500, 800, True, "softmax"),        # two parts per row, a row for every second CU
    (1, 130, 1, 131072, 65536, True, "softmax"),     # one part of more than 64K tokens: the larger sample
    (1, 130, 1, 100004, 9000, False, "softmax"),     # ... and a small budget there
    (1, 130, 1, 200001, 9000, True, "softmax"),      # one part of more than 128K tokens
    (1, 130, 1, 300003, 3000, False, "recent"),      # ... of more than 256K
    (1, 64, 1, 262144, 45000, False, "stretch"),     # a band that lies in one of four parts and overflows its list
    (1, 2, 2, 70001, 7000, False, "edge"),           # zeros from about the budget on
])
def test_sampled_selection(B, Hd, Tq, N, k, bf16, what):
    scores = make(what, B, Hd, Tq, N, N + k)
    scores = scores.to(torch.bfloat16) if bf16 else scores
    off = 1 if N % 2 else 0                          # an odd row length also starts at an odd element
    flat = torch.zeros(scores.numel() + 8, dtype=scores.dtype, device=DEV)
    sd = flat[off:off + scores.numel()].view(B, Hd, Tq, N)
    sd.copy_(scores)
    hm = [t // 2 for t in range(Hd)] + [Hd - 1]      # pairs share a draft head, the upper half but one is unread
    kh = [max(1, k - 5 * j) for j in range(Hd)]
    lens = torch.tensor([N, N - 13, N // 3][:B], dtype=torch.int32)
    idx, cnt, agg = sts.sts_select(sd, hm, k, seq_lens=lens.to(DEV), k_head=kh, want_agg=True)
    idx2, cnt2, _ = sts.sts_select(sd, hm, k, seq_lens=lens.to(DEV), k_head=kh)
    torch.cuda.synchronize()
    o_idx, o_cnt, o_agg = oracle.select_indices(scores.float().numpy(), np.asarray(hm, np.int32), k, k_head=kh, seq_lens=lens.numpy())
    np.testing.assert_array_equal(cnt.cpu().numpy(), o_cnt)
    np.testing.assert_array_equal(idx.cpu().numpy(), o_idx)
    np.testing.assert_array_equal(agg.cpu().numpy().view(np.uint32), stored_agg(o_agg, lens).view(np.uint32))
    assert torch.equal(idx2, idx) and torch.equal(cnt2, cnt)


def test_sampled_selection_without_the_other_parts():
    """A poll limit of 0: workgroups that do not find the other parts' words rank the row themselves."""
    scores = make("softmax", 1, 4, 2, 50001, 3)
    sts.set_knob("select_spin_limit", 0)
    try:
        idx, cnt, _ = sts.sts_select(scores.to(DEV), [0, 1, 2, 3], 5000)
        torch.cuda.synchronize()
    finally:
        sts.set_knob("select_spin_limit", None)
    o_idx, o_cnt, _ = oracle.select_indices(scores.numpy(), np.arange(4, dtype=np.int32), 5000)
    np.testing.assert_array_equal(idx.cpu().numpy(), o_idx)
    np.testing.assert_array_equal(cnt.cpu().numpy(), o_cnt)


@pytest.mark.parametrize("N,k,path", [(40002, 50, 0), (131072, 50, 0), (131072, 50, 5)])      # several parts; one part per row
def test_equal_scores_above_all_that_the_sample_saw(N, k, path):
    """More equal scores than are ranked one by one, far above the rest, where no sampled run lies."""
    s = make("softmax", 1, 2, 1, N, N) * 1e-20
    at, _ = between_samples(N)
    s[..., at:at + 250] = 3.0
    s[..., at + 250:at + 290] = torch.linspace(1.0, 2.0, 40)
    sts.set_knob("select_path", path)
    try:
        for budget in (k, 270):
            idx, cnt, _ = sts.sts_select(s.to(DEV), [0, 1, 1], budget)
            torch.cuda.synchronize()
            o_idx, o_cnt, _ = oracle.select_indices(s.numpy(), np.asarray([0, 1, 1], np.int32), budget)
            np.testing.assert_array_equal(idx.cpu().numpy(), o_idx)
            np.testing.assert_array_equal(cnt.cpu().numpy(), o_cnt)
    finally:
        sts.set_knob("select_path", None)


@pytest.mark.parametrize("N,n,step", [(131907, 34394, 4), (131072, 131072, 8), (400003, 390000, 8), (262144, 200001, 16)])
def test_scores_of_a_few_levels(N, n, step):
    """Rows of a few levels of very different weight, one part per row: one level or two at the edges of the band that much
    of the row shares, others between them."""
    B = 128
    s = torch.zeros(B, 1, 1, N, device=DEV)
    lens = torch.zeros(B, dtype=torch.int32)
    live = [0, 5]
    for b in live:
        s[b, 0, 0, :n] = torch.round(torch.randn(n, generator=torch.Generator().manual_seed(7 + b)) * step / 2).to(DEV) / step
        lens[b] = n
    for share in (0.03, 0.2, 0.4, 0.6, 0.75, 0.835, 0.9, 0.97):
        k = int(n * share)
        idx, cnt, _ = sts.sts_select(s, [0], max(k, int(0.4 * N)), k_head=[k], seq_lens=lens.to(DEV))
        for b in live:
            assert cnt[b, 0] == k
            want = torch.sort(s[b, 0, 0, :n] + 0.0, descending=True, stable=True).indices[:k].sort().values
            assert torch.equal(idx[b, 0, :k].long(), want), (b, share)


@pytest.mark.parametrize("budget", [36294, 35931])
def test_bins_that_run_past_the_band(budget):
    """A band that begins at the lowest key, overflows the list and ends inside the threshold's bin."""
    N, rows = 36294, 130
    g = torch.Generator().manual_seed(35)
    base = float(0.5 + torch.rand(1, generator=g) * 0.4)
    row = base * torch.exp(torch.softmax(2 * torch.randn(N, generator=g), -1).to(torch.bfloat16).float())
    s = torch.zeros(rows, 1, 1, N, device=DEV)
    s[0, 0, 0] = row.to(DEV)
    lens = torch.zeros(rows, dtype=torch.int32, device=DEV)
    lens[0] = N
    idx, cnt, _ = sts.sts_select(s, [0], N, k_head=[budget], seq_lens=lens)
    want = torch.sort(row, descending=True, stable=True).indices[:budget].sort().values
    assert cnt[0, 0] == budget and torch.equal(idx[0, 0, :budget].cpu().long(), want)
