"""Rows ranked in one workgroup's registers by a window of keys from a sample (select_row_kernel in
csrc/select_row.hip), and rows of block sums ranked by the same kernels, against the CPU oracle bit for
bit: scores that the sample, the windows and the slots beside them do not expect, at the edges of the
kernel's forms."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2605_15508_amd as sts
from paper_2605_15508_amd import binding
from test_select_emulated import by_keys, check, lib, route  # noqa: F401  (lib: the emulated library, a fixture)

DEV = "cuda:0"


def scores_of(what, rows, Tq, N, k, seed):
    g = torch.Generator().manual_seed(seed)
    r = torch.randn(rows, 1, Tq, N, generator=g)
    p = torch.softmax(r * 2, dim=-1)
    some = torch.rand(rows, 1, 1, N, generator=g).expand(rows, 1, Tq, N)
    if what == "softmax":
        return p
    if what == "zeros":                               # about as many scores as are kept, zeros otherwise
        return p * (some < k / N)
    if what == "zeros then scores":                   # exactly as many: the lowest one lies alone above the gap
        p[..., :N - k] = 0
        return p
    if what == "zeros then denormals":                # ... below where the window begins
        p[..., :N - k] = 0
        return p * 1e-41
    if what == "one value":
        return torch.full((rows, 1, Tq, N), 0.375)
    if what == "close together":                      # all keys share their upper 11 bits, some the next 11
        return 1 + r * 1e-6
    if what == "signed":
        r[some < 0.4] = 0.0
        r[some < 0.2] = -0.0
        return r
    if what == "levels":
        return torch.round(r * 2) / 8
    return torch.exp(r * 30)                          # "all over the range"


# (rows, scores per token, N, k): 1024 threads with four and eight quads each; 256 threads with eight and sixteen; 512
FORMS = [(256, 1, 8193, 800), (257, 2, 16384, 1638), (256, 1, 32767, 300), (513, 1, 4097, 409), (520, 1, 8192, 8000), (513, 1, 16383, 512),
         (513, 1, 32768, 3277)]


@pytest.mark.gpu
@pytest.mark.parametrize("what", ["softmax", "zeros", "zeros then scores", "zeros then denormals", "one value", "close together", "signed",
                                  "levels", "all over the range"])
@pytest.mark.parametrize("rows,Tq,N,k", FORMS)
def test_windows(rows, Tq, N, k, what):
    live = 6                                          # the other rows are empty
    s = scores_of(what, live, Tq, N, k, N + k)
    sd = torch.zeros(rows, 1, Tq, N, device=DEV)
    sd[:live] = s.to(DEV)
    lens = torch.zeros(rows, dtype=torch.int32)
    lens[:live] = torch.tensor([N, N - 3, N // 2, 1023, 1024, 5])
    idx, cnt, _ = sts.sts_select(sd, [0, 0], k, seq_lens=lens.to(DEV))
    assert (cnt[live:] == 0).all() and (idx[live:] == -1).all()
    o_idx, o_cnt, _ = oracle.select_indices(s.numpy(), np.zeros(2, np.int32), k, seq_lens=lens[:live].numpy())
    np.testing.assert_array_equal(cnt[:live].cpu().numpy(), o_cnt)
    np.testing.assert_array_equal(idx[:live].cpu().numpy(), o_idx)


@pytest.mark.parametrize("what", ["zeros", "zeros then denormals", "close together", "signed"])
@pytest.mark.parametrize("rows,Tq,N,k", [FORMS[0], FORMS[3], FORMS[5]])
def test_windows_emulated(lib, rows, Tq, N, k, what):  # noqa: F811
    lib.emu_schedule(N + k, -1, -1)
    s = torch.zeros(rows, 1, Tq, N)
    s[:2] = scores_of(what, 2, Tq, N, k, N + k)
    check(lib, s, [0], k, lens=[N, N - 3] + [0] * (rows - 2))


@pytest.mark.gpu
@pytest.mark.parametrize("rows,N", [(16, 4001), (16, 8190), (256, 9000), (256, 20001), (513, 4090), (513, 8190), (513, 9001), (513, 20001)])
def test_both_ends_of_the_key_range(rows, N):
    """NaNs of the highest and the lowest keys (their order is that of the bits), in rows whose end leaves a few places of a
    slab without a token."""
    for n in (1000, 1021, 2047, 4081, 8129, N - 3):
        if n > N:
            continue
        s = torch.rand(2, N, generator=torch.Generator().manual_seed(n))
        bits = s.view(torch.int32)
        bits[0, 100:800:100] = torch.tensor([0x7fffffff, 0x7fff0000, 0x7ffffffe, 0x7f800000, 0x7fffffff, 0x7fe00000, 0x7fefffff], dtype=torch.int32)
        bits[0, 700:705] = torch.tensor([-2, -0x200000, -9, -0x100, -3], dtype=torch.int32)
        bits[1, 5:990:98] = -9
        sd = torch.zeros(rows, 1, 1, N, device=DEV)
        sd[:2, 0, 0] = s.to(DEV)
        lens = torch.zeros(rows, dtype=torch.int32, device=DEV)
        lens[:2] = n
        for k in (1, 3, n - 9, n - 3, n - 1):
            idx, cnt, _ = sts.sts_select(sd, [0], k, seq_lens=lens)
            assert cnt[:2, 0].tolist() == [k, k]
            for b in range(2):
                np.testing.assert_array_equal(idx[b, 0].cpu().numpy(), by_keys(s[b], n, k), err_msg=f"row {b}, length {n}, k {k}")


@pytest.mark.gpu
@pytest.mark.parametrize("N,page,k", [(32784, 16, 300), (131072, 16, 820), (131072, 8, 16384), (65544, 8, 1), (66000, 16, 900)])
def test_rows_of_block_sums(N, page, k):
    B, Hd, Tq = 3, 2, 3
    g = torch.Generator().manual_seed(N + k)
    s = torch.softmax(torch.randn(B, Hd, Tq, N, generator=g) * 2, dim=-1)
    s[0, 1] = 0.0
    lens = torch.tensor([N, N - page - 3, 70], dtype=torch.int32)
    hm = [0, 1, 1]
    idx, cnt, _ = sts.sts_select(s.to(DEV), hm, k, seq_lens=lens.to(DEV), page_size=page)
    o_idx, o_cnt, _ = oracle.select_indices(s.numpy(), np.asarray(hm, np.int32), k, seq_lens=lens.numpy(), page=page)
    np.testing.assert_array_equal(cnt.cpu().numpy(), o_cnt)
    np.testing.assert_array_equal(idx.cpu().numpy(), o_idx)


# blocks a row: 256 threads with four, eight and sixteen quads, 512 threads (more than 512 rows), and 1024 threads
@pytest.mark.gpu
@pytest.mark.parametrize("what", ["softmax", "zeros", "levels"])
@pytest.mark.parametrize("rows,blocks,page,k", [(520, 2049, 8, 205), (513, 4096, 4, 4000), (600, 4097, 4, 400), (513, 8192, 2, 1), (520, 8193, 2, 819),
                                                (513, 16384, 2, 1638), (70, 2050, 12, 300)])
def test_many_rows_of_block_sums(rows, blocks, page, k, what):
    live, N = 6, blocks * page - 1                    # the other rows are empty; the last block is cut
    s = scores_of(what, live, 1, N, k * page, blocks + k)
    sd = torch.zeros(rows, 1, 1, N, device=DEV)
    sd[:live] = s.to(DEV)
    lens = torch.zeros(rows, dtype=torch.int32)
    lens[:live] = torch.tensor([N, N - page - 1, N // 2 + 1, 1024 * page - 1, 3 * page + 1, 1])
    idx, cnt, _ = sts.sts_select(sd, [0, 0], k, seq_lens=lens.to(DEV), page_size=page)
    assert (cnt[live:] == 0).all() and (idx[live:] == -1).all()
    o_idx, o_cnt, _ = oracle.select_indices(s.numpy(), np.zeros(2, np.int32), k, seq_lens=lens[:live].numpy(), page=page)
    np.testing.assert_array_equal(cnt[:live].cpu().numpy(), o_cnt)
    np.testing.assert_array_equal(idx[:live].cpu().numpy(), o_idx)


# both sides of the line between one workgroup per row and parts of a row: rows, scores per token, N, k, bf16 scores
@pytest.mark.gpu
@pytest.mark.parametrize("rows,Tq,N,k,bf16", [(8, 5, 8193, 819, False), (8, 10, 16384, 1, False), (8, 11, 16384, 1638, False), (9, 5, 16385, 16000, False),
                                              (16, 5, 32768, 3277, False), (16, 6, 32767, 3276, False), (16, 10, 32765, 3276, True), (64, 16, 16383, 512, False),
                                              (128, 8, 16391, 1639, False), (128, 9, 16391, 1639, False), (255, 2, 20003, 2000, True)])
def test_few_rows(rows, Tq, N, k, bf16):
    live = 6                                          # the other rows are empty
    s = scores_of("softmax", live, Tq, N, k, N + k)
    s[1:3] = scores_of("zeros then scores", 2, Tq, N, k, N + k)
    s = s.to(torch.bfloat16) if bf16 else s
    sd = torch.zeros(rows, 1, Tq, N, device=DEV, dtype=s.dtype)
    sd[:live] = s.to(DEV)
    lens = torch.zeros(rows, dtype=torch.int32)
    lens[:live] = torch.tensor([N, N, N - 3, N // 2, 1023, 5])
    idx, cnt, _ = sts.sts_select(sd, [0, 0], k, seq_lens=lens.to(DEV))
    a_idx, a_cnt, agg = sts.sts_select(sd, [0, 0], k, seq_lens=lens.to(DEV), want_agg=True)
    assert torch.equal(idx, a_idx) and torch.equal(cnt, a_cnt)
    assert (cnt[live:] == 0).all() and (idx[live:] == -1).all()
    o_idx, o_cnt, o_agg = oracle.select_indices(s.float().numpy(), np.zeros(2, np.int32), k, seq_lens=lens[:live].numpy())
    np.testing.assert_array_equal(cnt[:live].cpu().numpy(), o_cnt)
    np.testing.assert_array_equal(idx[:live].cpu().numpy(), o_idx)
    np.testing.assert_array_equal(agg[0].cpu().numpy(), o_agg[0])


# many rows with several scores per token (or one scaled logit): 256 threads with four and eight quads, 512 with eight and sixteen
@pytest.mark.gpu
@pytest.mark.parametrize("how", ["sum", "max", "bf16", "logits"])
@pytest.mark.parametrize("Tq,N,k", [(3, 4095, 400), (1, 4100, 410), (2, 8189, 8000), (9, 8193, 800), (4, 16384, 1638), (1, 16387, 300), (5, 32767, 3276)])
def test_many_rows_of_several_scores(Tq, N, k, how):
    rows, live = 513, 5                               # the other rows are empty
    s = scores_of("softmax", live, Tq, N, k, N + k)
    s[1] = scores_of("signed", 1, Tq, N, k, N + k)[0]
    lse = None
    kw = {}
    if how == "bf16":
        s = s.to(torch.bfloat16)
    if how == "max":
        kw["reduce"] = sts.STS_REDUCE_MAX
    if how == "logits":
        s = torch.log(s.abs().clamp_min(1e-30))
        lse = torch.zeros(rows, 1, Tq, device=DEV) + torch.arange(Tq, device=DEV) / 16
        kw.update(kind=sts.STS_SCORES_LOGITS_LSE, lse=lse)
    sd = torch.zeros(rows, 1, Tq, N, device=DEV, dtype=s.dtype)
    sd[:live] = s.to(DEV)
    lens = torch.zeros(rows, dtype=torch.int32)
    lens[:live] = torch.tensor([N, N - 1, N // 2, 1023, 6])
    idx, cnt, agg = sts.sts_select(sd, [0, 0], k, seq_lens=lens.to(DEV), want_agg=True, **kw)
    idx2, _, _ = sts.sts_select(sd, [0, 0], k, seq_lens=lens.to(DEV), **kw)
    assert torch.equal(idx, idx2) and (idx[live:] == -1).all()
    a = agg[:live].cpu()
    if how == "logits":
        want = torch.exp(s - lse[:live].cpu()[..., None]).sum(dim=2)
    else:
        want = s[:, :, 0].float()
        for i in range(1, Tq):
            want = torch.maximum(want, s[:, :, i].float()) if how == "max" else want + s[:, :, i].float()
    for b in range(live):
        n = int(lens[b])
        if how == "logits":
            # the device's exponential is good to 1e-5 relative (see prob_of)
            torch.testing.assert_close(a[b, 0, :n], want[b, 0, :n], rtol=1e-5, atol=0.0)
        else:
            assert torch.equal(a[b, 0, :n], want[b, 0, :n])
        assert (a[b, 0, n:] == 0).all()
    o_idx, o_cnt, _ = oracle.select_indices(a[:, :, None].numpy(), np.zeros(2, np.int32), k, seq_lens=lens[:live].numpy())
    np.testing.assert_array_equal(cnt[:live].cpu().numpy(), o_cnt)
    np.testing.assert_array_equal(idx[:live].cpu().numpy(), o_idx)


# calls of few rows whose scores are summed first and then ranked by one workgroup per row, on both sides of the host's lines: rows, scores
# per token, N, k, bf16 scores, the kernels' first name
SUMMED = [(8, 3, 16385, 1638, False, "select_row_sums"), (32, 3, 32768, 300, True, "select_row_sums"), (33, 4, 20000, 2000, False, "select_row_scores_kernel"),
          (33, 5, 20000, 2000, False, "select_row_sums"), (16, 2, 32768, 3277, False, "select_row_scores_kernel"), (16, 2, 32769, 3277, False, "select_row_sums"),
          (34, 2, 65536, 6554, False, "select_row_sums"), (35, 2, 65536, 655, True, "select_clear16"), (8, 9, 65537, 655, False, "select_clear16"),
          (16, 1, 32769, 3277, False, "select_row_long_kernel"), (127, 1, 65536, 6554, False, "select_row_long_kernel"), (16, 1, 65537, 6554, False, "select_clear16"),
          (16, 5, 40003, 20000, False, "select_clear16"), (7, 5, 33001, 3301, False, "select_clear16"), (65, 4, 49152, 4915, False, "select_row_sums"),
          (9, 2, 49153, 4000, False, "select_row_sums"), (66, 5, 49152, 4915, True, "select_clear16"), (64, 3, 45000, 4500, False, "select_clear16")]


@pytest.mark.parametrize("rows,Tq,N,k,bf16,first", SUMMED)
def test_summed_rows_route(lib, rows, Tq, N, k, bf16, first):  # noqa: F811
    assert route(lib, rows, 1, Tq, N, 2, k, bf16=bf16).startswith(first)
    assert not route(lib, rows, 1, Tq, N, 2, k, bf16=bf16, agg=True).startswith("select_row_sums")


def heavy_start(n, seed):
    """A row's scores with most of the heavy ones among the first 256 tokens (sinks)."""
    r = torch.randn(n, generator=torch.Generator().manual_seed(seed))
    r[:256] += 3
    return torch.softmax(r, dim=-1)


# rows, tokens, those that are valid, kept, bf16: forms that sample one quad of 2, 4, 6 and 8, filled, partly filled and nearly empty
CLUSTERED = [(256, 16384, 2048, 204, False), (513, 16384, 4096, 409, False), (16, 32768, 4096, 256, False), (16, 32768, 16384, 256, False), (16, 32768, 32768, 700, False),
             (513, 32768, 2048, 204, False), (16, 33001, 33001, 256, False), (16, 65536, 1024, 102, False), (16, 65536, 4096, 409, False), (16, 65536, 65536, 256, False),
             (64, 65536, 32773, 300, True), (300, 131072, 131072, 300, True),
             (300, 131072, 65541, 500, True)]


@pytest.mark.parametrize("rows,N,n,k,bf16", CLUSTERED)
def test_the_sample_is_of_all_parts_of_the_row(lib, rows, N, n, k, bf16):  # noqa: F811
    """Heavy tokens next to each other, or in the few registers that a short row fills, do not mislead the window: no more
    counting (barriers) than the same scores need in another order."""
    lib.emu_schedule(N + k, -1, -1)
    passed = []
    for order in (torch.arange(n), torch.randperm(n, generator=torch.Generator().manual_seed(n))):
        s = torch.zeros(rows, 1, 1, N, dtype=torch.bfloat16 if bf16 else torch.float32)
        s[0, 0, 0, :n] = heavy_start(n, N)[order].to(s.dtype)
        lib.emu_barriers()
        check(lib, s, [0], k, lens=[n] + [0] * (rows - 1))
        passed.append(lib.emu_barriers())
    assert passed[0] <= passed[1]


# Budgets next to the row's length: the rule for calls of few rows does not take those of 128 rows and more, of which one
# workgroup per row ranks up to 512 only where they are this long; and fewer rows have lists too long for it
@pytest.mark.parametrize("rows", [127, 128, 129, 255, 512, 513, 4000])
@pytest.mark.parametrize("N", [32769, 40000, 65536])
def test_rows_that_keep_nearly_everything_route(lib, rows, N):  # noqa: F811
    for k in (N * 92 // 100, N * 93 // 100, N - 1, N, N + 7):
        for Tq in (1, 2, 5):
            for lens in (False, True):
                got = route(lib, rows, 1, Tq, N, 2, k, lens=lens)        # (and status 0)
                assert "select_sampled_kernel" in got, (k, Tq, got)


def test_rows_that_keep_nearly_everything_emulated(lib):  # noqa: F811
    lib.emu_schedule(7, -1, -1)
    for rows, N, k in ((513, 32769, 32700), (512, 40000, 39999), (128, 33001, 33001)):
        s = torch.zeros(rows, 1, 1, N)
        s[:2] = scores_of("zeros then scores", 2, 1, N, N // 3, N)
        check(lib, s, [0], k, lens=[N, N - 9] + [0] * (rows - 2))


@pytest.mark.gpu
@pytest.mark.parametrize("rows,N,k", [(513, 32769, 32700), (600, 40000, 40000), (528, 65536, 65535), (200, 40000, 39900)])
def test_rows_that_keep_nearly_everything(rows, N, k):
    live = 2                                          # the other rows are empty
    s = scores_of("zeros then scores", live, 1, N, N // 3, N)
    sd = torch.zeros(rows, 1, 1, N, device=DEV)
    sd[:live] = s.to(DEV)
    lens = torch.zeros(rows, dtype=torch.int32)
    lens[:live] = torch.tensor([N, N - 9])
    idx, cnt, _ = sts.sts_select(sd, [0], k, seq_lens=lens.to(DEV))
    assert (cnt[live:] == 0).all() and (idx[live:] == -1).all()
    o_idx, o_cnt, _ = oracle.select_indices(s.numpy(), np.zeros(1, np.int32), k, seq_lens=lens[:live].numpy())
    np.testing.assert_array_equal(cnt[:live].cpu().numpy(), o_cnt)
    np.testing.assert_array_equal(idx[:live].cpu().numpy(), o_idx)


@pytest.mark.parametrize("S,R,Hd,Ht,N,k", [(1, 64, 16, 32, 40000, 38000), (1, 33, 16, 16, 65536, 65536), (1, 1, 40, 128, 33001, 32700)])
def test_head_mapping_that_keeps_nearly_everything_route(lib, S, R, Hd, Ht, N, k):  # noqa: F811
    p = binding.HeadmapParams(S=S, R=R, Hd=Hd, Ht=Ht, N=N, k=k, a_d=1 << 20, a_t=1 << 20, map=1 << 20)
    p.workspace, p.workspace_bytes = 1 << 20, lib.sts_headmap_workspace_bytes(ctypes.byref(p))
    lib.emu_only_names(1)
    try:
        assert lib.sts_head_map(ctypes.byref(p), None) == 0
        assert "headmap_overlap" in lib.emu_names().decode()
    finally:
        lib.emu_only_names(0)


def test_summed_rows_emulated(lib):  # noqa: F811
    """With room for the sums, and with the workspace that such a call needed for the sampled selection."""
    lib.emu_schedule(5, -1, -1)
    s = torch.zeros(8, 1, 3, 16401)
    s[:1] = scores_of("softmax", 1, 3, 16401, 1640, 3)
    for ws in (None, 8 * 3 * 1352 * 8):
        check(lib, s, [0, 0], 1640, lens=[16401] + [0] * 7, ws_bytes=ws)


@pytest.mark.gpu
@pytest.mark.parametrize("what", ["softmax", "zeros then scores", "one value", "signed", "logits"])
@pytest.mark.parametrize("rows,Tq,N,k,bf16,first", [x for x in SUMMED if x[5].startswith("select_row")])
def test_summed_rows(rows, Tq, N, k, bf16, first, what):
    live = 5                                          # the other rows are empty
    s = scores_of("softmax" if what == "logits" else what, live, Tq, N, k, N + k)
    kw = {}
    if what == "logits":
        s = torch.log(s.clamp_min(1e-30))
        kw = {"kind": sts.STS_SCORES_LOGITS_LSE, "lse": torch.zeros(rows, 1, Tq, device=DEV) + torch.arange(Tq, device=DEV) / 16}
    s = s.to(torch.bfloat16) if bf16 else s
    flat = torch.zeros(rows * Tq * N + 8, device=DEV, dtype=s.dtype)
    sd = flat[N % 2:N % 2 + rows * Tq * N].view(rows, 1, Tq, N)      # an odd row length also starts at an odd element
    sd[:live] = s.to(DEV)
    lens = torch.zeros(rows, dtype=torch.int32)
    lens[:live] = torch.tensor([N, N - 1, N // 2 + 3, 1023, 5])
    idx, cnt, _ = sts.sts_select(sd, [0, 0], k, seq_lens=lens.to(DEV), **kw)
    a_idx, a_cnt, agg = sts.sts_select(sd, [0, 0], k, seq_lens=lens.to(DEV), want_agg=True, **kw)      # (the sampled selection's way)
    assert torch.equal(idx, a_idx) and torch.equal(cnt, a_cnt)
    assert (cnt[live:] == 0).all() and (idx[live:] == -1).all()
    o_idx, o_cnt, _ = oracle.select_indices(agg[:live, :, None].cpu().numpy(), np.zeros(2, np.int32), k, seq_lens=lens[:live].numpy())
    np.testing.assert_array_equal(cnt[:live].cpu().numpy(), o_cnt)
    np.testing.assert_array_equal(idx[:live].cpu().numpy(), o_idx)


@pytest.mark.gpu
@pytest.mark.parametrize("k", [1, 3, 30, 300])
@pytest.mark.parametrize("rows,N,bf16", [(513, 16383, False), (513, 32768, False), (16, 17000, False), (16, 49000, False), (300, 65535, True), (300, 131071, True)])
def test_few_kept(rows, N, bf16, k):
    """Windows whose upper end is the sample's largest key; heavy tokens that the sample sees all of, or none."""
    live = 6                                          # the other rows are empty
    s = scores_of("softmax", live, 1, N, k, N + k)
    s[1, ..., N // 2:N // 2 + max(k, 64)] += 0.5
    for r in range(2, live):
        s[r, ..., r - 2::4][..., ::max(1, N // (8 * k))] += 0.25
    s = s.to(torch.bfloat16) if bf16 else s
    sd = torch.zeros(rows, 1, 1, N, device=DEV, dtype=s.dtype)
    sd[:live] = s.to(DEV)
    lens = torch.zeros(rows, dtype=torch.int32)
    lens[:live] = torch.tensor([N, N, N, N - 1, 1024, N // 3])
    idx, cnt, _ = sts.sts_select(sd, [0, 0], k, seq_lens=lens.to(DEV))
    o_idx, o_cnt, _ = oracle.select_indices(s.float().numpy(), np.zeros(2, np.int32), k, seq_lens=lens[:live].numpy())
    np.testing.assert_array_equal(cnt[:live].cpu().numpy(), o_cnt)
    np.testing.assert_array_equal(idx[:live].cpu().numpy(), o_idx)


# scores per token, N, page: one token past a sweep's 1024 and short of it, rows within one page, the longest row that is
# ranked by one workgroup and one past it
BLOCKS = [(1, 4, 4), (3, 5, 256), (9, 1025, 16), (2, 8191, 8), (5, 4099, 64), (2, 65531, 4), (2, 65538, 4)]


@pytest.mark.parametrize("Tq,N,page", BLOCKS)
def test_blocks_of_any_length_route(lib, Tq, N, page):  # noqa: F811
    for kw in ({}, {"bf16": True}, {"unaligned": True}):
        assert "select_aggblock" in route(lib, 3, 2, Tq, N, 2, 1, page=page, **kw)
    assert ("select_aggblock" in route(lib, 3, 2, Tq, N, 2, 1, page=page, agg=True, unaligned=True)) == (N % page == 0)


@pytest.mark.gpu
@pytest.mark.parametrize("how", ["fp32", "bf16", "logits", "max"])
@pytest.mark.parametrize("Tq,N,page", BLOCKS)
def test_blocks_of_any_length(Tq, N, page, how):
    """The same lists as the kernels that store the sums per token make (asked for them), and as the oracle, bit for bit."""
    B, Hd = 3, 2
    g = torch.Generator().manual_seed(N + page)
    s = torch.randn(B, Hd, Tq, N, generator=g)
    s = s if how == "logits" else torch.softmax(s * 2, dim=-1)
    s = s.to(torch.bfloat16) if how == "bf16" else s
    lens = torch.tensor([N, max(N - page // 2 - 1, 1), N // 2 + 1], dtype=torch.int32)
    kw = {"lse": torch.rand(B, Hd, Tq, generator=g).to(DEV), "kind": sts.STS_SCORES_LOGITS_LSE} if how == "logits" else {}
    if how == "max":
        kw = {"reduce": sts.STS_REDUCE_MAX}
    nblk = (N + page - 1) // page
    k = max(1, nblk // 5)
    flat = torch.zeros(s.numel() + 8, dtype=s.dtype, device=DEV)
    sd = flat[1:1 + s.numel()].view(s.shape)          # (an odd element to start at)
    sd.copy_(s.to(DEV))
    idx, cnt, agg = sts.sts_select(sd, [0, 1], k, seq_lens=lens.to(DEV), page_size=page, want_agg=True, **kw)
    plain, pcnt, _ = sts.sts_select(sd, [0, 1], k, seq_lens=lens.to(DEV), page_size=page, **kw)
    assert torch.equal(idx, plain) and torch.equal(cnt, pcnt)
    t_idx, t_cnt, t_agg = sts.sts_select(sd, [0, 1], N, seq_lens=lens.to(DEV), want_agg=True, **kw)
    assert torch.equal(agg, t_agg)                    # per token as without pages
    o_idx, o_cnt, _ = oracle.select_indices(agg[:, :, None].cpu().numpy(), np.array([0, 1], np.int32), k, seq_lens=lens.numpy(), page=page)
    np.testing.assert_array_equal(cnt.cpu().numpy(), o_cnt)
    np.testing.assert_array_equal(idx.cpu().numpy(), o_idx)
