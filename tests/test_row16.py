"""Rows of one bf16 score per token, ranked in one workgroup's registers (select_row16_kernel in
csrc/select_row.hip), against the CPU oracle bit for bit: at the edges of the kernel's forms, at odd
addresses and lengths, and on scores that its sample and its windows of keys do not expect. On the GPU,
and compiled for the CPU (tests/emulated), where the waves run in random order."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_15508_amd as sts
from test_select_emulated import by_keys, check, check_keys, lib, route  # noqa: F401  (lib: the emulated library, a fixture)

PATH_KNOB = 3


def scores_of(what, N, k, seed):
    g = torch.Generator().manual_seed(seed)
    r = torch.randn(N, generator=g)
    p = torch.softmax(r * 2, dim=-1)
    some = torch.rand(N, generator=g)
    if what == "softmax":
        return p
    if what == "zeros":                               # about as many scores as are kept, zeros otherwise
        return p * (some < k / N)
    if what == "zeros then a stretch":                # exactly as many: the lowest score lies alone above the gap
        p[:N - k] = 0
        return p
    if what == "constant":
        return torch.full((N,), -0.25)
    if what == "signed":                              # zeros of both signs in the middle
        r[some < 0.3] = 0.0
        r[some < 0.1] = -0.0
        return r
    if what == "infinite":                            # saturated scores above, masked ones below
        r[some < k / N / 2] = float("inf")
        r[some > 0.9] = float("-inf")
        return r
    if what == "heavy tail":                          # keys all over the range
        return torch.exp(r * 30)
    if what == "sorted":
        return p.sort().values
    p[N // 3:N // 3 + N // 8] *= 1e5                  # "stretch"
    return p


# lengths around the forms' limits (8192, 16384, 32768, 65536, 131072 tokens), below the sampled ones (1024), a
# list longer than what is staged at once, a budget of one, of all but one and of all
CASES = [
    ("softmax", 8, 3), ("signed", 1023, 100), ("softmax", 1024, 102), ("infinite", 4096, 400), ("constant", 8191, 4000),
    ("softmax", 8193, 8192), ("zeros", 16384, 1638), ("zeros then a stretch", 16385, 1638), ("signed", 32768, 20000),
    ("stretch", 32769, 3277), ("heavy tail", 65535, 6553), ("sorted", 65536, 1), ("zeros then a stretch", 65537, 6553),
    ("softmax", 100001, 10000), ("signed", 131071, 131071), ("zeros", 131072, 13107), ("constant", 131072, 9000),
]


@pytest.mark.parametrize("what,N,k", CASES)
def test_emulated(lib, what, N, k):  # noqa: F811
    lib.emu_schedule(N, -1, -1)
    lib.sts_set_knob(PATH_KNOB, 6.0)
    try:
        s = scores_of(what, N, k, N + k).to(torch.bfloat16)
        flat = torch.zeros(2 * N + 3, dtype=torch.bfloat16)
        at = flat[3:].view(2, 1, 1, N)                # an odd element
        at[0, 0, 0], at[1, 0, 0] = s, s.flip(0)
        check(lib, at, [0, 0], k, lens=[N, max(1, N - 9)])
    finally:
        lib.sts_set_knob(PATH_KNOB, float("nan"))


@pytest.mark.gpu
@pytest.mark.parametrize("what,N,k", CASES)
def test_on_the_gpu(what, N, k):
    B, Hd = 5, 3
    s = torch.stack([torch.stack([scores_of(what, N, k, N + k + 7 * b + j) for j in range(Hd)]) for b in range(B)]).to(torch.bfloat16)
    flat = torch.zeros(s.numel() + 3, dtype=torch.bfloat16, device="cuda:0")
    sd = flat[3:].view(B, Hd, 1, N)
    sd.copy_(s[:, :, None])
    hm = [0, 0, 2]                                    # draft head 1 is read by none
    kh = [k, 1, max(1, k - k // 3)]
    lens = torch.tensor([N, max(1, N - 9), N // 2 + 1, 0, min(N, 20)], dtype=torch.int32)
    sts.set_knob("select_path", 6)
    try:
        idx, cnt, _ = sts.sts_select(sd, hm, k, k_head=kh, seq_lens=lens.to("cuda:0"))
    finally:
        sts.set_knob("select_path", None)
    o_idx, o_cnt, _ = oracle.select_indices(s[:, :, None].float().numpy(), np.asarray(hm, np.int32), k, k_head=kh, seq_lens=lens.numpy())
    np.testing.assert_array_equal(cnt.cpu().numpy(), o_cnt)
    np.testing.assert_array_equal(idx.cpu().numpy(), o_idx)
    if N >= 4096:                                     # the library's own rule
        idx2, cnt2, _ = sts.sts_select(sd, hm, k, k_head=kh, seq_lens=lens.to("cuda:0"))
        assert torch.equal(idx, idx2) and torch.equal(cnt, cnt2)


# lengths on both sides of a quarter of what the workgroup's registers hold, and next to them; budgets below and beyond the length
SHORT = [(20001, 8192), (20000, 8193), (20001, 8185), (65536, 16384), (65535, 16385), (131072, 32768), (131071, 32769), (131072, 1025), (65536, 700)]


def short_row(N, n, seed):
    s = torch.full((2, N), float("inf"))              # (above all others, were they looked at)
    for b, what in enumerate(("softmax", "signed")):
        s[b, :n] = scores_of(what, n, max(1, n // 3), seed + b)
    return s.to(torch.bfloat16)


@pytest.mark.parametrize("N,n", SHORT)
def test_rows_that_are_mostly_empty_emulated(lib, N, n):  # noqa: F811
    lib.emu_schedule(n, -1, -1)
    for k in (n // 3, n - 1, n, min(N, n + 9)):
        check(lib, short_row(N, n, N)[:, None, None].contiguous(), [0, 0], k, lens=[n, n])


@pytest.mark.gpu
@pytest.mark.parametrize("N,n", SHORT)
def test_rows_that_are_mostly_empty_on_the_gpu(N, n):
    s = short_row(N, n, N)[:, None, None].contiguous()
    flat = torch.zeros(s.numel() + 1, dtype=torch.bfloat16, device="cuda:0")
    sd = flat[1:].view(s.shape)                       # an odd element
    sd.copy_(s)
    lens = torch.full((2,), n, dtype=torch.int32)
    for k in (1, n // 3, n - 1, n, min(N, n + 9)):
        idx, cnt, _ = sts.sts_select(sd, [0, 0], k, seq_lens=lens.to("cuda:0"))
        o_idx, o_cnt, _ = oracle.select_indices(s.float().numpy(), np.zeros(2, np.int32), k, seq_lens=lens.numpy())
        np.testing.assert_array_equal(cnt.cpu().numpy(), o_cnt)
        np.testing.assert_array_equal(idx.cpu().numpy(), o_idx)


@pytest.mark.parametrize("rows,N,kernel", [
    (1024, 65536, "select_row16_kernel<512, 16>"), (1024, 65544, "select_rowpass_kernel<256, true>"), (1024, 114680, "select_rowpass_kernel<256, true>"),
    (1024, 114688, "select_row16_kernel<1024, 16>"), (1023, 65544, "select_row16_kernel<1024, 16>"), (1024, 65545, "select_row16_kernel<1024, 16>"),
    (1024, 131080, "select_rowpass_kernel<256, true>"),
])
def test_many_rows_that_take_a_compute_unit_each(lib, rows, N, kernel):  # noqa: F811
    """Many rows of more than half of what fits registers go by plain passes over them."""
    assert route(lib, rows, 1, 1, N, 2, N // 10, bf16=True, lens=True) == kernel


def lowest_nans(N):
    """Every negative NaN of bf16 there is at the end of a row, the lowest ones last but one and before."""
    s = torch.rand(N, generator=torch.Generator().manual_seed(N)).to(torch.bfloat16)
    s.view(torch.int16)[-127:] = torch.arange(-1, -128, -1, dtype=torch.int16)
    s.view(torch.int16)[5] = -2
    return s


@pytest.mark.parametrize("N", [300, 4096, 16385])
def test_lowest_nans_emulated(lib, N):  # noqa: F811
    """The two lowest keys are told apart, as every path does that compares widened scores."""
    lib.emu_schedule(1, -1, -1)
    lib.sts_set_knob(PATH_KNOB, 6.0)
    try:
        for k in (N - 1, N - 2, N - 3, N - 100):
            check_keys(lib, torch.stack([lowest_nans(N), lowest_nans(N).flip(0)]), 2, k, [N, N])
    finally:
        lib.sts_set_knob(PATH_KNOB, float("nan"))


@pytest.mark.parametrize("rows,N", [(16, 4096), (256, 9000), (513, 8190)])
def test_lowest_nans_of_rows_in_fp32_emulated(lib, rows, N):  # noqa: F811
    lib.emu_schedule(1, -1, -1)
    s = torch.rand(N, generator=torch.Generator().manual_seed(N))
    s.view(torch.int32)[-9:] = torch.arange(-1, -10, -1, dtype=torch.int32)
    s.view(torch.int32)[5] = -2
    for k in (N - 1, N - 2, N - 3, N - 7):
        check_keys(lib, torch.stack([s, s.flip(0)]), rows, k, [N, N])


@pytest.mark.gpu
@pytest.mark.parametrize("N", [4096, 16384, 32768, 65536, 131072])
def test_lowest_nans_on_the_gpu(N):
    s = torch.stack([lowest_nans(N), lowest_nans(N).flip(0)])
    for k in (N - 1, N - 2, N - 100):
        idx, _, _ = sts.sts_select(s[:, None, None].to("cuda:0").contiguous(), [0], k)
        for b in range(2):
            np.testing.assert_array_equal(idx[b, 0].cpu().numpy(), by_keys(s[b], N, k))
