"""The selection's kernels compiled for the CPU (tests/emulated: a workgroup is a thread, its work-items are
fibers) under schedules that a GPU run does not take on demand: the order of the waves between two barriers is
random, and one wave of one part can be held back until nothing else in its workgroup can go on. Index lists
and counts against the CPU oracle, bit for bit. No GPU is involved."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

import oracle
from paper_2605_15508_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_15508_amd", "csrc")
HERE = os.path.join(ROOT, "tests", "emulated")
SOURCES = ["api.hip", "select.hip", "select_sampled.hip", "select_row.hip", "headmap.hip", "union.hip"]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    clang = shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"
    if not os.path.exists(clang):
        pytest.skip("clang++ not available")          # (the sources use its vector types)
    tmp = tmp_path_factory.mktemp("emulated")
    flags = ["-std=c++17", "-O1", "-fPIC", "-w", "-ffp-contract=off", "-I", HERE, "-I", CSRC]
    jobs = [(s, ["-x", "c++", "-include", os.path.join(HERE, "launch.h"), os.path.join(CSRC, s)]) for s in SOURCES]
    jobs.append(("emulator.cpp", [os.path.join(HERE, "emulator.cpp")]))
    procs = [(s, subprocess.Popen([clang, *flags, "-c", *a, "-o", str(tmp / (s + ".o"))], stderr=subprocess.PIPE, text=True))
             for s, a in jobs]
    for s, p in procs:
        err = p.communicate()[1]
        assert p.returncode == 0, f"{s}: {err[-3000:]}"
    so = str(tmp / "libemulated.so")
    subprocess.run([clang, "-shared", "-o", so, *[str(tmp / (s + ".o")) for s, _ in jobs], "-lpthread"], check=True)
    lib = ctypes.CDLL(so)
    lib.sts_select_workspace_bytes.restype = ctypes.c_size_t
    lib.sts_headmap_workspace_bytes.restype = ctypes.c_size_t
    lib.emu_loaded.restype = ctypes.c_uint64
    lib.emu_barriers.restype = ctypes.c_uint64
    lib.emu_names.restype = ctypes.c_char_p
    lib.sts_set_knob.argtypes = [ctypes.c_int, ctypes.c_double]
    return lib


def select(lib, scores, hm, k, k_head=None, lens=None, ws_offset=0, ws_bytes=None, status=0):
    B, Hd, Tq, N = scores.shape
    hm = np.asarray(hm, np.int32)
    kh = None if k_head is None else np.asarray(k_head, np.int32)
    lens = None if lens is None else np.asarray(lens, np.int32)
    idx, cnt = np.full((B, len(hm), k), -7, np.int32), np.full((B, len(hm)), -7, np.int32)
    at = lambda a: None if a is None else a.ctypes.data
    p = binding.SelectParams(B=B, Hd=Hd, Tq=Tq, N=N, Hq=len(hm), k=k, scores=scores.data_ptr(), head_map=at(hm), seq_lens=at(lens),
                             indices=at(idx), counts=at(cnt), k_head=at(kh), scores_bf16=int(scores.dtype == torch.bfloat16))
    need = lib.sts_select_workspace_bytes(ctypes.byref(p))
    ws = np.full(need + 512, 0xA5, np.uint8)
    p.workspace = ws.ctypes.data + -ws.ctypes.data % 256 + ws_offset if ws_bytes != 0 else None
    p.workspace_bytes = need if ws_bytes is None else ws_bytes
    assert lib.sts_select(ctypes.byref(p), None) == status
    return idx, cnt


def route(lib, B, Hd, Tq, N, Hq, k, bf16=False, page=1, lens=False, agg=False, logits=False, unaligned=False, status=0):
    """The kernels that a call launches, without running them: their names, in order."""
    hm = np.arange(Hq, dtype=np.int32) * Hd // Hq
    p = binding.SelectParams(B=B, Hd=Hd, Tq=Tq, N=N, Hq=Hq, k=k, page_size=page, kind=int(logits), scores=(1 << 20) + 2 * unaligned, head_map=hm.ctypes.data,
                             seq_lens=1 << 20 if lens else None, lse=1 << 20 if logits else None, agg_out=1 << 20 if agg else None, indices=1 << 20,
                             counts=1 << 20, scores_bf16=int(bf16))
    p.workspace_bytes = lib.sts_select_workspace_bytes(ctypes.byref(p))
    p.workspace = 1 << 20
    lib.emu_only_names(1)
    try:
        assert lib.sts_select(ctypes.byref(p), None) == status
        return lib.emu_names().decode()
    finally:
        lib.emu_only_names(0)


def check(lib, scores, hm, k, **kw):
    idx, cnt = select(lib, scores, hm, k, **kw)
    lens = kw.get("lens")
    o_idx, o_cnt, _ = oracle.select_indices(scores.float().numpy(), np.asarray(hm, np.int32), k, k_head=kw.get("k_head"),
                                            seq_lens=None if lens is None else np.asarray(lens, np.int32))
    np.testing.assert_array_equal(cnt, o_cnt)
    np.testing.assert_array_equal(idx, o_idx)


def softmax(B, Hd, Tq, N, seed):
    g = torch.Generator().manual_seed(seed)
    return torch.softmax(torch.randn(B, Hd, Tq, N, generator=g) * 2, dim=-1)


# (seed, part and wave held back; -1: none)
SCHEDULES = [(1, -1, -1), (2, -1, -1), (3, 0, 0), (4, 1, 0), (5, 1, 1), (6, 0, 15)]


@pytest.mark.parametrize("schedule", SCHEDULES)
@pytest.mark.parametrize("B,Hd,Tq,N,k", [
    (1, 2, 2, 20000, 2000),          # three parts
    (2, 1, 1, 33001, 3301),          # five
    (1, 1, 1, 70000, 300),           # nine; a small budget
])
def test_parts_that_exchange_the_keys_around_the_threshold(lib, B, Hd, Tq, N, k, schedule):
    """The keys that share the threshold's bin travel between the parts one by one: what a part publishes is its own
    keys only, however late the wave that publishes them comes."""
    lib.emu_schedule(*schedule)
    check(lib, softmax(B, Hd, Tq, N, N + k), list(range(Hd)) + [0], k, lens=[N, N - 777][:B])


def between_samples(N, run=32, at_least=300):
    """A stretch of a row of N tokens that no sampled run touches (one run in S, at a scattered place of its
    period, about 4096 keys, 8192 beyond 256K tokens)."""
    row_runs, target, S = -(-N // run), 8192 if N > 262144 else 4096, 1
    while -(-row_runs // S) * run > target:
        S *= 2
    starts = [(i * S + ((i * 0x9e3779b1 & 0xffffffff) >> 16 & (S - 1))) * run for i in range(row_runs // S)]
    gaps = [(b - a - run, a + run) for a, b in zip(starts, starts[1:])]
    size, at = max(gaps)
    assert size >= at_least
    return at, size


@pytest.mark.parametrize("late_wave", [-1, 0, 5, 15])
@pytest.mark.parametrize("N,k,path", [(40002, 50, 0), (131072, 50, 0), (131072, 50, 5)])      # several parts; one part per row
def test_equal_scores_above_all_that_the_sample_saw(lib, N, k, path, late_wave):
    """A few hundred equal scores far above the rest where no sampled run lies: the band has no upper edge, and the
    threshold is found by narrowing its last, open bin down to the one key."""
    s = softmax(1, 1, 1, N, N) * 1e-20
    at, _ = between_samples(N)
    s[..., at:at + 250] = 3.0
    s[..., at + 250:at + 290] = torch.linspace(1.0, 2.0, 40)
    lib.sts_set_knob(3, float(path))
    lib.emu_schedule(2, 0 if path == 5 else at // 8192, late_wave)       # in the part that holds the stretch
    try:
        check(lib, s, [0, 0], k)
        check(lib, s, [0], 270)
    finally:
        lib.sts_set_knob(3, float("nan"))


@pytest.mark.parametrize("B,Hd,N,k", [
    (1, 1, 4000, 700), (1, 1, 8190, 700),            # 1024 threads per row: one quad each, two
    (1, 256, 8193, 40), (3, 200, 4001, 40),          # many rows: 1024 threads and four quads, 256 threads
    (1, 1, 20000, 700),                              # the sampled selection
])
def test_more_equal_nans_than_are_kept(lib, B, Hd, N, k):
    """NaNs are ordered above +inf by their bits: the highest of them, 0x7fffffff, has no key above it."""
    lib.emu_schedule(1, -1, -1)
    bits = torch.rand(B, Hd, 1, N, generator=torch.Generator().manual_seed(N)).view(torch.int32)
    bits[..., 3::2] = 0x7fffffff
    bits[..., 1::10] = 0x7fc00000
    s = bits.view(torch.float32)
    for budget in (k, N - N // 3):                   # ... and all of them kept
        idx, cnt = select(lib, s, [0, Hd - 1], budget)
        for t, j in ((0, 0), (1, Hd - 1)):           # (no negative values: the keys are ordered like the bits)
            want = np.sort(np.argsort(-bits[0, j, 0].numpy().astype(np.int64), kind="stable")[:budget])
            np.testing.assert_array_equal(idx[0, t], want)
        assert (cnt == budget).all()


@pytest.mark.parametrize("ws_offset,ws_bytes", [(0, None), (64, None), (0, 256), (0, 0)])
def test_many_rows_are_served_without_a_usable_workspace(lib, ws_offset, ws_bytes):
    """A row for every second compute unit: one workgroup per row needs no scratch memory, so one that is missing, too
    small or not aligned is no reason to refuse the call; fewer rows need theirs."""
    lib.emu_schedule(1, -1, -1)
    check(lib, softmax(2, 64, 1, 8200, 5), [0, 63, 17], 500, lens=[8200, 8197], ws_offset=ws_offset, ws_bytes=ws_bytes)
    # (and a budget for which a workgroup's list is too short)
    check(lib, softmax(1, 1, 1, 140000, 5).expand(128, 1, 1, 140000).contiguous(), [0], 60000, lens=[140000] + [0] * 127,
          ws_offset=ws_offset, ws_bytes=ws_bytes)
    few = softmax(1, 2, 1, 20000, 5)
    select(lib, few, [0, 1], 500, ws_offset=ws_offset, ws_bytes=ws_bytes, status=0 if (ws_offset, ws_bytes) == (0, None) else -3)


@pytest.mark.parametrize("S,Hd,Ht,R,N,k", [
    (1, 4, 3, 1, 70001, 9000),       # few row pairs: 2048 tokens and several waves on a list
    (2, 33, 17, 1, 40000, 333),      # two groups of draft heads, chunks of 32768
    (1, 1, 1, 3, 9, 20),             # fewer tokens than asked for
    (1, 2, 20, 1, 33000, 33000),     # every token
])
def test_overlap_counts_of_chunks(lib, S, Hd, Ht, R, N, k):
    lib.emu_schedule(1, -1, -1)
    rng = np.random.default_rng(N + k)
    a_d = rng.random((S, Hd, R, N), dtype=np.float32)
    a_t = rng.random((S, Ht, R, N), dtype=np.float32)
    mp, ov = np.full(Ht, -7, np.int32), np.full((Ht, Hd), -7, np.int64)
    p = binding.HeadmapParams(S=S, R=R, Hd=Hd, Ht=Ht, N=N, k=k, a_d=a_d.ctypes.data, a_t=a_t.ctypes.data, map=mp.ctypes.data,
                              overlap=ov.ctypes.data)
    need = lib.sts_headmap_workspace_bytes(ctypes.byref(p))
    ws = np.full(need + 256, 0xA5, np.uint8)
    p.workspace, p.workspace_bytes = ws.ctypes.data + -ws.ctypes.data % 256, need
    assert lib.sts_head_map(ctypes.byref(p), None) == 0
    o_mp, o_ov = oracle.head_mapping(a_d, a_t, k)
    np.testing.assert_array_equal(ov, o_ov)
    np.testing.assert_array_equal(mp, o_mp)


def repeated(what, N, k, seed):
    """Rows in which one or two values, next to the threshold, are shared by much of the row."""
    g = torch.Generator().manual_seed(seed)
    s = softmax(1, 1, 1, N, seed)
    few = torch.rand(1, 1, 1, N, generator=g) < k / N
    if what == "zeros":                               # about as many scores as are kept, zeros otherwise
        return s * few
    if what == "window":                              # ... in one stretch
        s[..., :N - k] = 0
        return s
    if what == "two":                                 # two values, the threshold at the edge between them
        return torch.where(few, 0.5, 0.25)
    if what == "between":                             # ... and a few hundred values between the two
        return torch.where(torch.rand(1, 1, 1, N, generator=g) < 0.01, 0.3 + s, torch.where(few, 0.5, 0.25))
    if what == "top":                                 # saturated scores, more than are kept of them or not quite
        s[torch.rand(1, 1, 1, N, generator=g) < k / N] = float("inf")
        return s
    if what == "negative":                            # zeros of both signs above negative scores
        s = torch.where(few, -0.0, 0.0)
        return torch.where(torch.rand(1, 1, 1, N, generator=g) < 0.5, s, -torch.rand(1, 1, 1, N, generator=g))
    return torch.full((1, 1, 1, N), 0.25)


@pytest.mark.parametrize("what,k", [("zeros", 13000), ("window", 13000), ("two", 13000), ("between", 13000), ("top", 4000), ("top", 40000),
                                    ("negative", 66000), ("constant", 100), ("constant", 13000)])
def test_values_that_repeat_next_to_the_threshold(lib, what, k):
    """One part per row: the scores are read once (with the sample and what the waves ask for past the end 1.36 times),
    whatever values repeat and however often. Several parts: the same lists."""
    N = 131072
    lib.emu_schedule(1, -1, -1)
    for bf16 in (False, True):
        s = repeated(what, N, k, k)
        s = s.to(torch.bfloat16) if bf16 else s
        lib.sts_set_knob(3, 5.0)
        lib.emu_loaded()
        try:
            for budget in (k, k - k // 50, k + k // 50):
                check(lib, s, [0], budget, lens=[N - 13])
                assert lib.emu_loaded() <= 1.5 * N * s.element_size()
        finally:
            lib.sts_set_knob(3, float("nan"))
        check(lib, s, [0, 0], k)
        check(lib, s[..., :40001].contiguous(), [0], k // 4, lens=[39999])


@pytest.mark.parametrize("levels,one_part", [(0, False), (5, False), (0, True), (5, True)])
def test_bands_that_lie_in_one_part(lib, levels, one_part):
    """All tokens around the threshold next to each other, more than a part's list holds: that part reads its own
    tokens again, once, or, where the excess is one value, once per histogram; the others are done."""
    # one part of 512K tokens, or the two rows with tokens of 64, cut into four parts of 64K
    B, N, k, first, heavy = (1, 524288, 60000, 140000, 100000) if one_part else (64, 262144, 45000, 66000, 60000)
    lens = [N - 5, N] + [0] * (B - 2) if B > 1 else [N - 5]
    g = torch.Generator().manual_seed(levels)
    s = torch.rand(1, 1, 1, N, generator=g) * 1e-3
    s[..., first:first + heavy] = 1.0 + (torch.randint(1, levels + 1, (heavy,), generator=g) / levels if levels else torch.rand(heavy, generator=g))
    s = s.expand(B, 1, 1, N).contiguous()
    lib.emu_schedule(1, 1, 3)
    lib.sts_set_knob(3, 5.0 if one_part else 0.0)
    lib.emu_loaded()
    try:
        check(lib, s, [0], k, lens=lens)
    finally:
        lib.sts_set_knob(3, float("nan"))
    read = lib.emu_loaded() / (4 * N * min(B, 2))
    assert read < (2.5 if one_part else 2.2) + 3.0 * (levels > 0), read


def by_keys(scores, n, k):
    """The kept tokens of one row of scores of any bits: ascending, the largest of the order-preserving keys, ties to the lower token."""
    if scores.dtype == torch.bfloat16:
        u = scores.view(torch.int16).numpy().astype(np.int64) << 16 & 0xffffffff
    else:
        u = scores.view(torch.int32).numpy().astype(np.int64) & 0xffffffff
    key = np.where(u == 0x80000000, 0x80000000, np.where(u >> 31, u ^ 0xffffffff, u | 0x80000000))[:n]
    return np.sort(np.argsort(-key, kind="stable")[:k])


def check_keys(lib, live, rows, k, lens):
    """live [R,N] in a call of that many rows, the others empty."""
    s = torch.zeros(rows, 1, 1, live.shape[1], dtype=live.dtype)
    s[:len(live), 0, 0] = live
    idx, cnt = select(lib, s, [0], k, lens=lens + [0] * (rows - len(live)))
    for b, n in enumerate(lens):
        assert cnt[b, 0] == min(k, n)
        np.testing.assert_array_equal(idx[b, 0, :cnt[b, 0]], by_keys(live[b], n, k), err_msg=f"row {b}, length {n}")


# 1024 threads with one quad, two, four and eight; 256 threads with four, eight and sixteen; 512
ROW_FORMS = [(16, 4001), (16, 8190), (256, 9000), (256, 20001), (513, 4090), (513, 8190), (513, 9001), (513, 20001)]


@pytest.mark.parametrize("rows,N", ROW_FORMS)
@pytest.mark.parametrize("n", [1000, 2051])
def test_highest_keys_of_all(lib, rows, N, n):
    """The threshold next to the highest key there is, 0xffffffff: the keys of its bin do not run past it. Rows below 1024
    tokens are not sampled, their window is every key."""
    lib.emu_schedule(1, -1, -1)
    s = torch.rand(3, N, generator=torch.Generator().manual_seed(n))
    bits = s.view(torch.int32)
    bits[0, 500] = 0x7fffffff
    bits[1, 500:503] = 0x7fffffff
    bits[2, 100:800:100] = torch.tensor([0x7fffffff, 0x7fff0000, 0x7ffffffe, 0x7f800000, 0x7fffffff, 0x7fe00000, 0x7fefffff], dtype=torch.int32)
    bits[2, 5:900:200] = torch.tensor([-1, -2, -0x200000, -3, -0x100000], dtype=torch.int32)       # ... and the lowest
    for k in (1, 3, 6, 990):
        check_keys(lib, s, rows, k, [n, n, n])


@pytest.mark.parametrize("rows,N", ROW_FORMS)
def test_lowest_keys_of_all(lib, rows, N):
    """The threshold next to the lowest key there is, 1: a bin that begins there does not count the positions after the
    row's end, which hold key 0 and are not listed, whatever the list's memory holds."""
    lib.emu_schedule(1, -1, -1)
    lib.emu_lds(0x101)
    try:
        for n in (1000, 1021, 2047, 4081, 8129, N - 3):
            if n > N:
                continue
            s = torch.rand(3, N, generator=torch.Generator().manual_seed(n))
            bits = s.view(torch.int32)
            bits[0, 700:705] = torch.tensor([-2, -0x200000, -9, -0x100, -3], dtype=torch.int32)
            bits[1, 5:990:98] = -9
            bits[2, 0:900:2] = -0x7f0000 - torch.arange(450, dtype=torch.int32)            # many below all other scores
            for k in (n - 1, n - 3, n - 9, n - 400):
                check_keys(lib, s, rows, k, [n, n, n])
    finally:
        lib.emu_lds(0)


@pytest.mark.parametrize("rows,Tq,N,bf16", [
    (16, 5, 4001, False), (16, 3, 8190, True), (256, 2, 9000, False), (256, 9, 20001, False), (256, 2, 32768, True),
    (513, 1, 4090, False), (513, 2, 8190, False), (513, 1, 9001, False), (513, 3, 20001, True),
    (3, 1, 4099, True), (3, 1, 16384, True), (3, 1, 32765, True), (3, 1, 65536, True), (3, 1, 131071, True),       # packed in registers
])
def test_scores_past_the_valid_length_are_not_read(lib, rows, Tq, N, bf16):
    """A row that is an eighth full, in a tensor that is allocated for the longest sequence."""
    lib.emu_schedule(1, -1, -1)
    n = N // 8 - 3
    s = torch.zeros(rows, 1, Tq, N)
    s[:2] = softmax(2, 1, Tq, N, N)
    s = s.to(torch.bfloat16) if bf16 else s
    lib.emu_loaded()
    check(lib, s, [0], N // 20, lens=[n, n] + [0] * (rows - 2))
    assert lib.emu_loaded() <= 0.6 * 2 * Tq * N * s.element_size()


@pytest.mark.parametrize("rows,Hq,Tq,N,k,bf16,one", [
    (1, 1, 1, 131072, 13107, True, True), (1, 1, 1, 131072, 65536, True, False), (1, 64, 1, 131072, 60000, True, False), (1, 32, 1, 131072, 13107, True, False),
    (1, 2, 1, 65536, 32768, True, True), (1, 8, 1, 65536, 32768, True, False), (120, 256, 1, 131072, 13107, True, True), (4096, 64, 1, 65536, 32768, True, True),
    (1, 256, 1, 8192, 8192, True, True),
    (8, 8 * 2, 5, 32768, 3277, False, True), (8, 8 * 8, 5, 32768, 16384, False, False), (8, 8 * 2, 1, 32768, 16384, False, True),
    (8, 8 * 32, 1, 32768, 16384, False, False), (8, 8 * 32, 5, 32768, 3277, False, True), (8, 8 * 32, 1, 16384, 8192, False, False),
    (8, 8 * 8, 1, 16384, 8192, False, True), (8, 8 * 32, 1, 9000, 4500, False, False), (255, 2, 1, 20000, 10000, False, True),
])
def test_rows_whose_lists_one_workgroup_would_write_for_long(lib, rows, Hq, Tq, N, k, bf16, one):
    """Few rows with long lists, or a list for each of many target heads, are cut into parts that share the writing."""
    Hd = 8 if rows % 8 == 0 and Hq > 2 else 1
    got = route(lib, rows // Hd, Hd, Tq, N, max(Hq, Hd), k, bf16=bf16)
    assert got.startswith("select_row" if one else "select_clear16_kernel select_sampled_kernel"), got


@pytest.mark.parametrize("rows,blocks,kernel", [
    (6, 2048, "select_small_kernel<true>"), (6, 2049, "short_select_blocks_kernel<1024, 1>"), (6, 8192, "short_select_blocks_kernel<1024, 2>"),
    (6, 16384, "select_blocks_kernel<1024, 4>"), (513, 2049, "short_select_blocks_kernel<256, 4>"), (513, 8192, "select_blocks_kernel<256, 8>"),
    (513, 16384, "select_blocks_kernel<256, 16>"),
])
def test_kernels_that_rank_block_sums(lib, rows, blocks, kernel):
    """Rows of scores do not look at the page's size: their kernels are others."""
    assert route(lib, rows, 1, 1, 8 * blocks, 2, 100, page=8, lens=True).endswith(" " + kernel)
    if blocks <= 8192:
        assert route(lib, rows, 1, 1, blocks, 2, 100, lens=True).startswith(("short_select_row_kernel", "select_row_kernel"))


@pytest.mark.parametrize("budget", [28712, 28000, 30000, 26000])
def test_one_heavy_value_at_the_bands_upper_edge(lib, budget):
    """A value that much of the row shares at the upper edge of the band, none at the lower one, and many tokens in
    between: the list does not run into the bits of the heavy value's tokens."""
    N, n, rows = 131907, 34394, 130
    s = torch.zeros(rows, 1, 1, N)
    s[0, 0, 0, :n] = torch.round(torch.randn(n, generator=torch.Generator().manual_seed(7)) * 2) / 4
    lib.emu_schedule(1, -1, -1)
    check(lib, s, [0], 53920, k_head=[budget], lens=[n] + [0] * (rows - 1))


@pytest.mark.parametrize("budget", [36294, 35931])
def test_bins_that_run_past_the_band(lib, budget):
    """A band that begins at the lowest key and overflows the list: the bin of the threshold reaches beyond its upper edge,
    and the tokens above that, which are kept already, are not counted again when the part's tokens are."""
    N, rows = 36294, 130
    g = torch.Generator().manual_seed(35)
    base = float(0.5 + torch.rand(1, generator=g) * 0.4)
    s = torch.zeros(rows, 1, 1, N)
    s[0, 0, 0] = base * torch.exp(torch.softmax(2 * torch.randn(N, generator=g), -1).to(torch.bfloat16).float())
    lib.emu_schedule(1, -1, -1)
    check(lib, s, [0], N, k_head=[budget], lens=[N] + [0] * (rows - 1))


@pytest.mark.parametrize("order", ["ascending", "falling"])
@pytest.mark.parametrize("N", [32768, 32769, 65537, 100000, 131072, 131073])
def test_union_of_lists_of_every_length(lib, N, order):
    """One to five chunks of 32768 tokens: the searches for the ends of each list's segments, side by side, in lists around the
    64 entries of a probe, lists without one and lists that lie in one chunk alone."""
    lib.emu_schedule(N, -1, -1)
    rng = np.random.default_rng(N)
    Tq, k, lengths = 16, 4500, [0, 1, 2, 63, 64, 65, 127, 128, 129, 700, 4095, 4096, 4097, 4500, 100, 90]
    sel = np.full((1, 1, Tq, k), -1, np.int32)
    for i, n in enumerate(lengths):
        low, high = (N - 1 - n, N) if i == 14 else (0, n) if i == 15 else (0, N)
        row = np.sort(rng.choice(np.arange(low, high), size=n, replace=False))
        sel[0, 0, i, :n] = row[::-1] if order == "falling" and i == 9 else row
    cnt = np.asarray(lengths, np.int32).reshape(1, 1, Tq)
    hm, pitch = np.zeros(2, np.int32), 20000
    idx, mask, ucnt = np.full((1, 2, pitch), -7, np.int32), np.full((1, 2, pitch), 7, np.uint16), np.full((1, 2), -7, np.int32)
    p = binding.UnionParams(B=1, Hd=1, Hq=2, Tq=Tq, N=N, k=k, row_indices=sel.ctypes.data, row_counts=cnt.ctypes.data, head_map=hm.ctypes.data,
                            pitch=pitch, indices=idx.ctypes.data, row_mask=mask.ctypes.data, counts=ucnt.ctypes.data)
    assert lib.sts_union_rows(ctypes.byref(p), None) == 0
    o_idx, o_mask, o_cnt = oracle.union_rows(sel, cnt, hm.tolist(), pitch=pitch)
    np.testing.assert_array_equal(ucnt, o_cnt)
    np.testing.assert_array_equal(idx, o_idx)
    np.testing.assert_array_equal(mask, o_mask)
