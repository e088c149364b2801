"""Which sparse attention calls gather from a cache that their batch elements share by workgroups placed by die: the host's
rule, by the kernels that it launches (the library compiled for the CPU, nothing is run), at its lines."""
import ctypes

import numpy as np
import pytest

from paper_2605_15508_amd import binding
from test_select_emulated import lib  # noqa: F401  (lib: the emulated library, a fixture)


def launches(lib, B, Tq, Hq, Hkv, d, N, k, Hd, stride_b=0, page=1):
    hm = np.arange(Hq, dtype=np.int32) * Hd // Hq
    at = 1 << 20
    p = binding.AttnParams(B=B, Tq=Tq, Hq=Hq, Hkv=Hkv, d=d, N=N, q=at, k=at, v=at, kv_stride_b=stride_b, kv_stride_h=N * d, kv_stride_n=d, indices=at,
                           kmax=k, head_map=hm.ctypes.data, scale=0.09, out=at, out_dtype=0, page_size=page, workspace=at)
    lib.sts_attn_workspace_bytes.restype = ctypes.c_size_t
    p.workspace_bytes = lib.sts_attn_workspace_bytes(ctypes.byref(p), 1)
    lib.emu_only_names(1)
    try:
        assert lib.sts_sparse_attn(ctypes.byref(p), None) == 0
        return lib.emu_names().decode()
    finally:
        lib.emu_only_names(0)


@pytest.mark.parametrize("B,Tq,d,N,k,Hd,shared", [
    (16, 16, 128, 65536, 6554, 16, True), (16, 5, 128, 131072, 13107, 16, True), (2, 5, 128, 32768, 655, 16, True),
    (1, 5, 128, 32768, 3277, 16, False),
    # rows of a cache beyond the caches, asked for 0.4, 0.6 and 0.64 times; what fits the caches, asked for once or never
    (2, 5, 128, 1000000, 100000, 16, False), (3, 5, 128, 500000, 50000, 16, False), (16, 5, 128, 500000, 10000, 16, True),
    (2, 5, 128, 262144, 25601, 16, False), (2, 5, 128, 262144, 25600, 16, True), (4, 5, 128, 1000000, 20000, 16, False),
    (2, 5, 64, 262144, 51200, 16, True), (2, 5, 64, 1000000, 52000, 16, False),
    # eight waves: more than eight tiles a workgroup, and rows asked for 0.25 times
    (16, 16, 128, 4096, 256, 16, False), (16, 16, 128, 4096, 257, 16, True), (2, 16, 128, 4096, 600, 16, False), (2, 16, 128, 16384, 1200, 16, False), (4, 16, 128, 16384, 1200, 16, True),
    (4, 16, 128, 16384, 2400, 16, True), (16, 16, 128, 131072, 1023, 16, False), (16, 16, 128, 131072, 1024, 16, True),
    (2, 16, 64, 4096, 100, 16, True), (4, 16, 128, 4096, 600, 8, True),
])
def test_rule(lib, B, Tq, d, N, k, Hd, shared):  # noqa: F811
    got = launches(lib, B, Tq, 32, 8, d, N, k, Hd)
    assert got.split(" attn_combine")[0] == ("attn_split shared" if shared else "attn_split")
    assert "shared" not in launches(lib, B, Tq, 32, 8, d, N, k, Hd, stride_b=8 * N * d)


def test_blocks_count_their_tokens(lib):  # noqa: F811
    assert "shared" in launches(lib, 16, 16, 32, 8, 128, 4096, 33, 16, page=8)
    assert "shared" not in launches(lib, 16, 16, 32, 8, 128, 4096, 32, 16, page=8)
    assert "shared" not in launches(lib, 65536 // 2 + 1, 5, 32, 8, 128, 4096, 100, 16)
