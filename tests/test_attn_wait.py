"""The attention over a shared cache loads K straight to LDS (attn_split_kernel with two query tiles at head size 128 in
csrc/attn.hip), where the compiler adds no wait: the kernel waits by the number of loads that it sends after a
tile's K. Whether that is the number of loads in the compiled loop is looked at here, in the code of the last build."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2605_15508_amd import build

OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"
# with and without row bits
KERNELS = {"attn_split_kernelILi128ELi2ELb1ELb0ELb0ELb1ELb1E": 2, "attn_split_kernelILi128ELi2ELb1ELb0ELb0ELb0ELb1E": 1}


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    if not os.path.exists(OBJDUMP):
        pytest.skip("llvm-objdump not available")
    obj = os.path.join(os.path.dirname(build.RESOURCES), "attn.o")
    if not os.path.exists(obj) or build.needs_build():
        build.build(force=True)
    tmp = tmp_path_factory.mktemp("attn")
    shutil.copy(obj, tmp / "attn.o")
    subprocess.run([OBJDUMP, "--offloading", "attn.o"], cwd=tmp, check=True, capture_output=True)
    code = [f for f in os.listdir(tmp) if "gfx950" in f]
    assert len(code) == 1
    return subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", str(tmp / code[0])], check=True, capture_output=True, text=True).stdout


def body(listing, kernel):
    at = re.search(rf"^<\w*{kernel}\w*>:$", listing, re.M)
    assert at, kernel
    end = re.search(r"^<\w+>:$", listing[at.end():], re.M)
    return listing[at.end():at.end() + end.start()] if end else listing[at.end():]


def loads_and_waits(text, behind):
    """K: a load to LDS, V: a load of 16 bytes, E: of 4 or 2, O: any other access to memory, W: the wait that leaves `behind`
    loads under way, in the order of the code."""
    seq = []
    for line in text.splitlines():
        op = line.split("//")[0].strip()
        if op.startswith("buffer_load") and op.endswith(" lds"):
            seq.append("K")
        elif op.startswith("global_load_dwordx4"):
            seq.append("V")
        elif re.match(r"global_load_(dword|ushort) ", op):
            seq.append("E")
        elif re.match(r"(buffer|global|flat|scratch)_", op):
            seq.append("O")
        elif re.match(rf"s_waitcnt vmcnt\({behind}\)", op):
            seq.append("W")
    return "".join(seq)


def is_ordered(seq, entries):
    """The first tile's K and V, then twice in the loop: entries, the next tile's K and V, the wait."""
    first, half = "K" * 8 + "V" * 8, "E" * entries + "K" * 8 + "V" * 8 + "W"
    return seq.count("W") == 2 and first + 2 * half in seq


@pytest.mark.parametrize("kernel,entries", KERNELS.items())
def test_the_wait_counts_the_loads_behind_k(listing, kernel, entries):
    text = body(listing, kernel)
    assert is_ordered(loads_and_waits(text, 24 + entries), entries)
    # and the reads of a tile's K come after it: between a half's loads and its wait nothing is read from LDS in chunks of K
    for half in re.findall(rf"buffer_load_dwordx4 [^\n]* lds.*?s_waitcnt vmcnt\({24 + entries}\)", text, re.S):
        last = half[half.rindex(" lds"):]
        assert "ds_read_b128" not in last and "ds_load_b128" not in last


@pytest.mark.parametrize("seq", ["E" * 2 + "K" * 8 + "V" * 8 + "W" + "E" + "K" * 8 + "V" * 8 + "W",       # an entry's load less
                                 2 * ("E" * 2 + "K" * 8 + "V" * 7 + "W"),                               # V in fewer loads
                                 2 * ("K" * 8 + "E" * 2 + "V" * 8 + "W"),                               # entries after K
                                 "E" * 2 + "K" * 8 + "V" * 8 + "W"])                                     # one half of the loop
def test_fewer_or_other_loads_are_found(seq):
    assert is_ordered("K" * 8 + "V" * 8 + 2 * ("E" * 2 + "K" * 8 + "V" * 8 + "W"), 2)
    assert not is_ordered("K" * 8 + "V" * 8 + seq, 2)
