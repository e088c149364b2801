"""The attention over a shared cache loads K straight to LDS (attn_split_kernel with two query tiles at head size 128 in
csrc/attn.hip). Nothing in the source orders these loads before K's reads: the compiler puts in a wait for all but the loads that
go out after them, if it sees that both are of one array. Whether it did is looked at here, in the code of the last build."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2605_15508_amd import build

OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"
# with and without row bits: a load of an entry and one of its bits, or the first alone
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


def accesses(text):
    """K: a load to LDS, V: a load of 16 bytes, E: of 4 or 2, O: any other access to memory, R: a read of 16 bytes from LDS, (n): a wait
    that leaves n loads under way, P: a matrix product; in the order of the code."""
    seq = []
    for line in text.splitlines():
        op = line.split("//")[0].strip()
        wait = re.match(r"s_waitcnt .*vmcnt\((\d+)\)", op)
        if op.startswith("buffer_load") and op.endswith(" lds"):
            seq.append("K")
        elif op.startswith("global_load_dwordx4"):
            seq.append("V")
        elif re.match(r"global_load_(dword|ushort) ", op):
            seq.append("E")
        elif re.match(r"(buffer|global|flat|scratch)_", op):
            seq.append("O")
        elif op.startswith("ds_read_b128"):
            seq.append("R")
        elif op.startswith("v_mfma"):
            seq.append("P")
        elif wait:
            seq.append(f"({wait.group(1)})")
    return "".join(seq)


def is_ordered(seq, entries):
    """From the loop's list entries on: the row offsets (two reads), a wait that leaves V's eight loads and the entries under way at most,
    the reads of K and Q with their products, and, behind the last product, the loads of the next tile's K."""
    if seq.count("K" * 8) != 2 or seq.count("K") != 16:
        return False
    body = seq[:seq.rindex("K" * 8)].rpartition("E" * entries)[2]
    m = re.fullmatch(r"R{0,2}\((\d+)\)((?:R+P+)+)", body)
    return bool(m) and int(m.group(1)) <= 8 + entries and m.group(2).count("P") == 16 and m.group(2).count("R") >= 8


@pytest.mark.parametrize("kernel,entries", KERNELS.items())
def test_k_is_waited_for(listing, kernel, entries):
    assert is_ordered(accesses(body(listing, kernel)), entries)


LOOP = "RR(10)" + 4 * "RRRRPPPP"


@pytest.mark.parametrize("seq", [LOOP.replace("(10)", ""), LOOP.replace("(10)", "(11)"),       # no wait, or one that leaves a load of K under way
                                 "RRR" + LOOP[2:],                                             # K read before it
                                 LOOP[:-4] + "KKKKKKKK" + LOOP[-4:]])                          # the next K before the last products
def test_reads_and_loads_out_of_order_are_found(seq):
    start = "EEVVVVKKKKKKKKVVVVVVVVEE"
    assert is_ordered(start + LOOP + "KKKKKKKK", 2)
    assert not is_ordered(start + seq + "KKKKKKKK", 2)
