"""Every LDS array is read and written as one type, or as types that may alias: the compiler takes accesses of different
scalar types as unrelated and may move one past the other, also between two barriers. Host-only: reads the type tags of the
accesses in the compiler's intermediate code, before it optimises."""
import os
import re
import subprocess

import pytest

from paper_2605_15508_amd import build

GLOBAL = re.compile(r"@(_ZZN\S+?) = internal addrspace\(3\) global")
DEFINE = re.compile(r"^define .*@(\S+?)\(")
NAMES = re.compile(r"[%@][\w.$]+")
TAG = re.compile(r"!tbaa !(\d+)")


def access_types(text):
    """{LDS array: {type name: how many accesses}}"""
    meta = dict(re.findall(r"^!(\d+) = (.*)$", text, re.M))

    def type_name(tag):
        node = re.findall(r"!(\d+)", meta[tag])[1]                   # {base type, access type, offset}
        return re.search(r'!"([^"]*)"', meta[node]).group(1)

    lds = set(GLOBAL.findall(text))
    found = {}
    root = {}
    for ln in text.splitlines():
        if ln.startswith("define"):
            root = {}                                                # value -> the LDS array it points into
            continue
        if "@_ZZN" not in ln and not (root and ln.startswith("  ")):
            continue

        def of(part):
            for v in NAMES.findall(part):
                if v[0] == "@" and v[1:] in lds:
                    return v[1:]
                if v in root:
                    return root[v]
            return None

        m = re.match(r"  (%[\w.]+) = (\w+)( .*)", ln)
        if m and m.group(2) in ("getelementptr", "addrspacecast", "bitcast"):
            src = re.search(r"ptr(?: addrspace\(\d\))? (.*)", m.group(3))
            if src and of(src.group(1)):
                root[m.group(1)] = of(src.group(1).split(", i")[0])
        m = re.match(r"  store ptr (.*), ptr (?:addrspace\(5\) )?(%[\w.]+),", ln)
        if m and of(m.group(1)):
            root[m.group(2)] = ("pointer", of(m.group(1)))           # a pointer variable
            continue
        m = re.match(r"  (%[\w.]+) = load ptr, ptr (?:addrspace\(5\) )?(%[\w.]+),", ln)
        if m and isinstance(root.get(m.group(2)), tuple):
            root[m.group(1)] = root[m.group(2)][1]
            continue
        m = re.match(r"  %[\w.]+ = load [^,]*, ptr (.*?), align", ln) or re.match(r"  store .*?, ptr (.*?), align", ln)
        tag = TAG.search(ln)
        if m and tag and isinstance(of(m.group(1)), str):
            per = found.setdefault(of(m.group(1)), {})
            per[type_name(tag.group(1))] = per.get(type_name(tag.group(1)), 0) + 1
    return found


@pytest.mark.parametrize("src,seen", [("attn.hip", "lds_bits"), ("select_row.hip", "codes"), ("select.hip", ""), ("select_sampled.hip", ""),
                                      ("union.hip", ""), ("headmap.hip", "")])
def test_lds_arrays_are_accessed_as_one_type(src, seen, tmp_path):
    out = tmp_path / "x.ll"
    subprocess.run([build._hipcc(), "--offload-arch=gfx950", "--cuda-device-only", "-std=c++17", "-O3", "-w", "-Xclang", "-disable-llvm-passes",
                    "-S", "-emit-llvm", "-o", str(out), os.path.join(build.CSRC, src)], check=True)
    types = access_types(out.read_text())
    assert any(seen in k for k in types)
    bad = {k: v for k, v in types.items() if len(set(v) - {"omnipotent char"}) > 1}
    assert not bad, bad
