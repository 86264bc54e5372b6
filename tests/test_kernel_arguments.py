"""Kernels read their arguments where they use them, through the kernel argument segment's
address, which means something only in a kernel's own body.  Every device function that
asks for it, or calls one that does, is therefore one that the compiler always inlines,
whatever it does with the others: checked in the compiler's output before any inlining.
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2510_18221_amd import build as eco_build

NAME = r'(@(?:"[^"]+"|[\w.$]+))\('
SEGMENT = "@llvm.amdgcn.kernarg.segment.ptr"


def functions(text):
    """{name: (is a kernel, always inlined, names it calls)} of the definitions of an LLVM module."""
    always = {g for g, body in re.findall(r"^attributes (#\d+) = \{(.*)\}$", text, re.M) if "alwaysinline" in body}
    out = {}
    for head, body in re.findall(r"^define ([^\n]*)\{\n(.*?)^\}", text, re.M | re.S):
        name = re.search(NAME, head).group(1)
        calls = set(re.findall("call [^\n]*?" + NAME, body))
        out[name] = ("amdgpu_kernel" in head, bool(always & set(re.findall(r"#\d+", head))), calls)
    return out


@pytest.mark.skipif(shutil.which(eco_build.HIPCC) is None, reason="needs hipcc")
@pytest.mark.parametrize("unit", [u for u in eco_build._units() if u[0].endswith(".hip")], ids=lambda u: os.path.basename(u[1]))
def test_segment_address_only_in_kernels(tmp_path, unit):
    src, _, flags = unit
    ll = str(tmp_path / "unit.ll")
    subprocess.run([eco_build.HIPCC] + eco_build.COMMON + flags +
                   ["-w", "--offload-device-only", "-emit-llvm", "-S", "-Xclang", "-disable-llvm-passes", src, "-o", ll],
                   check=True)
    with open(ll) as f:
        fns = functions(f.read())
    users, known = set(), {SEGMENT}
    while True:   # the functions that ask for the address, and their callers
        more = {n for n, (_, _, calls) in fns.items() if calls & known} - users
        if not more:
            break
        users |= more
        known |= more
    assert any(fns[n][0] for n in users), "a kernel reads its arguments so"
    assert not [n for n in users if not (fns[n][0] or fns[n][1])]
