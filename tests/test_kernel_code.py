"""CPU checks of the built gfx950 code.  The small kernels between the GEMMs
(norm, split merge) are latency: a scalar load, its wait and a branch in front
of their first loads cost 0.28 us of each launch, 97 launches in a 7B verify."""
import os
import re
import struct
import subprocess

import pytest

from paper_2510_26843_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects():
    data = open(build.LIB, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        o = at + len(MAGIC) + 8
        for _ in range(struct.unpack_from("<Q", data, o - 8)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, o)
            if b"gfx950" in data[o + 24:o + 24 + n]:
                yield data[at + off:at + off + size]
            o += 24 + n
        at = data.find(MAGIC, at + 1)


@pytest.mark.skipif(not os.path.exists(OBJDUMP) or not os.path.exists(build.LIB), reason="no disassembler or library")
# (the merge has one uniform branch, around its loop over the splits)
@pytest.mark.parametrize("kernel,branches", [("k_rmsnorm", 0), ("k_attn_merge", 1)])
def test_latency_kernels_load_before_they_branch(kernel, branches, tmp_path):
    path = tmp_path / "code.o"
    path.write_bytes(max(_code_objects(), key=len))
    names = subprocess.run([OBJDUMP, "--syms", str(path)], capture_output=True, text=True, check=True).stdout
    syms = re.findall(r"F \.text\s+\S+ (?:\.\w+ )?(_ZN3cas\d+%sI\S+)" % kernel, names)
    assert syms
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--disassemble-symbols=" + ",".join(syms), str(path)],
                          capture_output=True, text=True, check=True).stdout
    bodies = re.split(r"\n[0-9a-f]+ <(_ZN\w+)>:\n", text)[1:]
    assert len(bodies) == 2 * len(syms)
    for name, body in zip(bodies[::2], bodies[1::2]):
        assert body[:body.index("global_load")].count("s_cbranch_scc") <= branches, name
