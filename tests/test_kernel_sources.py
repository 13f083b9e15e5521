"""CPU checks of the kernel sources, for faults that must not first show on a
GPU.  A direct-to-LDS load is in flight until the wave that issued it has
waited for it, and a barrier alone does not make a wave wait: a kernel that
stages LDS this way hands its stages over with stage_wait, which waits for the
wave's own loads before the barrier."""
import glob
import os
import re

from paper_2510_26843_amd import build


def _kernels():
    for path in sorted(glob.glob(os.path.join(build.CSRC, "*.hip"))):
        src = re.sub(r"//[^\n]*", "", open(path).read())
        for m in re.finditer(r"__global__ void [^;{]*?\b(k_\w+)\(", src):
            depth, i = 0, src.index("{", m.end())
            start = i
            while True:
                depth += {"{": 1, "}": -1}.get(src[i], 0)
                i += 1
                if depth == 0:
                    break
            yield m.group(1), src[start:i]


def test_direct_to_lds_stages_are_waited_for():
    seen = []
    for name, body in _kernels():
        if "lds_load16" in body:
            seen.append(name)
            assert "__syncthreads" not in body and "s_barrier" not in body, name
            assert "stage_wait<" in body, name
    assert {"k_gemm_rows", "k_attn_causal"} <= set(seen), seen
