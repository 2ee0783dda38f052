"""The kernels in which one wavefront hands values from lane to lane through LDS without a barrier: a fence stands at every
hand-over.  A missing one shows only if the compiler happens to move an access, so the source's own order of stores, fences
and loads is looked at, in the compiler's code before any optimisation."""
import os
import re
import subprocess

import pytest

from paper_2601_17702_amd import build


def wavefront_fences(src: str) -> dict:
    """Fences per kernel of csrc/<src>, helpers inlined by hand: every call of a function adds that function's fences."""
    flags = [f for f in build.FLAGS if f != "-O3"]
    ir = subprocess.run(["hipcc", *flags, "-O1", "-Xclang", "-disable-llvm-passes", "-S", "-emit-llvm", "--cuda-device-only",
                         os.path.join(build.CSRC, src), "-o", "-"], check=True, stdout=subprocess.PIPE, stderr=subprocess.DEVNULL,
                        text=True).stdout
    own, calls, kernels = {}, {}, []
    for m in re.finditer(r"^define ([^\n]*?)@([\w.$]+)\([^\n]*\{\n(.*?)^\}", ir, re.S | re.M):
        own[m.group(2)] = len(re.findall(r'fence syncscope\("wavefront"\)', m.group(3)))
        calls[m.group(2)] = re.findall(r"call [^\n]*?@([\w.$]+)\(", m.group(3))
        if "amdgpu_kernel" in m.group(1):
            kernels.append(m.group(2))

    def total(f):
        return own.get(f, 0) + sum(total(c) for c in calls.get(f, []) if c in own)
    return {f: total(f) for f in kernels}


@pytest.mark.parametrize("src,kernel,least", [
    ("select.hip", "sel_nms_kernel", 3),       # before the tiles are read again, before and after their new maxima
    ("select.hip", "sel_nms_long_kernel", 3),
    ("score.hip", "sc_topb_long_kernel", 3),  # behind the cleared tiles, before and behind the new maxima
])
def test_greedy_searches_fence_their_hand_overs(src, kernel, least):
    found = {f: n for f, n in wavefront_fences(src).items() if kernel in f}
    assert found and all(n >= least for n in found.values()), found
