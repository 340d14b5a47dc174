"""Lanes of a wave that exchange values through LDS order their accesses with
a fence at wavefront scope and a wave barrier.  The barrier alone orders no
memory: the compiler may move loads and stores across it.  Every wave barrier
in the kernels therefore stands right after such a fence."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2001_09792_amd", "csrc")
FENCE = '__builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");'


def test_wave_barriers_follow_a_fence():
    seen = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        code = [re.sub(r"//.*", "", line).strip() for line in open(path)]
        code = [line for line in code if line]
        for k, line in enumerate(code):
            if "__builtin_amdgcn_wave_barrier" in line:
                seen += 1
                assert line == "__builtin_amdgcn_wave_barrier();" and code[k - 1] == FENCE, (path, line)
    assert seen >= 2
