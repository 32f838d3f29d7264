"""A barrier builtin by itself does not keep the compiler from moving a memory
access across it: the device code uses __syncthreads or the helpers that put
fences, or at least memory clobbers, around it."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1505_04340_amd", "csrc")


def test_every_barrier_is_fenced():
    found = []
    for f in sorted(os.listdir(CSRC)):
        with open(os.path.join(CSRC, f)) as h:
            lines = h.read().splitlines()
        for i, line in enumerate(lines):
            if re.search(r"__builtin_amdgcn_s_barrier\s*\(", line):
                found.append((f, lines[i - 1].strip(), lines[i + 1].strip()))
    assert found, "no barrier found: the pattern is out of date"
    clobber = 'asm volatile("" ::: "memory");'
    for f, before, after in found:
        if (before, after) == (clobber, clobber):
            continue
        assert before.startswith("__builtin_amdgcn_fence(__ATOMIC_RELEASE"), (f, before)
        assert after.startswith("__builtin_amdgcn_fence(__ATOMIC_ACQUIRE"), (f, after)
