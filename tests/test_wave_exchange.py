"""LDS values that lanes of one wave hand to each other: the wave barrier orders
instructions only, so each stands between a release and an acquire fence
(common.h: wave_exchange) or behind a block fence."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_17978_amd", "csrc")
FENCE = re.compile(r"__threadfence_block\(\)|__builtin_amdgcn_fence\(__ATOMIC_RELEASE")


def test_wave_barriers_are_fenced():
    found = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h*"))):
        with open(path) as fh:
            lines = fh.read().split("\n")
        for at, line in enumerate(lines):
            if "__builtin_amdgcn_wave_barrier()" in line:
                found += 1
                assert FENCE.search(lines[at - 1]), f"{os.path.basename(path)}:{at + 1}"
    assert found
