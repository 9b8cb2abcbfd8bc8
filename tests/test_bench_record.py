"""CPU: what bench.py records."""
import os
import re

import bench

CSRC = os.path.join(bench.ROOT, "paper_1412_2293_amd", "csrc")


def test_profile_key_covers_every_file_of_the_profiled_kernels():
    """The stored counters count as those of the current build only while every file that the fused passes'
    kernels are compiled from is unchanged, headers included."""
    seen, todo = set(), ["fused.hip", "fused_c64.hip", "expand.hip"]
    while todo:
        f = todo.pop()
        if f in seen:
            continue
        seen.add(f)
        text = open(os.path.join(CSRC, f)).read()
        todo += [g for g in re.findall(r'#include "([^"]+)"', text) if os.path.exists(os.path.join(CSRC, g))]
    assert seen <= set(bench.PROFILED_SOURCES)
