"""The memory traffic that bench.py reports for its timed kernel holds for one source: the tag covers every file the kernel is
built from."""
import os
import re

import bench

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1802_07170_amd", "csrc")


def test_the_tag_covers_the_timed_kernel_s_file_and_all_that_it_includes():
    seen, todo = set(), ["loop.hip"]
    while todo:
        name = todo.pop()
        if name not in seen:
            seen.add(name)
            with open(os.path.join(CSRC, name)) as f:
                todo += re.findall(r'^#include "([^"]+)"', f.read(), re.M)
    assert seen == set(bench.LOOP_KERNEL_SOURCES)
