"""The counter summary's hash covers every source of the kernels it describes."""
import os
import re

import bench

CSRC = os.path.join(os.path.dirname(os.path.abspath(bench.__file__)), "paper_2108_12188_amd",
                    "csrc")


def test_hash_covers_the_included_headers():
    todo, seen = [f for f in bench.COUNTER_SOURCES if f.endswith(".hip")], set()
    while todo:
        f = todo.pop()
        if f in seen:
            continue
        seen.add(f)
        with open(os.path.join(CSRC, f)) as fh:
            todo += re.findall(r'^#include "(sem_\w+\.h)"', fh.read(), re.M)
    assert seen <= set(bench.COUNTER_SOURCES)
