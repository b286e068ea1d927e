"""Committed traffic figures count as current only while their sources are unchanged: the digest covers
every file that the tile passes and the planner are compiled from."""
import os
import re
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2406_17248_amd", "csrc")


def test_digest_covers_the_sources_of_the_passes():
    sys.path.insert(0, ROOT)
    import bench
    todo, seen = ["tile_rb.hip", "engine.cpp", "api.cpp"], set()
    while todo:
        name = todo.pop()
        seen.add(name)
        if name == "api.cpp":  # launches: its own headers are the library's other parts
            continue
        with open(os.path.join(CSRC, name)) as f:
            inc = re.findall(r'#include "([^"/]+)"', f.read())
        todo += [i for i in inc if i not in seen]
    assert seen <= set(bench.TRAFFIC_SOURCES), seen - set(bench.TRAFFIC_SOURCES)
