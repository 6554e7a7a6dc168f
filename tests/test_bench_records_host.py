"""Host logic of the benchmark (no GPU): what its recorded figures depend on."""
import json
import os
import re
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402

CSRC = os.path.join(ROOT, "paper_2009_00706_amd", "csrc")


def included(name, seen):
    """name and every header of this project that it includes, directly or not."""
    if name not in seen:
        seen.add(name)
        for h in re.findall(r'^#include "([^"]+)"', open(os.path.join(CSRC, name)).read(), re.M):
            included(h, seen)
    return seen


def test_recorded_traffic_depends_on_every_source_of_the_element_kernels():
    assert set(bench.KERNEL_SOURCES) == included("assemble2.hip", set())
    rec = json.load(open(os.path.join(ROOT, "profiles", "traffic.json")))
    for e in rec["entries"]:
        assert [os.path.basename(s) for s in e["kernel_sources"]] == list(bench.KERNEL_SOURCES)
