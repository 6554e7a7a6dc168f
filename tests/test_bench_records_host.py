"""Host logic of the benchmark (no GPU): what its recorded figures depend on."""
import json
import os
import re
import sys

import pytest

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


def test_break_even_of_assembly():
    # 10 ms of assembly are won back after 5 products that are 2 ms shorter each
    assert bench.products_before_assembly_pays(10.0, 3.0, 1.0) == pytest.approx(5.0)
    # never, where the product with the matrix takes as long or longer
    assert bench.products_before_assembly_pays(51.0, 3.4, 5.2) is None
    assert bench.products_before_assembly_pays(51.0, 5.2, 5.2) is None
