"""Host logic of the benchmark (no GPU): what its recorded figures depend on."""
import json
import os
import re
import sys
from types import SimpleNamespace

import numpy as np
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


class _Event:
    def __init__(self, enable_timing=False):
        pass

    def record(self, stream):
        pass

    def elapsed_time(self, other):
        return 1.0


class _Library:
    """libvms as run_single sees it: notes timing and schedule of every step."""

    def __init__(self):
        self.timing, self.overlap, self.steps = False, True, []
        lib = self

        class Assembler:
            def __init__(self, *a):
                self.ctx, self.stream, self.sizes, self.vals, self.resid = 1, None, {}, None, None

            def set_fields(self, f):
                pass

            def assemble(self, flags=0):
                lib.steps.append((lib.timing, lib.overlap, flags))

            def close(self):
                pass
        self.Assembler = Assembler

    def make_params(self, **kw):
        return None

    def vms_stats(self, ctx):
        return {"n_out": 7, "n_intercepted": 3}

    def vms_sizes(self, ctx):
        return {}

    def vms_relabel_stats(self, ctx):
        return {}

    def vms_set_timing(self, ctx, on=True):
        self.timing = bool(on)

    def vms_set_overlap(self, ctx, on=True):
        self.overlap = bool(on)

    def vms_last_timing(self, ctx):
        assert self.timing
        return [1.0] * 5


def test_timed_steps_take_the_schedule_of_a_caller(monkeypatch):
    """The warm-up and the timed steps run with stage timing off, as a caller's do
    (an overlapped call with it on starts its second stream later), whatever
    prepare left on; the stages come from steps of their own."""
    monkeypatch.setattr(bench, "inactive_entries", lambda *a: None)
    lib = _Library()
    marks = []
    torch = SimpleNamespace(cuda=SimpleNamespace(Event=_Event, synchronize=lambda: marks.append(len(lib.steps))))
    m = bench.run_single(torch, lib, None, object(), None, 0, 4, 2, 1, prepare=lambda asm: lib.vms_set_timing(1, True))
    a, b = marks[:2]                  # around the timed region
    assert (a, b) == (2, 6)
    assert lib.steps[:b] == [(False, True, 1)] * 6
    assert m["stage"].shape == (5,) and m["ms_step"] > 0
    # stages in both schedules, and timing off again at the end
    assert (True, True, 1) in lib.steps and (True, False, 1) in lib.steps and not lib.timing
    assert np.isfinite(list(m["step_device_ms"].values())).all()
