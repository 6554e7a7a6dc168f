"""CPU tests of what vms_assemble launches, and where.

The overlapped schedule when something fails: the second stream's kernels read the caller's fields and write the context's
records, so whatever vms_assemble has queued there must be waited for by the
context stream before it returns, an error included. libvms runs against a host
stand-in of the HIP runtime that logs the order of the streams and lets one
launch or call fail; no device is used. (The stand-in holds 12 workgroups of
every kernel on each of 256 CUs: 3072.)"""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_PROBE = r"""
import ctypes as C, sys
import numpy as np
sys.path.insert(0, sys.argv[1])
S = C.CDLL(sys.argv[2], C.RTLD_GLOBAL)   # before libvms: its HIP calls bind here
S.stand_in_log.restype = C.c_char_p
from paper_2009_00706_amd import inputs as I, vms
kernel, call, nth, timing, prec = sys.argv[3].encode(), sys.argv[4].encode(), int(sys.argv[5]), int(sys.argv[6]), int(sys.argv[7])
flags = int(sys.argv[8])
CTX = 0x10
S.stand_in_config(5, 9)
t = I.uniform_octree(3)
s = I.icosphere(1, 0.2, (0.5, 0.5, 0.5))
ctx = vms.vms_create(t, s, vms.make_params(precision=prec), stream=CTX)
st = vms.vms_stats(ctx)
assert st["n_out"] > 0 and st["n_intercepted"] > 0 and st["n_subgp"] == 9 * st["n_intercepted"]
sz = vms.vms_sizes(ctx)
f = [np.zeros(sz["n_nodes"]) for _ in range(7)]
F = vms.Fields(*(a.ctypes.data for a in f))
vals, res = np.zeros(sz["nnz"]), np.zeros(sz["n_rows"])
vms.vms_set_timing(ctx, timing)
L = vms.lib()
S.stand_in_reset(b"", b"", 0)
assert L.vms_assemble(ctx, C.byref(F), vals.ctypes.data, res.ctypes.data, flags) == 0
print("clean")
print(S.stand_in_log().decode(), end="")
S.stand_in_reset(kernel, call, nth)
rc = L.vms_assemble(ctx, C.byref(F), vals.ctypes.data, res.ctypes.data, flags)
print("failed", rc)
print(S.stand_in_log().decode(), end="")
"""


@pytest.fixture(scope="module")
def stand_in(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("stand_in") / "stand_in.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__",
                    "-D_Float16=unsigned short", "-I", "/opt/rocm/include",
                    "-I", os.path.join(ROOT, "paper_2009_00706_amd", "csrc"),
                    os.path.join(ROOT, "tests", "hip_stand_in.cpp"), "-o", so], check=True)
    return so


def run(stand_in, kernel, call, nth, timing, prec, flags=1):
    r = subprocess.run([sys.executable, "-c", _PROBE, ROOT, stand_in, kernel, call, str(nth), str(int(timing)), str(prec),
                        str(flags)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    lines = r.stdout.splitlines()
    k = next(i for i, x in enumerate(lines) if x.startswith("failed"))
    return [x.split() for x in lines[1:k]], int(lines[k].split()[1]), [x.split() for x in lines[k + 1:]]


def unjoined(log, ctx="10"):
    """Launches on other streams that ctx does not wait for by the end of the log."""
    done, recorded, queued = {}, {}, {}
    for op in log:
        if op[0] == "launch" and op[1] != ctx:
            queued.setdefault(op[1], []).append(op[2])
        elif op[0] == "record":
            recorded[op[1]] = (op[2], len(queued.get(op[2], [])))
        elif op[0] == "wait" and op[1] == ctx and op[2] in recorded:
            s, n = recorded[op[2]]
            done[s] = max(done.get(s, 0), n)
        elif op[0] == "sync":
            done[op[1]] = len(queued.get(op[1], []))
    return [k for s, q in queued.items() for k in q[done.get(s, 0):]]


# (timing on, kernel whose launch fails, call that fails, its how manieth). The events
# of a call with timing off are the fork and the join, with timing on the fork is
# the fifth and the join the ninth.
FAULTS = [(tm, *f) for tm in (False, True) for f in
          [("k_asm2", "", 1), ("k_asm2", "", 2), ("k_subquad", "", 1), ("k_gather", "", 1), ("k_gather_list", "", 1),
           ("", "wait", 1), ("", "wait", 2)]] + \
    [(False, "", "record", n) for n in (1, 2)] + [(True, "", "record", n) for n in range(4, 11)]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("timing,kernel,call,nth", FAULTS)
def test_second_stream_is_joined_on_errors(stand_in, timing, kernel, call, nth, prec):
    clean, rc, log = run(stand_in, kernel, call, nth, timing, prec)
    side = {op[1] for op in clean if op[0] == "launch"} - {"10"}
    assert len(side) == 1, clean        # the overlapped schedule: one other stream
    assert sum(op[0] == "launch" and op[1] in side for op in clean) >= 2
    assert unjoined(clean) == []
    assert rc == -3                     # VMS_EHIP
    assert unjoined(log) == [], log


@pytest.mark.parametrize("prec,relabel,timing,after_out", [
    (0, 1, False, False), (0, 0, False, True), (1, 1, False, False), (1, 0, False, True),
    (0, 1, True, True), (1, 0, True, True)])
def test_where_the_second_stream_starts(stand_in, prec, relabel, timing, after_out):
    """With the call; after the OUT elements with timing on, and where it then ends
    before the gather (here without the relabel, whose longest element outlasts it)."""
    clean, _, _ = run(stand_in, "", "", 0, timing, prec, relabel)
    side = next(op[1] for op in clean if op[0] == "launch" and op[1] != "10")
    forked = next(i for i, op in enumerate(clean) if op[0] == "wait" and op[1] == side)
    event = clean[forked][2]
    recorded = max(i for i, op in enumerate(clean[:forked]) if op[:2] == ["record", event])
    out = next(i for i, op in enumerate(clean) if op[0] == "launch" and op[1] == "10" and "k_asm2" in op[2])
    assert (recorded > out) == after_out
    assert unjoined(clean) == []


_GRID_PROBE = r"""
import ctypes as C, sys
import numpy as np
sys.path.insert(0, sys.argv[1])
S = C.CDLL(sys.argv[2], C.RTLD_GLOBAL)
S.stand_in_log.restype = C.c_char_p
from paper_2009_00706_amd import inputs as I, vms
for prec in (0, 1, 2):
    for ext in ((16, 16, 12), (16, 14, 14), (16, 16, 14), (16, 16, 15), (24, 32, 16), (25, 23, 23)):
        t = I.refined_octree(5, 5, lambda x, y, z, h, l: np.zeros(x.shape, bool), ext=ext)
        ctx = vms.vms_create(t, None, vms.make_params(precision=prec), stream=0x10)
        sz = vms.vms_sizes(ctx)
        f = np.zeros(sz["n_nodes"])
        F = vms.Fields(*([f.ctypes.data] * 7))
        vals, res = np.zeros(sz["nnz"]), np.zeros(sz["n_rows"])
        S.stand_in_reset(b"", b"", 0)
        assert vms.lib().vms_assemble(ctx, C.byref(F), vals.ctypes.data, res.ctypes.data, 0) == 0
        print(prec, t.n, next(l.split()[3] for l in S.stand_in_log().decode().splitlines() if "k_asm2" in l))
        vms.vms_destroy(ctx)
"""


def test_out_elements_per_workgroup(stand_in):
    """One OUT element per workgroup up to four rounds of workgroups, two above
    (the last of an odd count alone); FP64 also two where one each would leave a
    second round nearly empty."""
    r = subprocess.run([sys.executable, "-c", _GRID_PROBE, ROOT, stand_in], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    got = {tuple(map(int, x.split()[:2])): int(x.split()[2]) for x in r.stdout.splitlines()}
    one = {3072: 3072, 3136: 3136, 3584: 3584, 3840: 3840, 12288: 12288, 13225: 6613}
    want = {(p, n): g for p in (0, 1, 2) for n, g in one.items()}
    want.update({(0, 3136): 1568, (0, 3584): 1792})
    assert got == want
