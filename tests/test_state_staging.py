"""Staging of state transfers, on the host: the library's HIP calls go to a
recorder (tests/hip_recorder.cpp) in which device memory is host memory and
kernels do nothing.  Staging lies on the handle's device whatever the current
one; without device memory it lies inside the workspace; every byte of the
caller's arrays is copied once a pass."""
import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
import ctypes as C, json, sys
import numpy as np
rec = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
import paper_2406_15236_amd as m
job = json.loads(sys.argv[3])
u64 = C.c_uint64
rec.rec_workspace.argtypes = [u64, u64, C.c_int]
rec.rec_count.restype = u64
rec.rec_event.argtypes = [u64, C.POINTER(u64)]

def events():
    out = []
    for i in range(rec.rec_count()):
        e = (u64 * 5)()
        rec.rec_event(i, e)
        out.append([int(q) for q in e])
    rec.rec_clear()
    return out

p = [m.make_params(dict(L=L, density=10.0, mbs=True), job["form"]) for L in job["L"]]
nb = m.workspace_bytes(p)
raw = np.zeros(nb + 512, dtype=np.uint8)
ws = (raw.ctypes.data + 255) // 256 * 256
rec.rec_workspace(ws, nb, job["device"])
rec.hipSetDevice(job["current"])
h = m.create(p, ws, nb, 0)
rec.rec_refuse(job["refuse"])
out = dict(ws=ws, bytes=nb, calls=[])
for k, L in enumerate(job["L"]):
    n = 10 * L[0] * L[1] * L[2]
    x, v = np.full((3, n), 0.5), np.full((3, n), 0.25)
    for name in ("mpc_set_state", "mpc_get_state"):
        events()
        rc = getattr(m.lib(), name)(h, k, m._f64(x), m._f64(v), n)
        out["calls"].append(dict(name=name, rc=rc, n=n, x=x.ctypes.data, v=v.ctypes.data,
                                 events=events(), current=rec.rec_current()))
idx = np.array([0, 1], dtype=np.int64)
y = np.zeros((2, 3, 2))
rec.rec_refuse(0)
rc = m.lib().mpc_get_particles(h, 0, idx.ctypes.data_as(C.POINTER(C.c_int64)), 2, m._f64(y[0]),
                               m._f64(y[1]))
out["calls"].append(dict(name="mpc_get_particles", rc=rc, events=events(),
                         current=rec.rec_current()))
assert m.lib().mpc_destroy(h) == 0
print(json.dumps(out))
"""


@pytest.fixture(scope="module")
def record(tmp_path_factory):
    import paper_2406_15236_amd as m
    if not os.path.exists(m.LIB):
        pytest.skip("library not built")
    d = tmp_path_factory.mktemp("rec")
    so = str(d / "hip_recorder.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", os.path.join(ROOT, "tests", "hip_recorder.cpp"), "-o",
                    so], check=True)

    def run(**job):
        job = dict(dict(form="fp64", L=[(16, 12, 10)], device=0, current=0, refuse=0), **job)
        r = subprocess.run([sys.executable, "-c", PROGRAM, so, ROOT, json.dumps(job)],
                           capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr[-2000:]
        return json.loads(r.stdout)
    return run


@pytest.mark.parametrize("form", ["fp64", "split"])
def test_staging_is_on_the_handles_device(record, form):
    out = record(form=form, device=1, current=0, L=[(16, 12, 10), (130, 110, 100)])
    for c in out["calls"]:
        assert c["rc"] == 0, c["name"]
        assert all(e[1] == 1 for e in c["events"] if e[0] == 0), c["name"]
        assert c["current"] == 0
    assert any(e[0] == 0 for c in out["calls"] for e in c["events"])


@pytest.mark.parametrize("form,L", [("fp64", [(16, 12, 10)]), ("fp32", [(16, 12, 10), (31, 9, 7)]),
                                    ("split", [(2, 2, 1), (64, 50, 41)])])
def test_staging_inside_the_workspace(record, form, L):
    """No device memory: chunks through the run lists' part of the workspace."""
    out = record(form=form, L=L, refuse=1)
    lo, hi = out["ws"], out["ws"] + out["bytes"]
    for c in out["calls"]:
        if c["name"] == "mpc_get_particles":
            continue
        assert c["rc"] == 0, c["name"]
        into, size = (0, 24 * c["n"]) if "get" in c["name"] else (1, 24 * c["n"])
        covered = {c["x"]: 0, c["v"]: 0}
        for kind, _, to, frm, n in c["events"]:
            assert kind == 1
            host, dev = (to, frm) if into == 0 else (frm, to)
            base = [b for b in covered if b <= host and host + n <= b + size]
            if base:
                assert lo <= dev and dev + n <= hi
                covered[base[0]] += n
        if into == 0 and 2 * size <= 256 << 10:  # one copy of flag and arrays
            assert [(lo <= e[3] and e[3] + e[4] <= hi, e[4]) for e in c["events"] if
                    e[4] > 4096 or e[4] == 256 + 2 * size][-1] == (True, 256 + 2 * size)
            continue
        passes = 1 if into == 0 else max(1, covered[c["x"]] // size)
        assert set(covered.values()) == {passes * size} and passes <= 2


def test_several_chunks_of_device_staging(record):
    """Above 1 GiB of staging: chunks in one allocation of that size."""
    out = record(L=[(140, 130, 125)], form="fp32")
    for c in out["calls"][:2]:
        assert c["rc"] == 0
        alloc = [e for e in c["events"] if e[0] == 0]
        assert [e[4] for e in alloc] == [1 << 30]
        got = sum(e[4] for e in c["events"] if e[0] == 1 and
                  any(b <= e[2] < b + 24 * c["n"] or b <= e[3] < b + 24 * c["n"]
                      for b in (c["x"], c["v"])))
        assert got == 48 * c["n"] * (2 if c["name"] == "mpc_set_state" else 1)
