"""A handle of many boxes is made in time proportional to them, on the host:
the library's HIP calls go to a recorder (tests/hip_recorder.cpp)."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
import ctypes as C, sys, time
import numpy as np
rec = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
import paper_2406_15236_amd as m
best = {}
for n in (512, 4096, 512, 4096, 512, 4096):
    p = [m.make_params(dict(L=(8, 8 + b % 3, 9), density=10.0, seed=b)) for b in range(n)]
    nb = m.workspace_bytes(p)
    raw = np.empty(nb + 512, dtype=np.uint8)
    ws = (raw.ctypes.data + 255) // 256 * 256
    arr, k = m._arr(p)
    h = C.c_void_p()
    t0 = time.perf_counter()
    assert m.lib().mpc_create(arr, k, C.c_void_p(ws), nb, None, C.byref(h)) == 0
    best[n] = min(best.get(n, 1e9), time.perf_counter() - t0)
    assert m.lib().mpc_destroy(h) == 0
print(best[512], best[4096])
"""


def test_time_grows_with_the_boxes(tmp_path):
    """Eight times the boxes: eight times the tiles to list and copy.  Growing
    the list box by box took 60 times as long; 24 leaves room for caches."""
    import paper_2406_15236_amd as m
    if not os.path.exists(m.LIB):
        pytest.skip("library not built")
    so = str(tmp_path / "hip_recorder.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", os.path.join(ROOT, "tests", "hip_recorder.cpp"), "-o",
                    so], check=True)
    r = subprocess.run([sys.executable, "-c", PROGRAM, so, ROOT], capture_output=True, text=True,
                       timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    few, many = (float(q) for q in r.stdout.split())
    print(f"512 boxes {few * 1e3:.2f} ms, 4096 boxes {many * 1e3:.2f} ms")
    assert many < 24 * few
