"""Creating plans when device memory is short, on a host stand-in for the HIP runtime's memory
(tests/host_hip/device_memory.cpp): no GPU."""
import json
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

CHILD = r'''
import ctypes, json, sys
import numpy as np
sys.path.insert(0, sys.argv[1])
mem = ctypes.CDLL(sys.argv[2], mode=ctypes.RTLD_GLOBAL)
mem.device_memory_budget.argtypes = [ctypes.c_size_t]
mem.device_memory_used.restype = ctypes.c_size_t
from paper_2604_02624_amd import dpx, workloads as wk
lib = dpx.load_library()
n, pad, n_wl, layers = (int(x) for x in sys.argv[3:7])
wl = np.linspace(450e-9, 700e-9, n_wl)
arr, keep = dpx._c_designs([wk.make_design(n=n, layers=layers, wl=wl, n_mat=1.5, dx=300e-9, z=9e-6, fov=n, pad=pad)])

def create(budget, **opts):
    """Status, whether the plan runs LDS-resident, bytes held while it exists and after."""
    mem.device_memory_budget(budget)
    plan = ctypes.c_void_p()
    st = lib.dpx_plan_create(arr, 1, ctypes.byref(dpx._opts(lib, **opts)), ctypes.byref(plan))
    lds, held = None, mem.device_memory_used()
    if st == 0:
        lo = dpx.CLayout()
        lib.dpx_plan_layout(plan, 0, ctypes.byref(lo))
        lds = bool(lo.lds_path)
        lib.dpx_plan_destroy(plan)
    return st, lds, held, mem.device_memory_used()

full, passes = create(1 << 40), create(1 << 40, schedule=1)
print(json.dumps(dict(full=full, passes=passes, exact=create(full[2]), below=create(full[2] - 1),
                      least=create(passes[2]), too_little=create(passes[2] - 1))))
'''


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
@pytest.mark.parametrize("n,pad,n_wl,layers", [(32, 2, 6, 2), (48, 2, 100, 1), (64, 2, 4096, 4), (64, 1, 4099, 3)])
def test_a_plan_that_fits_without_the_lds_path_is_created(tmp_path, n, pad, n_wl, layers):
    """A small plan that would run LDS-resident by itself falls back to the multi-pass kernels where
    device memory holds only theirs, and fails only where it does not hold those either."""
    shim = tmp_path / "libdevice_memory.so"
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", os.path.join(HERE, "host_hip", "device_memory.cpp"), "-o", str(shim)],
                   check=True, capture_output=True, text=True)
    run = subprocess.run([sys.executable, "-c", CHILD, ROOT, str(shim)] + [str(x) for x in (n, pad, n_wl, layers)],
                         capture_output=True, text=True)
    assert run.returncode == 0, run.stderr
    r = json.loads(run.stdout)
    no_memory = 3
    assert r["full"][:2] == [0, True] and r["passes"][:2] == [0, False]
    assert r["full"][2] > r["passes"][2]  # the field after the first layer is kept too
    assert r["exact"][:2] == [0, True]
    for k in ("below", "least"):
        assert r[k][:2] == [0, False] and r[k][2] == r["passes"][2], (k, r)
    assert r["too_little"][0] == no_memory
    assert all(v[3] == 0 for v in r.values())  # nothing stays allocated
