"""How many launches a call of several Adam steps makes, without a GPU: a kernel of few registers takes up to 32 steps of an image that one
workgroup has; an image that is shared, or has many pixels, takes one."""
import ctypes as C
import json
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
pytestmark = pytest.mark.skipif(shutil.which("gcc") is None, reason="needs gcc")


def child(stub, cases):
    """Runs in the child process, on stand-ins of the HIP runtime (fake_hip.c): grid x of every launch of `steps` Adam steps, per case."""
    fake = C.CDLL(stub, mode=C.RTLD_GLOBAL)
    sys.path.insert(0, ROOT)
    from paper_2306_16699_amd import rinr_fit
    L = rinr_fit.lib()
    fake.fake_set.argtypes = [C.c_size_t, C.c_int, C.c_int]
    out = []
    for n, H, W, width, layers, resident, steps in cases:
        arch = rinr_fit.FitArch(layers, (C.c_int32 * 13)(2, *[width] * (layers - 1), 3), 30.0, -1.0, 1.0)
        h = C.c_void_p()
        fake.fake_set(2 ** 62, 256, resident)
        assert L.rinr_fit_create_ex(C.byref(arch), n, H, W, 0, C.byref(h)) == 0
        o = rinr_fit.FitOpts(1e-3, 0, 0, 0.0, 0.0, 0.0, 0.0)
        assert L.rinr_fit_steps(h, 16, steps, C.byref(o), None) == 0         # the targets' address is never followed here
        grids = (C.c_uint32 * 4096)()
        out.append([grids[4 * k] for k in range(fake.fake_launches(grids))])
        L.rinr_fit_destroy(h)
    print(json.dumps(out))


# images, height, width, units, layers, workgroups side by side on a CU, steps -> launches, whether an image is shared.  A workgroup takes 128 pixels at a time.
PLANS = [
    ((2048, 32, 32, 15, 3, 4, 70), 3, False),            # 32 + 32 + 6
    ((2048, 32, 32, 15, 3, 4, 64), 2, False),
    ((2048, 32, 32, 15, 3, 4, 1), 1, False),
    ((256, 32, 32, 40, 3, 1, 70), 70, False),            # no kernel of several steps
    ((1024, 64, 64, 8, 2, 4, 70), 3, False),             # 32 times 128 pixels: 32 steps
    ((1024, 65, 64, 8, 2, 4, 62), 2, False),             # a row more: 31
    ((1024, 128, 128, 8, 2, 4, 16), 2, False),           # 8
    ((8, 128, 128, 15, 3, 4, 5), 10, True),              # shared: a step's kernel and the one that adds up
    # images that are shared only where a step is a launch anyway
    ((600, 32, 32, 32, 3, 2, 70), 3, False),
    ((600, 32, 32, 32, 4, 2, 2), 4, True),
    # the second launch weighs less the deeper the model: measured on either side
    ((64, 24, 24, 15, 2, 4, 32), 1, False),
    ((64, 24, 24, 15, 5, 3, 1), 2, True),
    ((64, 24, 24, 15, 8, 2, 1), 2, True),
    ((128, 28, 28, 15, 6, 3, 1), 2, True),
    ((128, 28, 28, 32, 3, 2, 1), 2, True),
    ((800, 64, 64, 15, 8, 2, 1), 2, True),
    ((64, 24, 24, 15, 4, 3, 1), 2, True),
    ((400, 32, 32, 15, 4, 3, 32), 1, False),
    ((1000, 40, 40, 15, 7, 3, 32), 1, False),
    ((600, 32, 32, 15, 8, 2, 32), 1, False),
]


def test_launches_of_a_call(tmp_path):
    stub = str(tmp_path / "libfake_hip.so")
    subprocess.run(["gcc", "-O1", "-std=c11", "-Wall", "-Wextra", "-fPIC", "-shared", os.path.join(HERE, "fake_hip.c"), "-o", stub], check=True)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), stub, json.dumps([c for c, _, _ in PLANS])], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
    for (c, launches, shared), grids in zip(PLANS, json.loads(r.stdout)):
        assert len(grids) == launches and (grids[0] > c[0]) == shared, (c, grids[:4])


if __name__ == "__main__":
    child(sys.argv[1], json.loads(sys.argv[2]))
