"""Host side of the fit handle without a GPU: how many workgroups share an image, and what happens if the memory for their
partial sums cannot be had.  The library runs in a child process on stand-ins of the HIP runtime (fake_hip.c) that write
down each launch's grid."""
import ctypes as C
import json
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CUS = 256


def child(stub, cases):
    """Runs in the child process: the launches of one Adam step and what the handle answered, per case."""
    fake = C.CDLL(stub, mode=C.RTLD_GLOBAL)
    sys.path.insert(0, ROOT)
    from paper_2306_16699_amd import rinr_fit
    L = rinr_fit.lib()
    fake.fake_set.argtypes = [C.c_size_t, C.c_int, C.c_int]
    fake.fake_live.restype = C.c_int64
    out = []
    for c in cases:
        arch = rinr_fit.FitArch(len(c["widths"]) - 1, (C.c_int32 * 13)(*c["widths"]), 30.0, -1.0, 1.0)
        h = C.c_void_p()
        fake.fake_set(c.get("limit", 2 ** 62), CUS, c["resident"])
        rc = [L.rinr_fit_create_ex(C.byref(arch), c["n"], c["H"], c["W"], c["fp32"], C.byref(h))]
        grids = (C.c_uint32 * 4096)()
        n = 0
        if rc[0] == 0:
            o = rinr_fit.FitOpts(1e-3, 0, 0, 0.0, 0.0, 0.0, 0.0)
            rc.append(L.rinr_fit_steps(h, 16, 1, C.byref(o), None))          # the targets' address is never followed here
            n = fake.fake_launches(grids)
            rc.append(L.rinr_fit_destroy(h))
        out.append(dict(rc=rc, launches=[list(grids[4 * k:4 * k + 4]) for k in range(n)], live=fake.fake_live()))
    print(json.dumps(out))


def on_fake_runtime(tmp_path, cases):
    stub = str(tmp_path / "libfake_hip.so")
    subprocess.run(["gcc", "-O1", "-std=c11", "-Wall", "-Wextra", "-fPIC", "-shared", os.path.join(HERE, "fake_hip.c"), "-o", stub], check=True)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), stub, json.dumps(cases)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads(r.stdout)


pytestmark = pytest.mark.skipif(shutil.which("gcc") is None, reason="needs gcc")


def case(n, H, W, width, L, fp32=0, resident=1, **more):
    return dict(n=n, H=H, W=W, widths=[2] + [width] * (L - 1) + [3], fp32=fp32, resident=resident, **more)


def test_without_memory_for_partial_sums_a_workgroup_takes_a_whole_image(tmp_path):
    roomy = case(8, 171, 219, 32, 10)
    n_params = sum((i + 1) * o for i, o in zip(roomy["widths"], roomy["widths"][1:]))
    got = on_fake_runtime(tmp_path, [roomy, dict(roomy, limit=8 * n_params * 4), dict(roomy, fp32=1, limit=8 * n_params * 4),
                                     dict(roomy, limit=8 * n_params * 4 - 1)])
    assert got[0]["rc"] == [0, 0, 0] and len(got[0]["launches"]) == 2
    for g in got[1:3]:                              # the rest fits, the partial sums do not
        assert g["rc"] == [0, 0, 0], g
        assert [l[:2] for l in g["launches"]] == [[8, 1]]
    assert got[3]["rc"] == [-8]                     # nor do the parameters: RINR_E_HIP, as ever
    assert all(g["live"] == 0 for g in got)


if __name__ == "__main__":
    child(sys.argv[1], json.loads(sys.argv[2]))
