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
        log = C.create_string_buffer(1)
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
            log = C.create_string_buffer(4096)
            if "current" in c:                   # the calls that overwrite the state, with another GPU current
                n_params, keep = L.rinr_fit_n_params(h), (C.c_uint8 * (c["n"] * L.rinr_fit_n_params(h)))()
                fake.hipSetDevice(c["current"])
                fake.fake_log(log, C.c_size_t(len(log)))
                rc += [L.rinr_fit_set_params(h, (C.c_float * (c["n"] * n_params))()), L.rinr_fit_set_keep(h, keep), L.rinr_fit_reset_optimizer(h)]
                fake.fake_log(None, C.c_size_t(0))
                now = C.c_int()
                fake.hipGetDevice(C.byref(now))
                log.value += b"now %d" % now.value
                fake.hipSetDevice(0)
            rc.append(L.rinr_fit_destroy(h))
        out.append(dict(rc=rc, launches=[list(grids[4 * k:4 * k + 4]) for k in range(n)], live=fake.fake_live(), log=log.value.decode()))
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


# case, the pixels a workgroup takes at a time, workgroups that run side by side on a CU (four wavefronts per SIMD at most), workgroups per image (None: more than one)
PLANS = {
    "few photographs": (case(8, 171, 219, 32, 10), 128, 1, 30),              # one round of 256, ten chunks each
    "one photograph": (case(1, 224, 224, 40, 10), 64, 1, 196),              # four chunks each; shorter shares pay more for their start
    "one per CU": (case(256, 224, 224, 40, 10), 64, 1, 1),
    "one more than CUs": (case(257, 224, 224, 40, 10), 64, 1, None),        # a second round for one image would double the step
    "two full rounds": (case(2048, 32, 32, 15, 3, resident=4), 128, 4, 1),
    "many": (case(5000, 64, 64, 40, 10), 64, 1, 1),                         # 16 rounds and more: the last one's idle part does not matter
    "two chunks": (case(2, 16, 16, 32, 10), 128, 1, 1),                     # sharing would cost the second launch what it saves
    "three chunks": (case(2, 18, 18, 32, 10), 128, 1, 3),                   # no share without pixels
    "one chunk": (case(3, 5, 7, 16, 3, resident=8), 128, 4, 1),
    "fp32 kernels": (case(8, 171, 219, 32, 10, fp32=1, resident=2), 64, 2, None),
    "fp32, one per CU": (case(256, 224, 224, 64, 7, resident=1), 64, 1, 1),
}


def test_workgroups_per_image(tmp_path):
    got = on_fake_runtime(tmp_path, [c for c, _, _, _ in PLANS.values()])
    for (name, (c, pixels, side, want)), g in zip(PLANS.items(), got):
        assert g["rc"] == [0, 0, 0] and g["live"] == 0
        n, slots, chunks = c["n"], CUS * side, -(-c["H"] * c["W"] // pixels)
        grid = g["launches"][0][0]
        s = grid // n
        assert grid == n * s and 1 <= s <= chunks, (name, s)
        assert s == want if want else s > 1, (name, s)

        def cost(s):                                # chunk times: rounds of workgroups x (a share and its start), and the second launch
            return -(-n * s // slots) * (-(-chunks // s) + 2) + (s > 1)
        assert cost(s) <= cost(1) and all(cost(s) <= cost(t) for t in range(2, min(chunks, 8 * slots // n) + 1) if n < 16 * slots), (name, s)
        n_params = sum((i + 1) * o for i, o in zip(c["widths"], c["widths"][1:]))
        second = [[n_params // 64 + 1, n, 256 if s <= 16 else 1024]] if s > 1 else []
        assert [l[:3] for l in g["launches"][1:]] == second, name


def test_state_is_overwritten_on_the_handles_gpu(tmp_path):
    """Steps in flight on the handle's GPU are waited for, and its memory is written from there, whatever GPU is current; that one is
    current again afterwards."""
    for current in (0, 3):
        g, = on_fake_runtime(tmp_path, [case(3, 8, 8, 15, 3, current=current)])
        assert g["rc"] == [0] * 6
        assert g["log"] == "sync 0, copy 0, launch 0, " * 2 + "sync 0, launch 0, now %d" % current


if __name__ == "__main__":
    child(sys.argv[1], json.loads(sys.argv[2]))
