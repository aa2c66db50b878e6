"""Host side of a decode without a GPU: the LDS and the workgroups of a launch.  The library runs in a child process on stand-ins of the HIP
runtime (fake_hip.c), where as many workgroups share a CU as its LDS holds."""
import ctypes as C
import json
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)
from paper_2306_16699_amd import rinr, synth  # noqa: E402

pytestmark = pytest.mark.skipif(shutil.which("gcc") is None, reason="needs gcc")
CU_LDS = 160 * 1024


def models_of(groups):
    """groups: (width, sine layers, bits of the hidden layers); one model of each."""
    return sum((synth.make_models(3 + k, np.arange(1), w, d, [0] + [b] * (d - 1) + [0], 0.6) for k, (w, d, b) in enumerate(groups)), [])


def child(stub, cases):
    fake = C.CDLL(stub, mode=C.RTLD_GLOBAL)
    fake.fake_set.argtypes = [C.c_size_t, C.c_int, C.c_int]
    fake.fake_cu_lds.argtypes = [C.c_size_t]
    fake.fake_cu_lds(CU_LDS)
    L = rinr.lib()
    out = []
    for c in cases:
        fake.fake_set(2 ** 62, 256, c.get("resident", 8))
        blob = rinr.pack(models_of(c["groups"]))
        held = np.empty(blob.size + 16, np.uint8)                       # the device blob: never read here, but its alignment is checked
        at = (held.ctypes.data + 15) & ~15
        s, info = C.c_void_p(), (C.c_int32 * 6)()
        opts = rinr.OpenOpts()
        opts.lds_budget = c.get("budget", 0)
        rc = [L.rinr_store_open_ex(at, blob.ctypes.data, blob.size, C.byref(opts), C.byref(s))]
        if rc[0] == 0:
            o = rinr.DecodeOpts()
            o.out_dtype, o.flags, o.one_grid_min_tiles = rinr.OUT_F32, c.get("flags", 0), c.get("one_grid_min_tiles", 0)
            if c.get("order"):
                o.workspace, o.workspace_bytes = 16, rinr.workspace_bytes(c["n"])
            rc.append(L.rinr_decode_batch_ex(s, 16, c["n"], c["H"], c["W"], 16, C.byref(o), None))       # the addresses are never followed here
            rc.append(L.rinr_last_launch_info(s, C.byref(info)))
            rc.append(L.rinr_store_close(s))
        out.append(dict(rc=rc, launches=info[0], blocks=info[1], threads=info[2], lds=info[3], streamed=info[5]))
    print(json.dumps(out))


def on_fake_runtime(tmp_path, cases):
    stub = str(tmp_path / "libfake_hip.so")
    subprocess.run(["gcc", "-O1", "-std=c11", "-Wall", "-Wextra", "-fPIC", "-shared", os.path.join(HERE, "fake_hip.c"), "-o", stub], check=True)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), stub, json.dumps(cases)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads(r.stdout)


FAST, FASTEST = rinr.FLAG_FP16_ACT | rinr.FLAG_FP16_UNCHECKED, rinr.FLAG_FP16_ALL | rinr.FLAG_FP16_UNCHECKED


def expanded(width, sines, bits, flags):
    """Bytes of the expanded model in the layout of the kernel that takes a store of this one width: layer table and selectors, biases, the
    first layer's variants, hidden layers and the output layer with their last quads' steps."""
    wq, reduced = -(-width // 8) * 8, flags != 0
    wp, ints = -(-wq // 16) * 16, bits == 8
    tm = 32 if wq == 24 or (wq == 32 and reduced) else 16
    mt, quads = wp // tm, (wp // 16 if tm == 16 else wq // 8)
    pairs, odd = quads // 2, quads % 2
    two_rows = odd and tm == 16 and wq != wp                    # low parts beside the others
    tail = 0 if not odd else (1024 if two_rows or tm == 32 or (ints and not reduced) else 512)
    low = 0 if two_rows else tail
    hidden = mt * (pairs * 1024 + tail) + (0 if ints or flags == FASTEST else mt * (pairs * 1024 + low))
    return 320 + 4 * (sines * wp + tm) + 64 // tm * mt * 1024 + (sines - 1) * hidden + 2 * pairs * 1024 + tail + low


@pytest.mark.parametrize("flags", [0, FAST, FASTEST])
def test_a_launch_takes_the_lds_of_its_own_layout(tmp_path, flags):
    """A model is charged what the kernel that takes it builds, and its record: neither the largest layout of the width class nor that of
    another mode."""
    cases, want = [], []
    for width in (1, 8, 9, 16, 17, 24, 25, 32, 33, 40, 41, 48, 49, 56, 57, 64):
        for sines, bits in ((2, 8), (5, 8), (4, 16)):
            g = [(width, sines, bits)]
            record = int(rinr.pack(models_of(g)).view(np.uint32)[(64 + 8) // 4])
            cases.append(dict(groups=g, n=300, H=32, W=32, flags=flags))
            want.append(expanded(width, sines, bits, flags) + 16 + record)
    for c, w, g in zip(cases, want, on_fake_runtime(tmp_path, cases)):
        assert g["rc"] == [0] * 4 and g["launches"] == 1 and not g["streamed"], c
        assert g["lds"] == w, (c, g["lds"], w)


RAGGED = [(w, d, 8) for w in (24, 40, 64) for d in (3, 6)]
# images, side, ordered -> threads, workgroups: a tile for each wavefront in as many workgroups as can run at once without sharing a CU in vain
SPLITS = [((1, 100, False), (256, 40)), ((4, 64, False), (256, 64)), ((16, 64, False), (256, 256)), ((16, 64, True), (256, 256)), ((64, 32, False), (256, 256)),
          ((17, 64, False), (512, 136)), ((16, 16, False), (512, 16)), ((16, 100, False), (768, 224)), ((16, 100, True), (512, 320)),
          ((4, 224, False), (512, 392)), ((4, 224, True), (512, 392)), ((64, 64, False), (512, 512)), ((64, 64, True), (512, 512)),
          ((256, 32, False), (512, 512)), ((256, 32, True), (512, 512))]


def test_few_ragged_images_are_split_into_what_runs_at_once(tmp_path):
    got = on_fake_runtime(tmp_path, [dict(groups=RAGGED, n=n, H=side, W=side, order=order, resident=2) for (n, side, order), _ in SPLITS])
    for (c, want), g in zip(SPLITS, got):
        assert g["rc"] == [0] * 4 and (g["threads"], g["blocks"]) == want, (c, g)


def test_a_class_is_split_by_its_own_heaviest_model(tmp_path):
    """Class by class, the models of another class do not count: 64 units are split as in a store without the deep 16-unit model."""
    alone = [(64, d, 8) for d in (2, 3)]
    cases = [dict(groups=g, n=n, H=side, W=side, order=order, resident=2, one_grid_min_tiles=1 << 30)
             for n in (4, 16, 64, 300) for side in (32, 64, 100, 224) for order in (False, True) for g in (alone, [(16, 15, 8)] * 2 + alone)]
    got = on_fake_runtime(tmp_path, cases)
    for c, a, b in zip(cases[::2], got[::2], got[1::2]):
        assert a["rc"] == b["rc"] == [0] * 4 and b["launches"] == a["launches"] + 1, c
        assert (a["threads"], a["blocks"]) == (b["threads"], b["blocks"]), (c, a, b)


if __name__ == "__main__":
    child(sys.argv[1], json.loads(sys.argv[2]))
