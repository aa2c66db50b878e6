"""Builds librinr.so (hipcc, gfx950) in-tree.  `python -m paper_2306_16699_amd.build`."""
from __future__ import annotations

import os
import re
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
SO = os.path.join(HERE, "librinr.so")

HIP_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-Wall", "-Wno-unused-command-line-argument"]
# Sources, the one that takes longest first, with flags of their own.  The fit kernels that run one wavefront per SIMD use all
# 512 of its registers: matrix results that vector instructions read next go to the directly addressable half, else every
# one of them is copied there first, and six kernels spill beyond 256 registers, which must not be (10 layers x 40: 360).
SOURCES = {"rinr_fit.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"], "rinr_api.hip": [], "rinr_pack.cpp": [], "rinr_bounds.cpp": [],
           "rinr_encode.cpp": []}


def lost_reloads(remarks: str) -> list:
    """Kernels of more than 256 registers that spill, from the compiler's remarks on kernel resources: (name, registers, spilled).
    The compiler loses reloads of parts of a matrix result in such a kernel (the fit kernels' gradients were wrong)."""
    bad = []
    for part in remarks.split("remark: Function Name: ")[1:]:
        vgprs, agprs, spilled = (int(re.search(key + r": (\d+)", part).group(1)) for key in (" VGPRs", " AGPRs", " VGPRs Spill"))
        if vgprs + agprs > 256 and spilled:
            bad.append((part.split()[0], vgprs + agprs, spilled))
    return bad


def build(verbose: bool = False, extra=()) -> str:
    with tempfile.TemporaryDirectory() as tmp:
        objs = [os.path.join(tmp, n + ".o") for n in SOURCES]
        cmds = [["hipcc", *HIP_FLAGS, *own, *extra, "-Rpass-analysis=kernel-resource-usage", "-fno-caret-diagnostics", "-c", "-o", o,
                 os.path.join(CSRC, n)] for o, (n, own) in zip(objs, SOURCES.items())]
        running = []
        for o, cmd in zip(objs, cmds):
            if verbose:
                print(" ".join(cmd), flush=True)
            with open(o + ".log", "w") as log:
                running.append(subprocess.Popen(cmd, stderr=log))
        failed = [cmd for cmd, p in zip(cmds, running) if p.wait() != 0]
        spilled = []
        for o in objs:
            with open(o + ".log") as f:
                text = f.read()
            sys.stderr.write("".join(ln for ln in text.splitlines(True) if ": remark: " not in ln))
            spilled += lost_reloads(text)
        if failed:
            raise RuntimeError("failed: " + " ".join(failed[0]))
        if spilled:
            raise RuntimeError(f"kernels of more than 256 registers spill (this compiler would compute wrong gradients): {spilled}")
        link = ["hipcc", "--offload-arch=gfx950", "-fno-gpu-rdc", "-shared", "-o", SO, *objs]
        if verbose:
            print(" ".join(link), flush=True)
        subprocess.run(link, check=True)
    return SO


if __name__ == "__main__":
    build(verbose=True, extra=sys.argv[1:])
