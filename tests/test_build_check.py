"""The build refuses a library in which a kernel of more than 256 registers spills (CPU: the compiler needs no GPU)."""
import shutil

import pytest

from paper_2306_16699_amd import build

# 640 values live at once per thread; a launch bound of `threads` leaves it 512 registers (256 threads) or 256 (512)
KERNEL = """#include <hip/hip_runtime.h>
extern "C" __global__ __launch_bounds__(%d) void many(float *p, int n) {
    float v[%d], sum = 0.0f;
    _Pragma("unroll") for (int i = 0; i < %d; ++i) v[i] = p[threadIdx.x] * i;
    for (int k = 0; k < n; ++k)
        _Pragma("unroll") for (int i = 0; i < %d; ++i) v[i] = v[i] * v[i] + p[k];
    _Pragma("unroll") for (int i = 0; i < %d; ++i) sum += v[i];
    p[threadIdx.x] = sum;
}
"""


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not found")
@pytest.mark.parametrize("threads,live,refused", [(256, 640, True), (512, 320, False), (256, 300, False)],
                         ids=["512 registers, spills", "256 registers, spills", "512 registers, fits"])
def test_a_big_kernel_that_spills_is_refused(tmp_path, monkeypatch, threads, live, refused):
    (tmp_path / "many.hip").write_text(KERNEL % ((threads,) + (live,) * 4))
    monkeypatch.setattr(build, "CSRC", str(tmp_path))
    monkeypatch.setattr(build, "SO", str(tmp_path / "many.so"))
    monkeypatch.setattr(build, "SOURCES", {"many.hip": []})
    if refused:
        with pytest.raises(RuntimeError, match="spill.*many"):
            build.build()
        assert not (tmp_path / "many.so").exists()
    else:
        build.build()
        assert (tmp_path / "many.so").exists()
