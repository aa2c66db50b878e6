"""Where a lane's pixels go: planes and outputs that begin anywhere in a vector, images whose last lane has fewer pixels than a vector.
Whatever the place, the values are those of an aligned decode, and nothing beside them is touched."""
import numpy as np
import pytest

from paper_2306_16699_amd import rinr, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [8, 24, 40])                        # tiles of 16 and of 32 rows: four and two pixels a lane
@pytest.mark.parametrize("H,W", [(1, 1), (1, 3), (5, 13), (8, 8), (7, 10), (33, 31), (64, 65)])
def test_any_place_of_the_outputs(width, H, W):
    import torch
    n = 3
    models = synth.make_models(5, np.arange(n), width, 2, [0, 8, 0], 0.7)
    st = rinr.Store(rinr.pack(models))
    ids = torch.arange(n, device="cuda")
    size = n * 3 * H * W
    want, want8 = st.decode_batch_ex(ids, H, W, rinr.OUT_F32_AND_U8)
    for skew, skew8 in ((1, 1), (2, 3), (3, 2), (0, 1), (1, 0)):
        f = torch.full((size + 8,), -7.0, device="cuda")
        b = torch.full((size + 8,), 201, dtype=torch.uint8, device="cuda")
        st.decode_batch_ex(ids, H, W, rinr.OUT_F32_AND_U8, out=f[skew:skew + size].view(n, 3, H, W), out_u8=b[skew8:skew8 + size].view(n, 3, H, W))
        torch.cuda.synchronize()
        assert torch.equal(f[skew:skew + size].view(n, 3, H, W), want) and torch.equal(b[skew8:skew8 + size].view(n, 3, H, W), want8), (skew, skew8)
        assert (f[:skew] == -7.0).all() and (f[skew + size:] == -7.0).all()
        assert (b[:skew8] == 201).all() and (b[skew8 + size:] == 201).all()
    # ... and the aligned decode against the other family of kernels, whose stores are its own
    ref = st.decode_batch_ex(ids, H, W, rinr.OUT_F32, rinr.FLAG_FP32_MFMA)
    assert float((want - ref).abs().max()) <= 2e-5
    assert int((want8.int() - torch.round(255.0 * want).int()).abs().max()) <= 1
    st.close()
