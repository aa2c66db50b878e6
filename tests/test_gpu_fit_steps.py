"""Several Adam steps of the fit kernels: what they are made of, and that it does not matter how they are cut into calls and launches."""
import numpy as np
import pytest

from paper_2306_16699_amd import rinr_fit, synth

pytestmark = pytest.mark.gpu

f32 = np.float32


def fma(a, b, c):
    """a * b + c rounded once: the product of two 32-bit numbers is exact in 64 bits (the sum may round twice, one in 2^28 times)."""
    return (np.float64(a) * np.float64(b) + np.float64(c)).astype(f32)


def targets(seed, n, H, W):
    import torch
    return torch.from_numpy(np.ascontiguousarray(synth.images(seed, n, H, W))).cuda()


def some_keep(seed, widths, n, ratio):
    """Flags of every parameter; biases are kept."""
    rng = np.random.default_rng(seed)
    mats = [[rng.random(o * i) < ratio for i, o in zip(widths, widths[1:])] for _ in range(n)]
    return np.stack([rinr_fit.weight_keep_flags(widths, m) for m in mats])


# a workgroup per image (entries of Adam four at a time; 10 x 48: one at a time), shares of an image with the second launch, fp32 kernels
@pytest.mark.parametrize("width,L,n,H,fp32", [(15, 3, 256, 8, False), (40, 5, 256, 9, False), (64, 4, 256, 8, False), (48, 10, 256, 8, False), (32, 4, 3, 32, False),
                                              (40, 6, 2, 40, False), (24, 4, 256, 8, True), (32, 3, 3, 24, True)])
@pytest.mark.parametrize("masked", [False, True])
def test_adam_to_the_bit(width, L, n, H, fp32, masked):
    """Every kernel rounds Adam alike, the gradient being the one that the handle reports."""
    widths = [2] + [width] * (L - 1) + [3]
    p = synth.init_params(9, widths, n).astype(f32)
    t = targets(4, n, H, H)
    f = rinr_fit.Fit(widths, n, H, H, fp32=fp32)
    keep = some_keep(5, widths, n, 0.7) if masked else np.ones_like(p, dtype=np.uint8)
    if masked:
        f.set_keep(keep)
    f.set_params(p)
    p = f.get_params()
    m, v, b1, b2, eps, lr = np.zeros_like(p), np.zeros_like(p), f32(0.9), f32(0.999), f32(1e-8), f32(1e-3)
    for k in range(1, 4):
        _, g = f.loss_grad(t)
        f.steps(t, 1, float(lr))
        m = fma(f32(1) - b1, g, b1 * m)
        v = fma((f32(1) - b2) * g, g, b2 * v)
        c1, c2 = f32(1.0 / (1.0 - float(b1) ** k)), f32(1.0 / (1.0 - float(b2) ** k))
        p = np.where(keep, p - lr * (m * c1) / (np.sqrt(v * c2) + eps), f32(0))
        got = f.get_params()
        assert p.dtype == f32 and np.mean(got != p) < 1e-5, (k, np.mean(got != p))
        p = got                                                    # (where the 64-bit sum rounded twice)
    f.close()
