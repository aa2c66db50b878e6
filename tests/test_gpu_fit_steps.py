"""Several Adam steps of the fit kernels: what they are made of, and that it does not matter how they are cut into calls and launches."""
import numpy as np
import pytest

from oracle import fit_oracle as fo
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


# every kernel that takes several steps a launch: padded widths 16 and 32, last tile whole and half-filled.  17 x 16 pixels are too few to share
@pytest.mark.parametrize("width,L", [(w, L) for w in (8, 15) for L in range(2, 9)] + [(w, L) for w in (24, 32) for L in (2, 3)])
@pytest.mark.parametrize("masked", [False, True])
def test_steps_of_one_launch_are_steps_of_their_own(width, L, masked):
    """One call of 32 steps and five more, then three, against a call for each: rates, corrections, error history, the form of the error's way down (which
    an image with large weights takes)."""
    widths, n, H, W = [2] + [width] * (L - 1) + [3], 5, 17, 16
    p = synth.init_params(11, widths, n).astype(f32)
    p[1::2] *= f32(2.0)
    rng = np.random.default_rng(L)
    import torch
    t = torch.from_numpy(rng.random((n, 3, H, W), dtype=f32)).cuda()
    keep = some_keep(5, widths, n, 0.7)
    got = []
    for calls in ([37, 3], [1] * 40):
        f = rinr_fit.Fit(widths, n, H, W)
        if masked:
            f.set_keep(keep)
        f.set_params(p)
        at = 0
        for k in calls:
            f.steps(t, k, 2e-3, t0=at, T=40)
            at += k
        got.append((f.get_params(), f.last_loss()))
        f.close()
    assert np.isfinite(got[0][0]).all() and np.isfinite(got[0][1]).all() and not np.array_equal(got[0][0], p)
    np.testing.assert_array_equal(got[0][0], got[1][0])
    np.testing.assert_array_equal(got[0][1], got[1][1])


# images of so many pixels that a launch takes fewer steps than 32, or one: with the rounds full, none is shared
@pytest.mark.parametrize("H,W,n", [(64, 64, 1024), (65, 64, 1024), (128, 128, 1024), (129, 128, 1024)])
def test_launches_of_fewer_steps(H, W, n):
    import torch
    widths = [2, 8, 3]
    p = synth.init_params(12, widths, n).astype(f32)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    t = torch.rand(n, 3, H, W, generator=g, device="cuda")
    got = []
    for calls in ([34], [1] * 34):
        f = rinr_fit.Fit(widths, n, H, W)
        f.set_params(p)
        for at, k in enumerate(calls):
            f.steps(t, k, 1e-3, t0=at, T=34)
        got.append((f.get_params(), f.last_loss()))
        f.close()
    np.testing.assert_array_equal(got[0][0], got[1][0])
    np.testing.assert_array_equal(got[0][1], got[1][1])


@pytest.mark.parametrize("width,L", [(8, 3), (15, 2), (15, 5), (24, 3), (32, 2)])
@pytest.mark.parametrize("masked", [False, True])
def test_one_launch_follows_the_oracle(width, L, masked):
    """The bars of the tests that go step by step: an entry whose gradient is lost in rounding may move the other way, few do."""
    widths, n, H, W, steps, lr = [2] + [width] * (L - 1) + [3], 8, 16, 16, 6, 1e-3
    p = synth.init_params(14, widths, n).astype(f32)
    keep = some_keep(6, widths, n, 0.7) if masked else np.ones_like(p, dtype=np.uint8)
    img = np.ascontiguousarray(synth.images(8, n, H, W))
    import torch
    f = rinr_fit.Fit(widths, n, H, W)
    if masked:
        f.set_keep(keep)
    f.set_params(p)
    f.steps(torch.from_numpy(img).cuda(), steps, lr, t0=0, T=8)
    got, loss = f.get_params(), f.last_loss()
    f.close()
    refs = [fo.fit(widths, p[i], img[i], steps, lr, T=8, keep=keep[i]) for i in range(n)]
    np.testing.assert_allclose(loss, [losses[-1] for _, losses in refs], rtol=3e-4)
    diff = np.abs(got - np.stack([r for r, _ in refs]))
    assert diff.max() <= 2.0 * steps * lr and np.mean(diff > 0.02 * lr) < 0.01, (diff.max(), np.mean(diff > 0.02 * lr))
    assert not got[keep == 0].any()
