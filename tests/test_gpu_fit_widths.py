"""Split-precision fit kernels of models that leave half of their last 16-unit tile empty (widths 8 below a multiple of 16), and layers' inputs
that wait in LDS, against the fp64 oracle: every depth there is a kernel for, widths at either end, ragged and masked models."""
import numpy as np
import pytest

from oracle import fit_oracle as fo
from paper_2306_16699_amd import rinr_fit, synth
from test_gpu_fit import keep_flags, targets_of

pytestmark = pytest.mark.gpu

BAR = 2e-5            # of the largest gradient entry, as in the suite's other gradient tests


def check(widths, n=2, H=9, W=15, keep=None, gain=1.0, copies=1):
    p0 = np.tile((synth.init_params(41, widths, n) * gain).astype(np.float32), (copies, 1))
    tgt, tgt_d = targets_of(43, n, H, W)
    tgt_d = tgt_d.repeat(copies, 1, 1, 1)
    n, first = n * copies, n
    if keep is not None:
        keep = np.tile(keep, (copies, 1))
    f = rinr_fit.Fit(widths, n, H, W)
    assert f.kernel_family == rinr_fit.KERNEL_SPLIT16
    if keep is not None:
        f.set_keep(keep)
    f.set_params(p0)
    loss, grad = f.loss_grad(tgt_d)
    f.close()
    for i in list(range(first)) + list(range(n - first if copies > 1 else n, n)):
        k = None if keep is None else keep[i]
        p = p0[i].astype(np.float64) if k is None else p0[i].astype(np.float64) * k
        want_loss, want_g = fo.loss_grad(widths, p, tgt[i % first], k)
        assert abs(loss[i] - want_loss) <= BAR * want_loss
        assert np.abs(grad[i] - want_g).max() <= BAR * np.abs(want_g).max(), widths


@pytest.mark.parametrize("L", range(2, 13))
def test_every_depth_of_half_filled_tiles(L):
    for width in (8, 5, 1, 24, 17, 21) + ((40, 33, 37) if L <= 10 else ()) + ((56, 49, 51) if L <= 6 else ()):
        check([2] + [width] * (L - 1) + [3])


@pytest.mark.parametrize("L", range(2, 13))
def test_every_depth_where_a_workgroup_takes_many_pixels(L):
    """With many images a workgroup takes a whole one, and the kernels of half-filled tiles run from 256 pixels a share (49 to 56 units:
    832 times the depth less 3) on: just below that and at it."""
    for width in (8, 24, 17) + ((40, 33) if L <= 10 else ()):
        for H, W in ((15, 17), (16, 16), (17, 17)):
            check([2] + [width] * (L - 1) + [3], H=H, W=W, copies=600)
    if 4 <= L <= 6:
        for width, H in ((56, 26 * (L - 3)), (49, 26 * (L - 3)), (51, 26 * (L - 3) - 1)):
            check([2] + [width] * (L - 1) + [3], n=1, H=H, W=32, copies=1024)


def test_masks_and_large_weights_where_a_workgroup_takes_many_pixels():
    """The other forms of the same kernels."""
    for widths in ([2, 40, 3, 40, 3], [2, 7, 39, 16, 3], [2, 24, 5, 20, 3], [2, 17, 16, 18, 3]):
        check(widths, n=3, H=17, W=16, keep=keep_flags(np.random.default_rng(5), widths, 3, 0.6), copies=400)
        check(widths, n=3, H=17, W=16, gain=2.0, copies=400)
    for gain in (1.0, 2.0):
        widths = [2, 56, 24, 50, 3]
        check(widths, n=1, H=32, W=27, keep=keep_flags(np.random.default_rng(6), widths, 1, 0.6), gain=gain, copies=1024)


@pytest.mark.parametrize("widths", [[2, 40, 3, 40, 3], [2, 7, 39, 16, 3], [2, 33, 32, 31, 34, 3], [2, 1, 40, 3], [2, 8, 1, 7, 3], [2, 3, 8, 3], [2, 24, 5, 20, 3], [2, 56, 24, 50, 3], [2, 17, 16, 18, 3]], ids=str)
@pytest.mark.parametrize("masked", [False, True])
def test_layers_of_unequal_width(widths, masked):
    keep = keep_flags(np.random.default_rng(5), widths, 3, 0.6) if masked else None
    check(widths, n=3, H=17, W=13, keep=keep)


@pytest.mark.parametrize("width,L", [(40, 3), (36, 5), (8, 4), (24, 5), (56, 4)])
def test_large_weights_take_the_form_that_scales_the_cosine(width, L):
    """A layer whose estimated gain is above 1.4 applies its factor of the error to the cosine: the second form of the kernels."""
    check([2] + [width] * (L - 1) + [3], gain=2.0)


@pytest.mark.parametrize("width,L", [(15, 3), (16, 4), (12, 9), (24, 5), (32, 4), (30, 7), (46, 3), (40, 4), (8, 10), (20, 6), (24, 8), (56, 3)])
def test_many_chunks_of_pixels(width, L):
    """Layers' inputs wait in LDS from the forward to the backward pass: many chunks one after the other, the last one ragged."""
    check([2] + [width] * (L - 1) + [3], n=2, H=61, W=47)
