"""Split-precision fit kernels of models that leave half of their last 16-unit tile empty (widths 8 below a multiple of 16), and layers' inputs
that wait in LDS, against the fp64 oracle: every depth there is a kernel for, widths at either end, ragged and masked models."""
import numpy as np
import pytest

from oracle import fit_oracle as fo
from paper_2306_16699_amd import rinr_fit, synth
from test_gpu_fit import keep_flags, targets_of

pytestmark = pytest.mark.gpu

BAR = 2e-5            # of the largest gradient entry, as in the suite's other gradient tests


def units(widths, half):
    """What the handle says its kernels compute of a layer: the widest layer's last tile by half, or whole."""
    step = 8 if half else 16
    return -(-max(widths[1:-1]) // step) * step


def half_from(width, L):
    """Pixels of a workgroup's share from which a handle takes the half-filled kernel."""
    if width <= 8:
        return 0
    if width <= 24 and L >= 8:
        return 448 if L == 8 else 257
    return 256 if width <= 40 else 832 * (L - 3)


def error_factors(widths, p, w0=30.0):
    """The power of two each layer but the first multiplies the error by on the way down: the nearest to the inverse of its estimated gain."""
    out = []
    for l, (W, _) in enumerate(rinr_fit.split_params(widths, p)):
        if l > 0:
            gain = 0.7 * np.sqrt((W.astype(np.float64) ** 2).sum() / widths[l]) * (w0 / (2 * np.pi) if l < len(widths) - 2 else 1.0)
            out.append(2.0 ** np.rint(-np.log2(gain)))
    return out


def with_large_layers(widths, p0, keep=None, factor=0.25):
    """Image i with an estimated gain of 4 in layer 1 + i.  What makes it large are the weights of one of the layer's inputs, its last
    unit, whose own weights are zero: that unit is always 0, so the model computes what the others make of it, as well conditioned as
    before, and only the error that arrives at it is large."""
    p0 = p0.copy()
    for i, p in enumerate(p0):
        l = 1 + i % (len(widths) - 2)
        mats = rinr_fit.split_params(widths, p)                          # views
        kept = np.ones(widths[l + 1]) if keep is None else rinr_fit.split_params(widths, keep[i])[l][0][:, -1]
        assert kept.any()
        mats[l - 1][0][-1], mats[l - 1][1][-1] = 0.0, 0.0
        size = 1.0 / factor / 0.7 * np.sqrt(widths[l] / kept.sum()) / (30.0 / (2 * np.pi) if l < len(widths) - 2 else 1.0)
        mats[l][0][:, -1] = size * np.where(np.arange(widths[l + 1]) % 2, -1.0, 1.0)
        q = p if keep is None else p * keep[i]
        assert error_factors(widths, q)[l - 1] < 1.0, (widths, l)
    return p0


def check(widths, n=2, H=9, W=15, keep=None, copies=1, half=None, large=False):
    """half: whether the handle takes the kernel of a half-filled last tile.  large: n images with a layer each that multiplies the error by
    more than 1.4, which makes their workgroups take the form that scales the cosine."""
    if large:
        n = len(widths) - 2
    p0 = synth.init_params(41, widths, n)
    if large:
        p0 = with_large_layers(widths, p0, keep)
    p0 = np.tile(p0, (copies, 1))
    tgt, tgt_d = targets_of(43, n, H, W)
    tgt_d = tgt_d.repeat(copies, 1, 1, 1)
    n, first = n * copies, n
    if keep is not None:
        keep = np.tile(keep, (copies, 1))
    f = rinr_fit.Fit(widths, n, H, W)
    assert f.kernel_family == rinr_fit.KERNEL_SPLIT16
    if half is not None:
        assert f.kernel_units == units(widths, half), (widths, H, W)
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
        off, want = np.abs(grad[i] - want_g), np.abs(want_g)
        if large:        # at the suite's bar with the large error's unit in the measure of the others: its gradient by the size of the weights that bring it
            l = 1 + i % first
            norms = np.sqrt((rinr_fit.split_params(widths, p)[l][0] ** 2).sum(0))
            for v in (off, want):
                row = rinr_fit.split_params(widths, v)[l - 1]
                row[0][-1] /= norms[-1] / norms[:-1].max()
                row[1][-1] /= norms[-1] / norms[:-1].max()
        assert off.max() <= BAR * want.max(), (widths, i)


@pytest.mark.parametrize("L", range(2, 13))
def test_every_depth_where_a_workgroup_takes_few_pixels(L):
    """Up to 8 units the kernels of half-filled tiles run at any size, above that those of whole tiles do."""
    for width in (8, 5, 1, 24, 17, 21) + ((40, 33, 37) if L <= 10 else ()) + ((56, 49, 51) if L <= 6 else ()):
        check([2] + [width] * (L - 1) + [3], half=width <= 8)


@pytest.mark.parametrize("L", range(2, 13))
def test_every_depth_where_a_workgroup_takes_many_pixels(L):
    """With many images a workgroup takes a whole one, and the kernels of half-filled tiles run from 256 pixels a share on (8 layers of 17 to 24
    units 448, more of them 257; 49 to 56 units 832 times the depth less 3): just below that and at it."""
    for width in (8, 24, 17) + ((40, 33) if L <= 10 else ()):
        for H, W in ((15, 17), (16, 16), (17, 17)) if (width > 24 or L != 8) else ((17, 17), (21, 21), (16, 28)):
            check([2] + [width] * (L - 1) + [3], H=H, W=W, copies=600, half=H * W >= half_from(width, L))
    if 4 <= L <= 6:
        for width, H in ((56, 26 * (L - 3)), (49, 26 * (L - 3)), (51, 26 * (L - 3) - 1)):
            check([2] + [width] * (L - 1) + [3], n=1, H=H, W=32, copies=1024, half=width != 51)


def test_masks_where_a_workgroup_takes_many_pixels():
    for widths in ([2, 40, 3, 40, 3], [2, 7, 39, 16, 3], [2, 24, 5, 20, 3], [2, 17, 16, 18, 3], [2] + [24] * 11 + [3], [2] + [40] * 9 + [3]):
        check(widths, n=3, H=17, W=16, keep=keep_flags(np.random.default_rng(5), widths, 3, 0.6), copies=400, half=True)
    widths = [2, 56, 24, 50, 3]
    check(widths, n=1, H=32, W=27, keep=keep_flags(np.random.default_rng(6), widths, 1, 0.6), copies=1024, half=True)


@pytest.mark.parametrize("L", range(2, 13))
def test_large_layers_take_the_form_that_scales_the_cosine(L):
    """A layer whose estimated gain is above 1.4 applies its factor of the error to the cosine: the second form of every half-filled kernel, each
    layer of a model in turn."""
    copies = -(-1200 // (L - 1))
    for width in (8, 5, 24, 17) + ((40, 33) if L <= 10 else ()):
        check([2] + [width] * (L - 1) + [3], H=28 if half_from(width, L) > 257 else 17, W=16, copies=copies, half=True, large=True)
    if 4 <= L <= 6:
        for width in (56, 49):
            check([2] + [width] * (L - 1) + [3], H=26 * (L - 3), W=32, copies=1024 // (L - 1), half=True, large=True)


def test_large_layers_under_a_mask():
    for widths in ([2, 7, 8, 6, 3], [2, 24, 5, 20, 3], [2, 40, 9, 40, 38, 3]):
        keep = keep_flags(np.random.default_rng(5), widths, len(widths) - 2, 0.6)
        check(widths, H=17, W=16, keep=keep, copies=-(-1200 // (len(widths) - 2)), half=True, large=True)


@pytest.mark.parametrize("width,L", [(15, 3), (16, 5), (12, 8), (30, 4), (32, 6), (46, 3), (48, 5), (47, 10), (64, 4), (63, 6)])
def test_large_layers_of_whole_tiles(width, L):
    check([2] + [width] * (L - 1) + [3], H=13, W=9, half=False, large=True)


@pytest.mark.parametrize("widths", [[2, 8, 8, 3], [2, 24, 20, 24, 3], [2] + [40] * 9 + [3], [2] + [17] * 11 + [3]], ids=str)
@pytest.mark.parametrize("large", [False, True])
def test_adam_steps_of_half_filled_kernels(widths, large):
    """Four steps against the oracle's, at the bars of the suite's other trajectories, where the half-filled kernel runs."""
    H, W, n, steps, lr, T = 16, 17, len(widths) - 2, 4, 5e-4, 10
    copies = -(-1200 // n)
    p0 = synth.init_params(5, widths, n)
    if large:
        p0 = with_large_layers(widths, p0)
    tgt, tgt_d = targets_of(13, n, H, W)
    f = rinr_fit.Fit(widths, n * copies, H, W)
    assert f.kernel_units == units(widths, True)
    f.set_params(np.tile(p0, (copies, 1)))
    many, losses = tgt_d.repeat(copies, 1, 1, 1), []
    for s in range(steps):
        f.steps(many, 1, lr, t0=s, T=T)
        losses.append(f.last_loss())
    got = f.get_params()
    f.close()
    for i in range(n):
        ref, ref_losses = fo.fit(widths, p0[i], tgt[i], steps, lr, T=T)
        for j in (i, n * (copies - 1) + i):
            np.testing.assert_allclose([x[j] for x in losses], ref_losses, rtol=3e-4)
            diff = np.abs(got[j] - ref)
            assert diff.max() <= 2.0 * steps * lr
            assert np.mean(diff > 0.02 * lr) < 0.01, np.mean(diff > 0.02 * lr)


@pytest.mark.parametrize("widths", [[2, 40, 3, 40, 3], [2, 7, 39, 16, 3], [2, 33, 32, 31, 34, 3], [2, 1, 40, 3], [2, 8, 1, 7, 3], [2, 3, 8, 3], [2, 24, 5, 20, 3], [2, 56, 24, 50, 3], [2, 17, 16, 18, 3]], ids=str)
@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("many", [False, True])
def test_layers_of_unequal_width(widths, masked, many):
    keep = keep_flags(np.random.default_rng(5), widths, 3, 0.6) if masked else None
    if many:
        check(widths, n=3, H=26, W=33, keep=keep, copies=341, half=max(widths) <= 40 or len(widths) == 5)
    else:
        check(widths, n=3, H=17, W=13, keep=keep, half=max(widths) <= 8)


@pytest.mark.parametrize("width,L", [(15, 3), (16, 4), (12, 9), (24, 5), (32, 4), (30, 7), (46, 3), (40, 4), (8, 10), (20, 6), (24, 8), (56, 3)])
def test_many_chunks_of_pixels(width, L):
    """Layers' inputs wait in LDS from the forward to the backward pass: many chunks one after the other, the last one ragged."""
    check([2] + [width] * (L - 1) + [3], n=2, H=61, W=47)
