"""GPU parity of the fitting kernels (include/rinr_fit.h) against the fp64 encode oracle."""
import numpy as np
import pytest

from oracle import fit_oracle as fo
from oracle import oracle as dec
from paper_2306_16699_amd import rinr, rinr_fit, synth

pytestmark = pytest.mark.gpu

ARCHS = {
    "cifar 3x15 @32x32": ([2, 15, 15, 3], 32, 32),
    "flowers 10x32 ragged": ([2] + [32] * 9 + [3], 24, 20),
    "mini-imagenet 10x40 ragged": ([2] + [40] * 9 + [3], 17, 13),
    "width 64 x6": ([2] + [64] * 6 + [3], 16, 16),
    "tapered": ([2, 24, 48, 32, 3], 9, 31),
    "narrow, 6 layers": ([2] + [12] * 5 + [3], 11, 9),             # the deep kernel of the width-16 class
    "12 layers x 20": ([2] + [20] * 11 + [3], 10, 10),            # the deep kernel of the width-32 class, the API's depth limit
    "width 20": ([2, 20, 20, 3], 13, 11),                          # widths round up to 8: 24 ...
    "widths 50, 56": ([2, 50, 56, 50, 3], 10, 9),                 # ... and 56
    "width 64 x3": ([2, 64, 64, 64, 3], 12, 11),                  # full padded widths: the bias unit takes a column tile of its own
    "widths 48, 16 exact": ([2, 48, 16, 48, 3], 9, 14),
    "widths 64, 17, 33": ([2, 64, 17, 33, 3], 8, 19),
    "one unit between wide layers": ([2, 1, 64, 1, 3], 7, 6),
    "one hidden unit": ([2, 1, 3], 5, 7),
    "one pixel": ([2, 8, 3], 1, 1),
}


def targets_of(seed, n, H, W):
    import torch
    t = synth.images(seed, n, H, W)
    return t, torch.from_numpy(t).cuda()


def keep_flags(rng, widths, n, prob):
    ks = []
    for _ in range(n):
        mats = [(rng.uniform(size=(widths[l + 1], widths[l])) < prob).astype(np.uint8) for l in range(len(widths) - 1)]
        ks.append(rinr_fit.weight_keep_flags(widths, mats))
    return np.stack(ks)


FAMILIES = {"split16": False, "fp32": True}      # the two kernel families of rinr_fit_create_ex, each held to the same bars


@pytest.mark.parametrize("family", list(FAMILIES))
@pytest.mark.parametrize("name", list(ARCHS))
@pytest.mark.parametrize("masked", [False, True])
def test_loss_and_gradient(name, masked, family):
    widths, H, W = ARCHS[name]
    n = 3
    rng = np.random.default_rng(len(name))
    p0 = synth.init_params(7, widths, n)          # the method's own initial scale: larger weights make deep sine nets chaotic in fp32
    tgt, tgt_d = targets_of(11, n, H, W)
    keep = keep_flags(rng, widths, n, 0.6) if masked else None
    lo, hi = (0.0, 1.0) if "tapered" in name else (-1.0, 1.0)
    f = rinr_fit.Fit(widths, n, H, W, coord_lo=lo, coord_hi=hi, fp32=FAMILIES[family])
    # the split-precision kernels serve every shape here but 7 layers x 64, which only the fp32 kernels hold
    want_family = rinr_fit.KERNEL_FP32 if (FAMILIES[family] or name == "width 64 x6") else rinr_fit.KERNEL_SPLIT16
    assert f.kernel_family == want_family
    if keep is not None:
        f.set_keep(keep)
    f.set_params(p0)
    loss, grad = f.loss_grad(tgt_d)
    got_p = f.get_params()
    for i in range(n):
        k = None if keep is None else keep[i]
        pe = p0[i].astype(np.float64) if k is None else p0[i].astype(np.float64) * k
        assert np.array_equal(got_p[i], pe.astype(np.float32))              # masked parameters were zeroed
        want_loss, want_g = fo.loss_grad(widths, pe, tgt[i], k, lo=lo, hi=hi)
        assert abs(loss[i] - want_loss) <= 2e-5 * want_loss + 1e-9, (i, loss[i], want_loss)
        scale = np.abs(want_g).max()
        err = np.abs(grad[i] - want_g).max()
        print(f'{name} masked={masked} image {i}: loss rel err {abs(loss[i] - want_loss) / want_loss:.1e}, grad err / max|grad| {err / scale:.1e}')
        assert err <= 2e-5 * scale + 1e-9, (i, err, scale)
        if k is not None:
            assert not grad[i][k == 0].any()
    # the printed sum of Eq. 1 (loss_scale = 1) differs from the mean by the factor 3 H W only
    loss1, grad1 = f.loss_grad(tgt_d, loss_scale=1.0)
    np.testing.assert_allclose(loss1, loss * 3 * H * W, rtol=1e-5)
    np.testing.assert_allclose(grad1, grad * 3 * H * W, rtol=1e-4, atol=1e-6 * np.abs(grad1).max())
    f.close()


@pytest.mark.parametrize("width,L", [(16, 2), (16, 4), (15, 5), (16, 7), (16, 8), (12, 12), (31, 4), (32, 5), (32, 6), (17, 7), (32, 8), (29, 9),
                                     (32, 12), (47, 4), (33, 5), (48, 7), (48, 8), (48, 10), (64, 2), (64, 3), (49, 4), (64, 5), (64, 6)])
def test_split_kernels_at_the_edges_of_their_depth_buckets(width, L):
    """Every depth bucket at its deepest model and at the first one past the bucket before it, gradient against the oracle."""
    widths, H, W, n = [2] + [width] * (L - 1) + [3], 9, 15, 2
    p0 = synth.init_params(41, widths, n)
    tgt, tgt_d = targets_of(43, n, H, W)
    f = rinr_fit.Fit(widths, n, H, W)
    assert f.kernel_family == rinr_fit.KERNEL_SPLIT16
    f.set_params(p0)
    loss, grad = f.loss_grad(tgt_d)
    f.close()
    for i in range(n):
        want_loss, want_g = fo.loss_grad(widths, p0[i].astype(np.float64), tgt[i], None)
        assert abs(loss[i] - want_loss) <= 2e-5 * want_loss
        assert np.abs(grad[i] - want_g).max() <= 2e-5 * np.abs(want_g).max()


@pytest.mark.parametrize("width,L", [(9, 3), (16, 6), (14, 9), (16, 10), (13, 11), (18, 2), (32, 3), (25, 10), (32, 11), (40, 2), (48, 3), (41, 6), (40, 9)])
def test_split_kernels_at_the_other_depths(width, L):
    """The depths between: there is a kernel for each."""
    test_split_kernels_at_the_edges_of_their_depth_buckets(width, L)


@pytest.mark.parametrize("family", list(FAMILIES))
@pytest.mark.parametrize("widths,n,H,W", [([2, 15, 15, 3], 40000, 7, 9), ([2, 40, 40, 3], 4200, 9, 15), ([2, 30, 3], 20000, 5, 26)])
def test_many_images_and_few_agree_with_the_oracle(widths, n, H, W, family):
    """With many images a workgroup takes a whole image and updates it itself; with few, workgroups share an image's pixels
    and a second launch adds their gradients up.  The same image through both: gradient against the oracle, one Adam step."""
    import torch
    few = 3
    p0 = synth.init_params(3, widths, few)
    tgt, tgt_d = targets_of(5, few, H, W)
    got = {}
    for m in (few, n):
        f = rinr_fit.Fit(widths, m, H, W, fp32=FAMILIES[family])
        f.set_params(np.tile(p0, ((m + few - 1) // few, 1))[:m])
        t = tgt_d.repeat((m + few - 1) // few, 1, 1, 1)[:m].contiguous()
        loss, grad = f.loss_grad(t)
        f.steps(t, 1, 5e-4)
        got[m] = loss[-few:], grad[-few:], f.get_params()[-few:], f.last_loss()[-few:]
        f.close()
    order = [(n - few + i) % few for i in range(few)]                 # which image the last slots of the big batch hold
    for i in range(few):
        want_loss, want_g = fo.loss_grad(widths, p0[order[i]].astype(np.float64), tgt[order[i]], None)
        for m, k in ((few, order[i]), (n, i)):
            loss, grad, params, last = got[m]
            assert abs(loss[k] - want_loss) <= 2e-5 * want_loss and last[k] == loss[k]
            assert np.abs(grad[k] - want_g).max() <= 2e-5 * np.abs(want_g).max()
            clear = np.abs(grad[k]) > 1e-4 * np.abs(grad[k]).max()    # the first Adam step is lr in the gradient's direction
            np.testing.assert_allclose((p0[order[i]] - params[k])[clear], 5e-4 * np.sign(want_g[clear]), rtol=1e-3, atol=1e-7)


@pytest.mark.parametrize("family", list(FAMILIES))
@pytest.mark.parametrize("name", ["cifar 3x15 @32x32", "mini-imagenet 10x40 ragged", "tapered"])
def test_adam_steps_follow_the_oracle(name, family):
    widths, H, W = ARCHS[name]
    n, steps, lr, T = 2, 4, 5e-4, 10
    rng = np.random.default_rng(3)
    p0 = synth.init_params(5, widths, n)
    tgt, tgt_d = targets_of(13, n, H, W)
    keep = keep_flags(rng, widths, n, 0.8)
    f = rinr_fit.Fit(widths, n, H, W, fp32=FAMILIES[family])
    f.set_keep(keep)
    f.set_params(p0)
    losses = []
    for s in range(steps):                  # one step per call, so that every step's loss can be read
        f.steps(tgt_d, 1, lr, t0=s, T=T)
        losses.append(f.last_loss())
    got = f.get_params()
    for i in range(n):
        ref, ref_losses = fo.fit(widths, p0[i], tgt[i], steps, lr, T=T, keep=keep[i])
        np.testing.assert_allclose([l[i] for l in losses], ref_losses, rtol=3e-4)
        diff = np.abs(got[i] - ref)
        # Adam normalises the step to about lr whatever the gradient's size, so an entry whose gradient is
        # lost in fp32 rounding may move the other way: allow that for a few entries, hold the rest tight
        assert diff.max() <= 2.0 * steps * lr
        assert np.mean(diff > 0.02 * lr) < 0.01, np.mean(diff > 0.02 * lr)
        assert not got[i][keep[i] == 0].any()
    # the same four steps in one call
    f.set_params(p0)
    f.steps(tgt_d, steps, lr, t0=0, T=T)
    np.testing.assert_array_equal(f.get_params(), got)
    f.close()


@pytest.mark.parametrize("widths,n", [([2, 1, 3], 1), ([2, 15, 15, 3], 1), ([2, 15, 15, 3], 3), ([2] + [40] * 9 + [3], 173)])
def test_start_of_a_fit_under_a_mask(widths, n):
    """Pruned parameters are zero and all others keep their bits, whichever of mask and parameters comes first, whatever the count
    leaves behind its last four (and beyond one pass of the grid); a new mask leaves the moments, new parameters clear them."""
    rng = np.random.default_rng(6)
    p0 = synth.init_params(8, widths, n)
    keep, other = keep_flags(rng, widths, n, 0.7), keep_flags(rng, widths, n, 0.5)
    _, tgt = targets_of(9, n, 4, 3)
    f = rinr_fit.Fit(widths, n, 4, 3)
    f.set_params(p0)
    np.testing.assert_array_equal(f.get_params(), p0)
    f.set_keep(keep)
    np.testing.assert_array_equal(f.get_params(), np.where(keep, p0, np.float32(0)))
    f.set_params(p0)
    np.testing.assert_array_equal(f.get_params(), np.where(keep, p0, np.float32(0)))
    f.steps(tgt, 2, 1e-3, t0=0, T=8)
    moved = f.get_params()
    f.set_keep(other)
    np.testing.assert_array_equal(f.get_params(), np.where(other, moved, np.float32(0)))
    f.set_keep(None)
    f.set_params(p0)
    f.steps(tgt, 2, 1e-3, t0=0, T=8)
    again = f.get_params()
    g = rinr_fit.Fit(widths, n, 4, 3)
    g.set_params(p0)
    g.steps(tgt, 2, 1e-3, t0=0, T=8)
    np.testing.assert_array_equal(again, g.get_params())       # nothing is left of the first fit: moments, error history
    # a mask that prunes nothing, set in the middle: the moments and the count of steps go on (without them this step would be 0.64 lr where it is
    # near lr); only the error's scale starts anew, which moves no more than rounding
    f.set_keep(np.ones_like(keep))
    f.steps(tgt, 1, 1e-3, t0=2, T=8)
    g.steps(tgt, 1, 1e-3, t0=2, T=8)
    off = np.abs(f.get_params() - g.get_params())
    assert np.mean(off > 0.02e-3) < 0.01 and off.max() <= 2e-3
    f.close()
    g.close()


def test_split_kernels_carry_the_error_at_any_size():
    """The split-precision kernels carry the back-propagated error in fp16 times a power of two chosen from the size of
    the error (the last step's, once there is one) and from the weights' gains.  Parity of the gradient must not depend on
    that size: loss scales from 1e-9 to 1e3, targets far off the prediction, and the state after some steps, when the
    scale comes from the steps' own history."""
    widths, H, W, n = [2, 24, 40, 24, 3], 12, 10, 2
    p0 = synth.init_params(31, widths, n)
    tgt, tgt_d = targets_of(37, n, H, W)
    f = rinr_fit.Fit(widths, n, H, W)
    assert f.kernel_family == rinr_fit.KERNEL_SPLIT16
    f.set_params(p0)

    def check(targets, targets_d, params, loss_scale):
        loss, grad = f.loss_grad(targets_d, loss_scale=loss_scale)
        assert np.isfinite(grad).all() and np.isfinite(loss).all()
        ls = loss_scale if loss_scale else 1.0 / (3 * H * W)
        for i in range(n):
            want_loss, want_g = fo.loss_grad(widths, params[i].astype(np.float64), targets[i], None)
            want_loss, want_g = want_loss * ls * 3 * H * W, want_g * ls * 3 * H * W
            assert abs(loss[i] - want_loss) <= 2e-5 * want_loss
            assert np.abs(grad[i] - want_g).max() <= 2e-5 * np.abs(want_g).max(), (loss_scale, i)

    for ls in (0.0, 1e-9, 1.0, 1e3):
        check(tgt, tgt_d, p0, ls)
    far = (tgt * 40.0 - 7.0).astype(np.float32)                       # errors of tens, not fractions
    import torch
    check(far, torch.from_numpy(far).cuda(), p0, 0.0)
    f.steps(tgt_d, 60, 1e-3, t0=0, T=60)                              # the scale now follows the steps' own error
    check(tgt, tgt_d, f.get_params(), 0.0)
    check(far, torch.from_numpy(far).cuda(), f.get_params(), 0.0)        # ... and is wrong by two orders for these targets
    f.close()


@pytest.mark.parametrize("family", list(FAMILIES))
@pytest.mark.parametrize("width,L", [(16, 3), (15, 7), (16, 8), (24, 4), (32, 12), (40, 3), (48, 7), (40, 10), (64, 4), (64, 6)])
def test_large_weights_lose_nothing_on_the_way_down(width, L, family):
    """A layer that multiplies the error by far more than one: its small weights arrive with all their bits.  With zero weights
    below it every pre-activation is 0 and every cosine 1, and one unit alone gets an error from above, a power of two, so
    the bias gradient of each unit is one weight times a power of two."""
    H = W = 4
    widths = [2] + [width] * (L - 1) + [3]
    rng = np.random.default_rng(width + L)
    small = rng.uniform(0.02, 0.2, (2, width)) * rng.choice([-1.0, 1.0], (2, width))
    p0 = np.zeros((2, fo.n_params(widths)), np.float32)
    mats = [rinr_fit.split_params(widths, p) for p in p0]
    mats[0][L - 1][0][0] = small[0]                           # image 0: the output layer, channel 0
    mats[0][L - 1][0][1:] = 40.0                              # (channels 1 and 2 set the layer's size and see no error)
    mats[1][L - 2][0][:] = 40.0                               # image 1: the last hidden layer, unit 2
    mats[1][L - 2][0][2] = small[1]
    mats[1][L - 1][0][0, 2] = 1.0
    tgt = np.zeros((2, 3, H, W), np.float32)
    tgt[:, 0] = -8.0                                          # the output is 0: an error of 8 in channel 0
    import torch
    f = rinr_fit.Fit(widths, 2, H, W, fp32=FAMILIES[family])
    f.set_params(p0)
    _, grad = f.loss_grad(torch.from_numpy(tgt).cuda(), loss_scale=2.0 ** -10)
    f.close()
    for i, l in ((0, L - 2), (1, L - 3)):
        _, want = fo.loss_grad(widths, p0[i].astype(np.float64), tgt[i], None, loss_scale=2.0 ** -10)
        got, want = rinr_fit.split_params(widths, grad[i])[l][1], rinr_fit.split_params(widths, want)[l][1]
        # split of the weight 2^-23 of itself or 2^-25; split of the error, toward zero twice, 2^-20 of itself or 2^-24 (it is 0.3 or
        # more); sum over 16 equal terms and six factors in fp32
        bound = (2.0 ** -23 + 2.0 ** -25 / 0.02 + 2.0 ** -20 + 2.0 ** -24 / 0.3 + 21 * 2.0 ** -24) * np.abs(want)
        assert want.all() and np.all(np.abs(got - want) <= bound), (i, np.max(np.abs(got / want - 1.0)))


@pytest.mark.parametrize("widths,H,W,steps,lr,tol", [([2, 15, 15, 3], 32, 32, 600, 2e-3, 2e-3),
                                                     ([2] + [32] * 4 + [3], 40, 56, 400, 1e-3, 2e-2),
                                                     ([2] + [40] * 9 + [3], 48, 48, 400, 5e-4, 0.5)],
                         ids=["3x15", "5x32", "10x40"])
def test_both_kernel_families_train_alike(widths, H, W, steps, lr, tol):
    """Whole fits, loss falling by an order of magnitude, with the split-precision and the fp32 kernels from the same start:
    the losses stay together at every quarter of the schedule (shallow models: to 1e-3; a 10-layer sine network amplifies
    any rounding difference over hundreds of Adam steps, so there the two must only reach the same quality)."""
    import torch
    n = 6
    tgt = torch.from_numpy(synth.images(3, n, H, W)).cuda()
    traj = {}
    for name, fp32 in FAMILIES.items():
        f = rinr_fit.Fit(widths, n, H, W, fp32=fp32)
        f.set_params(synth.init_params(9, widths, n))
        first, _ = f.loss_grad(tgt, want_grad=False)
        stages = []
        for k in range(4):
            f.steps(tgt, steps // 4, lr, t0=k * (steps // 4), T=steps)
            stages.append(f.last_loss().copy())
        traj[name] = np.array(stages)
        assert np.isfinite(traj[name]).all()
        assert np.all(traj[name][-1] < 0.2 * first), (name, first, traj[name][-1])
        f.close()
    rel = np.abs(traj["split16"] - traj["fp32"]) / traj["fp32"]
    assert rel.max() <= tol, rel.max(axis=1)


def test_fit_prune_quantise_pack_decode_round_trip():
    import torch
    widths, H, W, n = [2, 24, 24, 24, 3], 24, 24, 8
    tgt, tgt_d = targets_of(17, n, H, W)
    f = rinr_fit.Fit(widths, n, H, W)
    f.set_params(synth.init_params(19, widths, n))
    l0, _ = f.loss_grad(tgt_d, want_grad=False)
    f.steps(tgt_d, 600, 2e-3, t0=0, T=600)
    l1 = f.last_loss()
    assert np.all(l1 < 0.1 * l0), (l0, l1)
    psnr = -10.0 * np.log10(l1)                                  # mean squared error on a 0..1 scale
    assert psnr.min() > 22.0, psnr
    # dynamic pruning (Sec. IV-A): ratio from each image's PSNR, magnitude masks per weight matrix, re-fit
    p = f.get_params()
    keeps, mats_all = [], []
    for i in range(n):
        ratio = rinr_fit.prune_ratio(0, float(psnr[i]) + 8.0)      # shifted so that this small test prunes something
        mats = [rinr_fit.l1_mask(w, ratio).reshape(w.shape) for w, _ in rinr_fit.split_params(widths, p[i])]
        mats_all.append(mats)
        keeps.append(rinr_fit.weight_keep_flags(widths, mats))
    f.set_keep(np.stack(keeps))
    f.reset_optimizer()
    f.steps(tgt_d, 300, 1e-3, t0=0, T=300)
    l2 = f.last_loss()
    assert np.all(l2 < 0.2 * l0), (l0, l2)                       # pruned and re-fitted: still a fit, if a coarser one
    p = f.get_params()
    assert not p[np.stack(keeps) == 0].any()
    # quantise the hidden layers to 8 bits (Sec. IV-B), pack, decode with the decode kernels
    models = [rinr_fit.to_model(widths, p[i], mats_all[i], hidden_bits=8) for i in range(n)]
    st = rinr.Store(rinr.pack(models))
    ids = torch.arange(n, dtype=torch.int64, device="cuda")
    out = st.decode_batch(ids, H, W).cpu().numpy()
    ref = dec.decode(models, np.arange(n), H, W)
    assert np.abs(out - ref).max() <= 1e-3
    mse_q = ((out - tgt) ** 2).reshape(n, -1).mean(axis=1)
    psnr_q = -10.0 * np.log10(mse_q)
    assert np.all(psnr_q > -10.0 * np.log10(l2) - 3.0), (psnr_q, -10.0 * np.log10(l2))   # 8-bit hidden layers cost little
    st.close()
    f.close()


def test_encode_images_is_the_sequence_of_its_steps():
    """rinr_encode_images (Sec. IV in one call) against the same procedure issued call by call through the
    entry points the tests above check one by one: the two blobs are the same bytes."""
    import ctypes as C
    import torch
    widths, H, W, n = [2, 24, 24, 24, 3], 24, 24, 6
    tgt, tgt_d = targets_of(23, n, H, W)
    p0 = synth.init_params(29, widths, n)
    sched, first, fit_steps, refit_steps, lr, refit_lr = 0, 0.2, 500, 200, 2e-3, 1e-3
    f = rinr_fit.Fit(widths, n, H, W)
    f.set_params(p0)
    blob, psnr = f.encode(tgt_d, sched, first, fit_steps, refit_steps, lr, refit_lr, hidden_bits=8)
    final = f.get_params()
    f.close()

    g = rinr_fit.Fit(widths, n, H, W)
    g.set_params(p0)
    g.steps(tgt_d, fit_steps, lr, t0=0, T=fit_steps)
    keep_mats = [None] * n
    for rnd in range(2):
        p = g.get_params()
        if rnd == 1:
            loss, _ = g.loss_grad(tgt_d, want_grad=False)
        keeps = []
        for i in range(n):
            ratio = first if rnd == 0 else rinr_fit.prune_ratio(sched, -10.0 * np.log10(float(loss[i])))
            prev = keep_mats[i]
            keep_mats[i] = [rinr_fit.l1_mask(w, ratio, None if prev is None else prev[l]).reshape(w.shape)
                            for l, (w, _) in enumerate(rinr_fit.split_params(widths, p[i]))]
            keeps.append(rinr_fit.weight_keep_flags(widths, keep_mats[i]))
        g.set_keep(np.stack(keeps))
        g.reset_optimizer()
        g.steps(tgt_d, refit_steps, refit_lr, t0=0, T=refit_steps)
    loss, _ = g.loss_grad(tgt_d, want_grad=False)
    p = g.get_params()
    np.testing.assert_array_equal(p, final)
    np.testing.assert_allclose(psnr, -10.0 * np.log10(loss), rtol=0, atol=1e-4)
    models = [rinr_fit.to_model(widths, p[i], keep_mats[i], hidden_bits=8) for i in range(n)]
    want = rinr.pack(models)
    assert blob.size == want.size and np.array_equal(blob, want)
    g.close()
    # it is a store: opens, decodes to the quality the call reported (8-bit hidden layers cost little)
    pruned = 1.0 - np.mean([np.concatenate([k.ravel() for k in keep_mats[i]]).mean() for i in range(n)])
    assert pruned >= first - 0.01, pruned
    st = rinr.Store(blob)
    out = st.decode_batch(torch.arange(n, dtype=torch.int64, device="cuda"), H, W).cpu().numpy()
    psnr_q = -10.0 * np.log10(((out - tgt) ** 2).reshape(n, -1).mean(axis=1))
    assert np.all(psnr_q > psnr - 3.0), (psnr_q, psnr)
    assert psnr.min() > 20.0, psnr
    st.close()

    # errors: a blob that does not fit reports the size needed; options out of range
    h = rinr_fit.Fit(widths, 2, 8, 8)
    h.set_params(p0[:2])
    t2 = torch.from_numpy(np.ascontiguousarray(tgt[:2, :, :8, :8])).cuda()
    L = rinr_fit.lib()
    o = rinr_fit.EncodeOpts(0, 0.0, 3, 2, 1e-3, 1e-3, 8)
    size = C.c_size_t()
    small = np.empty(16, np.uint8)
    assert L.rinr_encode_images(h._h, t2.data_ptr(), C.byref(o), None, small.ctypes.data, 16, C.byref(size), None) == rinr.E_SIZE
    bound = C.c_size_t()
    assert L.rinr_encode_blob_bound(h._h, 8, C.byref(bound)) == 0 and 16 < size.value <= bound.value
    for bad in (rinr_fit.EncodeOpts(3, 0.0, 3, 2, 1e-3, 1e-3, 8), rinr_fit.EncodeOpts(0, 1.5, 3, 2, 1e-3, 1e-3, 8),
                rinr_fit.EncodeOpts(0, 0.0, -1, 2, 1e-3, 1e-3, 8), rinr_fit.EncodeOpts(0, 0.0, 3, 2, 0.0, 1e-3, 8),
                rinr_fit.EncodeOpts(0, 0.0, 3, 2, 1e-3, 1e-3, 9)):
        assert L.rinr_encode_images(h._h, t2.data_ptr(), C.byref(bad), None, small.ctypes.data, 16, C.byref(size), None) == rinr.E_ARG
    assert L.rinr_encode_images(None, t2.data_ptr(), C.byref(o), None, small.ctypes.data, 16, C.byref(size), None) == rinr.E_NULL
    h.close()


def test_fit_argument_errors_and_empty():
    import torch
    with pytest.raises(rinr.RinrError) as e:
        rinr_fit.Fit([3, 8, 3], 1, 4, 4)
    assert e.value.code == rinr.E_ARG
    with pytest.raises(rinr.RinrError) as e:
        rinr_fit.Fit([2, 65, 3], 1, 4, 4)
    assert e.value.code == rinr.E_ARG
    with pytest.raises(rinr.RinrError):
        rinr_fit.Fit([2, 8, 3], 1, 0, 4)
    # depth limits per width: 12 linear layers up to width 32, 10 up to 48, 7 up to 64
    for widths, ok in (([2] + [32] * 11 + [3], True), ([2] + [33] * 11 + [3], False), ([2] + [48] * 9 + [3], True),
                       ([2] + [48] * 10 + [3], False), ([2] + [64] * 6 + [3], True), ([2] + [64] * 7 + [3], False),
                       ([2] + [8] * 12 + [3], False)):
        if ok:
            rinr_fit.Fit(widths, 1, 4, 4).close()
        else:
            with pytest.raises(rinr.RinrError) as e:
                rinr_fit.Fit(widths, 1, 4, 4)
            assert e.value.code in (rinr.E_UNSUPPORTED, rinr.E_ARG), widths
    f = rinr_fit.Fit([2, 8, 3], 0, 4, 4)
    f.steps(torch.empty((0, 3, 4, 4), device="cuda"), 3, 1e-3)
    assert f.get_params().shape == (0, f.n_params)
    f.close()
    f = rinr_fit.Fit([2, 8, 3], 1, 4, 4)
    t = torch.zeros((1, 3, 4, 4), device="cuda")
    with pytest.raises(rinr.RinrError):
        f.steps(t, -1, 1e-3)
    with pytest.raises(rinr.RinrError):
        f.steps(t, 1, 1e-3, beta1=1.5)
    f.close()


def test_psnr_batch_matches_the_oracle():
    import torch
    rng = np.random.default_rng(21)
    for n, shape in ((5, (3, 17, 13)), (3, (3, 64, 64)), (2, (1,)), (4, (3, 224, 224))):
        a = rng.uniform(0, 1, (n,) + shape).astype(np.float32)
        b = np.clip(a + rng.normal(scale=0.03, size=a.shape), 0, 1).astype(np.float32)
        b[0] = a[0]                                             # identical pair: +inf
        got = rinr_fit.psnr_batch(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()).cpu().numpy()
        assert np.isinf(got[0]) and got[0] > 0
        for i in range(1, n):
            assert abs(got[i] - fo.psnr(a[i], b[i])) < 2e-4, (shape, i, got[i], fo.psnr(a[i], b[i]))
        got255 = rinr_fit.psnr_batch(torch.from_numpy(a * 255).cuda(), torch.from_numpy(b * 255).cuda(), peak=255.0).cpu().numpy()
        np.testing.assert_allclose(got255[1:], got[1:], atol=2e-3)
    # a view that is 4- but not 16-byte aligned takes the scalar path
    base = torch.from_numpy(rng.uniform(0, 1, 2 * 101 + 1).astype(np.float32)).cuda()
    x, y = base[1:].view(2, 101), (base[1:] * 0.5).view(2, 101).contiguous()
    got = rinr_fit.psnr_batch(x, y).cpu().numpy()
    xh = base[1:].cpu().numpy().reshape(2, 101)
    for i in range(2):
        assert abs(got[i] - fo.psnr(xh[i], xh[i] * 0.5)) < 2e-4
    with pytest.raises(rinr.RinrError):
        rinr_fit.psnr_batch(x, y, peak=0.0)
