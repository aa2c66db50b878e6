"""Decode of models whose widest layer does not fill its tiles: half of the last 16-row tile, one quad less of a 32-row tile, and
the odd last quad in a step of its own, at the widths where the padding starts and ends, in every kind of store, against the
fp64 oracle."""
import numpy as np
import pytest

from oracle import oracle
from paper_2306_16699_amd import rinr, synth
from test_gpu_parity import TIGHT, check_split_blocks, check_workload, ids_dev, image_like, torch  # noqa: F401

pytestmark = pytest.mark.gpu

WIDTHS = (1, 7, 8, 9, 15, 16, 17, 23, 24, 25, 33, 39, 40, 41, 47, 48, 49, 55, 56, 57)


def models_of(width, kind, sines=4):
    bits = {"ints": [0, 8, 5, 6], "fp32": [0] * 4, "16 bits": [0, 16, 16, 16], "mixed": [0, 8, 0, 16]}[kind][:sines] + [0]
    taper = ([width, max(1, width - 1)] + [max(1, width // 2), width])[:sines]          # the widest first and last, odd inner layers
    return (synth.make_models(70 + width, np.arange(2), width, sines, bits, 0.6) +
            synth.make_models(71 + width, np.arange(1), width, sines, bits, None, widths=taper))


class Batch:
    w0, coord_lo, coord_hi, H, W = 30.0, -1.0, 1.0, 9, 23
    image_ids = np.array([0, 2, 1, 2])


@pytest.mark.parametrize("kind", ["ints", "fp32", "16 bits", "mixed"])
def test_every_width_of_a_class(torch, kind):  # noqa: F811
    for width in WIDTHS:
        b = Batch()
        b.models = image_like(models_of(width, kind))
        check_workload(torch, b, u8=True)                       # every kernel family, at the suite's bars


@pytest.mark.parametrize("kind", ["ints", "fp32", "mixed"])
def test_operand_blocks_and_streamed_layers_of_half_filled_tiles(torch, kind):  # noqa: F811
    """The blocks element by element (every copy of a weight that a step holds twice must agree), and the streamed kernels' bytes."""
    for width in (8, 24, 40, 48, 56):
        ms = models_of(width, kind)
        blob = rinr.pack(ms)
        st = rinr.Store(blob)
        for mi, m in enumerate(ms):
            for li, ly in enumerate(m.layers):
                check_split_blocks(st, mi, li, len(m.layers), ly, oracle.dequant(ly).astype(np.float32))
        deep = rinr.pack(synth.make_models(72 + width, np.arange(2), width, 14, [0] + [8 if kind == "ints" else 0] * 13 + [0], 0.8))
        big, small = rinr.Store(deep), rinr.Store(deep, lds_budget=20 * 1024)
        ids = ids_dev(torch, [1, 0, 1])
        for flags in (0, rinr.FLAG_FP16_ACT | rinr.FLAG_FP16_UNCHECKED, rinr.FLAG_FP16_ALL | rinr.FLAG_FP16_UNCHECKED):
            a, b = (s.decode_batch_ex(ids, 31, 17, rinr.OUT_F32, flags) for s in (big, small))
            assert torch.equal(a, b) and (width < 24 or small.last_launch_info()["streamed"]), (width, flags)
        for s in (st, big, small):
            s.close()


def test_all_widths_in_one_grid(torch):  # noqa: F811
    """One launch for a store of all widths: every model takes the body of its own width."""
    ms = sum((models_of(w, "ints") for w in WIDTHS), [])
    st = rinr.Store(rinr.pack(ms))
    sel = np.arange(len(ms))[::-1]
    got = st.decode_batch_ex(ids_dev(torch, sel), 65, 64, rinr.OUT_F32, rinr.FLAG_NO_CLAMP).cpu().numpy()
    assert st.last_launch_info()["launches"] == 1 and st.status() == 0
    assert np.abs(got - oracle.decode(ms, sel, 65, 64, clamp=False)).max() <= TIGHT
    st.close()


def test_streamed_layers_of_a_store_of_all_widths(torch):  # noqa: F811
    """Deep models of every width: streamed by the bodies of the one grid, for the bytes of the resident kernels."""
    ms = sum((synth.make_models(90 + w, np.arange(1), w, 14, [0] + [8] * 13 + [0], 0.8) for w in (8, 16, 24, 32, 40, 48, 56, 64)), [])
    blob = rinr.pack(ms)
    big, small = rinr.Store(blob), rinr.Store(blob, lds_budget=20 * 1024)
    ids = ids_dev(torch, np.arange(len(ms))[::-1].copy())
    for flags in (0, rinr.FLAG_FP16_ACT | rinr.FLAG_FP16_UNCHECKED, rinr.FLAG_FP16_ALL | rinr.FLAG_FP16_UNCHECKED):
        a, b = (s.decode_batch_ex(ids, 31, 17, rinr.OUT_F32, flags) for s in (big, small))
        assert torch.equal(a, b) and small.last_launch_info()["streamed"], flags
    big.close()
    small.close()


@pytest.mark.parametrize("n,H,W", [(1, 1, 1), (1, 65, 129), (3, 8, 8), (40, 64, 63), (255, 16, 17), (257, 9, 23)])
def test_splits_of_ragged_batches(torch, n, H, W):  # noqa: F811
    """However a ragged batch is split over workgroups, with the order's scratch and without: the bytes of one workgroup an image."""
    ms = image_like(synth.ragged_pool(5, 48))
    st = rinr.Store(rinr.pack(ms))
    sel = (np.arange(n) * 7) % len(ms)
    ids, ws = ids_dev(torch, sel), torch.empty(rinr.workspace_bytes(n), dtype=torch.uint8, device="cuda")
    got = st.decode_batch_ex(ids, H, W, rinr.OUT_F32)
    tiles = -(-H * W // 64)
    assert st.last_launch_info()["workgroups"] > n or tiles <= 8
    copies = -(-torch.cuda.get_device_properties(0).multi_processor_count // n)            # a workgroup a CU is then one for each image, or less
    whole = st.decode_batch_ex(ids.repeat(copies), H, W, rinr.OUT_F32, blocks_per_cu=1)
    assert st.last_launch_info()["workgroups"] == n * copies
    for k in range(copies):
        assert torch.equal(got, whole[k * n:k * n + n]), k
    assert torch.equal(got, st.decode_batch_ex(ids, H, W, rinr.OUT_F32, workspace=ws))
    some = np.unique(np.linspace(0, n - 1, 13).astype(int))
    assert np.abs(got.cpu().numpy()[some] - oracle.decode(ms, sel[some], H, W)).max() <= TIGHT
    st.close()


@pytest.mark.parametrize("W", [1, 2, 3, 7, 31, 33, 62, 63, 64, 65, 66, 127, 128, 129, 1000])
def test_rows_and_columns_of_every_pixel(torch, W):  # noqa: F811
    """A lane's row and column follow from those of its tile's first pixel: rows shorter than a tile, as long, a little longer."""
    ms = models_of(16, "fp32", 2) + models_of(24, "ints", 2)
    st = rinr.Store(rinr.pack(ms))
    for H in (1, 2, 67):
        sel = np.array([0, 5, 2, 3])
        got = st.decode_batch_ex(ids_dev(torch, sel), H, W, rinr.OUT_F32, rinr.FLAG_NO_CLAMP).cpu().numpy()
        assert np.abs(got - oracle.decode(ms, sel, H, W, clamp=False)).max() <= TIGHT, (H, W)
    st.close()
