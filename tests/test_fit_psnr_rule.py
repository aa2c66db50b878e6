"""When PSNR takes scratch memory: the binding asks the library only where the answer may be other than none."""
from paper_2306_16699_amd import rinr_fit


def test_the_binding_asks_wherever_the_library_takes_scratch_memory():
    L = rinr_fit.lib()
    images, elems = rinr_fit.PSNR_SHARED_IMAGES, rinr_fit.PSNR_SHARED_ELEMS
    for n in [1, 2, 3, 50, images - 1, images, images + 1, 4096, 2 ** 31 - 1]:
        for e in [0, 1, 3072, elems - 1, elems, elems + 1, 10 ** 6, 2 ** 31, 2 ** 40]:
            assert (L.rinr_psnr_workspace_bytes(n, e) > 0) == (n < images and e >= elems), (n, e)
    assert L.rinr_psnr_workspace_bytes(0, 10 ** 6) == 0
