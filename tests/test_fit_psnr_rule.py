"""When PSNR takes scratch memory, and how much at most: what the binding holds ready without asking the library."""
from paper_2306_16699_amd import rinr_fit


def test_the_binding_has_scratch_memory_ready_wherever_the_library_takes_it():
    L = rinr_fit.lib()
    images, elems = rinr_fit.PSNR_SHARED_IMAGES, rinr_fit.PSNR_SHARED_ELEMS
    most = 0
    for n in [*range(1, images), images, images + 1, 4096, 2 ** 31 - 1]:
        for e in [0, 1, 3072, elems - 1, elems, elems + 1, 10 ** 6, 2 ** 31, 2 ** 40]:
            need = L.rinr_psnr_workspace_bytes(n, e)
            assert (need > 0) == (n < images and e >= elems), (n, e)
            most = max(most, need)
    assert most == rinr_fit.PSNR_WORK_BYTES
    assert L.rinr_psnr_workspace_bytes(0, 10 ** 6) == 0
