"""Host-only checks of the workspace plan: every batch up to the cap fits what is reserved for the cap (no GPU call is made)."""
import ctypes as C

import pytest

from paper_2406_13936_amd import binding as B


def _workspace(dims, prec, M, cap, mask=3, N=8192):
    arr = (C.c_int * len(dims))(*dims)
    cfg = B._Config(len(dims) - 1, arr, 1, 1, prec, M, cap, 0, 0, 0.9, 0.999, 1e-8, 0, mask, None, None, 0)
    n = C.c_size_t(0)
    assert B.load_library().abs_workspace_bytes(C.byref(cfg), N, C.byref(n)) == 0
    return n.value


# The chunks of the one-launch fp32 step are no monotone function of the batch (16 samples each up to b = 128 of 512 to 1024 features, 32 above)
@pytest.mark.parametrize("dims", [(512, 10), (784, 10), (1024, 16), (513, 2), (256, 10), (2048, 16), (1, 2)])
def test_the_workspace_never_shrinks_as_the_cap_grows(dims):
    sizes = [_workspace(dims, B.PREC_F32, 4, cap) for cap in range(2, 1101)]
    assert all(a <= b for a, b in zip(sizes, sizes[1:]))


def test_the_chunks_reserved_for_a_cap_cover_every_batch_up_to_it():
    lib = B.load_library()
    chunks, fits, most = (lib["_ZN4absk" + n] for n in ("19softmax_step_chunksEii", "17softmax_step_fitsEiii", "23softmax_step_max_chunksEiii"))
    for d in [1, 3, 255, 256, 257, 511, 512, 513, 640, 784, 1000, 1023, 1024, 1025, 1536, 2047, 2048, 2049]:
        for K in (2, 10, 16, 17):
            need = 0
            for b in range(2, 1101):
                if fits(K, d, b):
                    need = max(need, chunks(d, b))
                assert most(K, d, b) == need, (K, d, b)
