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
    chunks, fits, most = (lib["_ZN4absk" + n] for n in ("19softmax_step_chunksEii", "17softmax_step_fitsEiiii", "23softmax_step_max_chunksEiiii"))
    fits.restype = C.c_bool
    for d in [1, 3, 255, 256, 257, 511, 512, 513, 640, 784, 1000, 1023, 1024, 1025, 1536, 2047, 2048, 2049]:
        for K, M in ((2, 1), (10, 4), (16, 40), (16, 1), (3, 300), (17, 4)):
            need = 0
            for b in range(2, 1101):
                if fits(K, d, b, M):
                    need = max(need, chunks(d, b))
                assert most(K, d, b, M) == need, (K, d, b)


# Which fp32 steps without hidden layers take one launch: up to 16 classes, 2048 features and 32 chunks; several chunks not for many small
# replicas nor where one work-group would add up many partial gradients of few replicas
@pytest.mark.parametrize("d,K,M,b,taken", [
    (256, 10, 4, 16, 1), (256, 10, 4, 512, 1), (784, 10, 4, 128, 1), (784, 16, 1, 1024, 0), (784, 16, 8, 1024, 1), (1, 2, 600, 64, 1), (1, 2, 600, 65, 0), (1, 17, 1, 2, 0),
    (2048, 16, 1, 16, 1), (2049, 2, 1, 16, 0), (64, 2, 384, 40, 1), (64, 2, 256, 96, 1), (64, 2, 257, 96, 0), (256, 2, 257, 96, 1), (256, 2, 682, 96, 1),
    (256, 2, 683, 96, 0), (23, 6, 540, 588, 0), (1511, 16, 1, 199, 0), (1511, 16, 8, 199, 1), (1511, 5, 1, 199, 1), (954, 11, 1, 58, 0), (954, 8, 1, 58, 1),
    (1372, 13, 2, 288, 1), (1372, 13, 2, 289, 0), (100, 7, 3, 1024, 1), (100, 7, 3, 1025, 0)])
def test_which_fp32_steps_take_one_launch(d, K, M, b, taken):
    f = B.load_library()["_ZN4absk17softmax_step_fitsEiiii"]
    f.restype = C.c_bool
    assert f(K, d, b, M) == bool(taken)


# Which launches take blocks of rows through all layers (mlp_rows.hip), and how many rows to a block: up to 512 wide hidden layers, 128 classes,
# 896 inputs, four layers; the tiles' are many rows of narrow layers and blocks that would be mostly empty or leave most CUs idle
@pytest.mark.parametrize("dims,M,b,rows", [
    ((784, 512, 512, 10), 8, 501, 16), ((784, 512, 512, 10), 8, 1000, 32), ((784, 512, 512, 10), 8, 2048, 64), ((784, 512, 512, 10), 8, 4096, 0),
    ((784, 256, 256, 10), 8, 4096, 32), ((784, 264, 10), 8, 431, 16), ((784, 264, 10), 8, 416, 0), ((8, 8, 2), 14, 145, 16), ((8, 8, 2), 14, 144, 0),
    ((896, 256, 128), 16, 160, 16), ((904, 256, 128), 16, 160, 0), ((896, 256, 129), 16, 160, 0), ((784, 520, 10), 16, 256, 0),
    ((784, 64, 64, 64, 10), 16, 160, 16), ((784, 64, 64, 64, 64, 10), 16, 160, 0), ((784, 10), 16, 160, 0),
    ((16, 56, 8, 8, 4), 24, 1024, 32), ((16, 56, 8, 8, 4), 24, 1025, 0), ((16, 56, 8, 8, 4), 31, 3547, 0), ((32, 40, 40, 16), 25, 4883, 0),
    ((64, 32, 224, 10), 16, 1500, 32), ((64, 32, 224, 10), 16, 4096, 0), ((64, 128, 10), 32, 8192, 0),
    # many of 32 rows: each hidden layer from 64, 128 on average, then to 1536 of them and 64 classes, from 320 inputs to 2048 and 96
    ((56, 128, 240, 40, 35), 20, 2902, 0), ((24, 64, 208, 112, 54), 39, 6218, 0), ((32, 152, 40, 256, 103), 95, 4599, 0), ((896, 248, 248, 8, 6), 35, 1726, 0),
    ((64, 64, 192, 64), 48, 1024, 32), ((64, 64, 192, 64), 48, 1025, 0), ((64, 64, 184, 64), 48, 1024, 0), ((64, 56, 200, 64), 48, 1024, 0),
    ((64, 64, 192, 65), 48, 1024, 0), ((320, 64, 192, 96), 64, 1024, 32), ((312, 64, 192, 64), 64, 1024, 0), ((320, 64, 192, 97), 64, 1024, 0),
    ((320, 64, 192, 96), 64, 1025, 0), ((64, 64, 192, 65), 24, 1024, 32),
    # 64 rows in one round only; replicas of less than half a block; half a round of wide layers behind few inputs
    ((264, 64, 10), 30, 517, 32), ((264, 64, 10), 28, 517, 64), ((400, 56, 272, 64, 18), 133, 77, 0), ((56, 16, 109), 273, 3, 0),
    ((56, 16, 109), 300, 15, 0), ((56, 16, 109), 300, 16, 32), ((8, 360, 104, 3), 14, 740, 0), ((8, 360, 104, 3), 16, 740, 64),
    ((48, 288, 78), 14, 640, 0), ((784, 512, 512, 10), 8, 1025, 64)])
def test_which_steps_take_blocks_of_rows(dims, M, b, rows):
    f = B.load_library()["_ZN4absk14mlp_rows_blockEiPKiiix"]
    assert f(len(dims) - 1, (C.c_int * len(dims))(*dims), b, M, C.c_longlong(60000)) == rows


# Which steps take forward, head and backward-data in one launch of chains (gemm_small.hip): two to four layers whose launches are all 32-row
# tiles, up to 224 blocks of 32 rows, which more of them are slower in
@pytest.mark.parametrize("dims,M,b,taken", [
    ((784, 512, 512, 10), 8, 32, 1), ((784, 512, 512, 10), 8, 64, 1), ((784, 512, 512, 10), 8, 501, 0), ((8, 8, 2), 2, 2, 1), ((72, 40, 32), 3, 65, 1), ((72, 40, 33), 3, 65, 0),
    ((264, 72, 104, 17), 2, 96, 1), ((40, 1096, 64, 8, 5), 2, 40, 1), ((1096, 136, 520, 10), 1, 66, 1), ((40, 24, 24, 24, 24, 6), 2, 33, 0),
    ((8, 2), 4, 32, 0), ((16, 48, 10), 224, 4, 1), ((16, 48, 10), 225, 4, 0), ((56, 16, 10), 486, 6, 0), ((56, 16, 10), 112, 33, 1), ((56, 16, 10), 113, 33, 0)])
def test_which_steps_take_chains_of_tiles(dims, M, b, taken):
    f = B.load_library()["_ZN4absk16small_chain_fitsEiPKiiixS1_"]
    f.restype = C.c_bool
    assert f(len(dims) - 1, (C.c_int * len(dims))(*dims), b, M, C.c_longlong(60000), None) == bool(taken)


# Partial sums of squares that a weight gradient's launch leaves, a slot to each wavefront of each of its tiles: tiles of 128 x 128, 64 x 128
# and, by GemmP::fine, 256 x 256 outputs
@pytest.mark.parametrize("fine,tile,waves", [(0, (128, 128), 4), (1, (64, 128), 4), (2, (256, 256), 8)])
def test_slots_of_weight_gradient_tiles(fine, tile, waves):
    lib = B.load_library()
    shape, slots = (lib["_ZN4absk" + n] for n in ("21gemm_bf16_wgrad_shapeEiiiiiPKi", "19gemm_bf16_upd_slotsEiiiiiiPKi"))
    for Md, Nd in ((512, 512), (128, 128), (520, 136), (264, 784)):
        assert shape(Md, Nd, 4096, 8, 0, None) == 1
        assert slots(Md, Nd, 4096, 8, 0, fine, None) == -(-Md // tile[0]) * -(-Nd // tile[1]) * waves, (Md, Nd)


# Replicas of one work-group each and few features: more than 384 of them are faster in the general launches, except with inner products
@pytest.mark.parametrize("d,K,M,b,ip,taken", [
    (7, 14, 743, 10, 0, 0), (7, 14, 743, 10, 1, 1), (30, 4, 500, 8, 0, 0), (95, 2, 385, 64, 0, 0), (95, 2, 384, 64, 0, 1), (96, 2, 5000, 64, 0, 1),
    (2, 10, 4, 16, 0, 1), (64, 2, 384, 40, 0, 1), (64, 2, 385, 40, 0, 0), (64, 2, 256, 96, 0, 1), (1, 2, 600, 65, 1, 0), (17, 17, 4, 16, 1, 0)])
def test_which_replicas_of_one_work_group_take_one_launch(d, K, M, b, ip, taken):
    f = B.load_library()["_ZN4absk18softmax_step_takenEiiiii"]
    f.restype = C.c_bool
    assert f(K, d, b, M, ip) == bool(taken)
