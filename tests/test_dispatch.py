"""CPU-only checks of the rules that choose between kernels: what a kernel cannot address must not reach it."""
import ctypes

import pytest

from paper_2110_11199_amd import binding as Bd
from tests.test_gpu_lstm import ACROSS_XCDS

STAGED, DIRECT, SPLIT = 0, 1, 2


def _step_kind(precision, backward, pairs, hidden, batch):
    # adpsgd::rec_step_kind(int, bool, int, int, int), an internal symbol of the library
    return ctypes.CDLL(Bd.LIB_PATH)["_ZN6adpsgd13rec_step_kindEibiii"](precision, ctypes.c_bool(backward), pairs, hidden, batch)


@pytest.mark.parametrize("backward", [False, True])
@pytest.mark.parametrize("precision,esz,largest", [(Bd.FP32, 4, 16384), (Bd.BF16_GEMM, 2, 23168)])
def test_direct_step_kernels_only_where_32_bit_offsets_reach_all_of_w_h(precision, esz, largest, backward):
    step = 16 // esz
    for batch in (1, 33, 128):
        for pairs in (1, 2, 64):
            for hidden in (1024, 8192, largest, largest + step, 16640, 24000, 32768):
                kind = _step_kind(precision, backward, pairs, hidden, batch)
                # the furthest 16 bytes a lane of the direct kernels addresses: the last row of the fourth gate, a stage of 128 bytes
                furthest = (3 * hidden + hidden - 1) * hidden * esz + 128
                assert kind != DIRECT or furthest < 1 << 32, (pairs, hidden, batch)
    assert _step_kind(precision, backward, 2, largest, 64) == DIRECT
    assert _step_kind(precision, backward, 2, largest + step, 64) == STAGED


def test_small_batches_on_the_split_contraction_where_it_is_the_shorter():
    for pairs, hidden, batch in ((32, 640, 2), (32, 640, 32), (128, 512, 16)):
        assert _step_kind(Bd.FP32, False, pairs, hidden, batch) == SPLIT
        assert _step_kind(Bd.FP32, True, pairs, hidden, batch) == DIRECT
    for pairs, hidden, batch in ((48, 256, 32), (24, 512, 16), (16, 768, 8)):
        assert _step_kind(Bd.BF16_GEMM, True, pairs, hidden, batch) == SPLIT
        assert _step_kind(Bd.BF16_GEMM, False, pairs, hidden, batch) == DIRECT
    assert _step_kind(Bd.BF16_GEMM, True, 20, 768, 8) == DIRECT and _step_kind(Bd.FP32, False, 48, 1024, 2) == DIRECT


class _Gemm(ctypes.Structure):         # adpsgd::GemmDesc
    _fields_ = [(n, ctypes.c_int) for n in ("precision", "a_kc", "b_kc", "c_elem", "M", "N", "K")] + \
               [(n, ctypes.c_int64) for n in ("A", "lda", "sAi", "sAd", "B", "ldb", "sBi", "sBd", "C", "ldc", "sCi", "sCd", "bias", "sBiasI", "sBiasD")] + \
               [(n, ctypes.c_int) for n in ("groupsI", "groupsD", "k_padded", "tile")] + [("lmap", ctypes.c_uint8 * 128)]


class _Colsum(ctypes.Structure):       # adpsgd::ColsumDesc
    _fields_ = [("precision", ctypes.c_int), ("L", ctypes.c_int), ("lmap", ctypes.c_uint8 * 128), ("in_", ctypes.c_int64), ("ld", ctypes.c_int64), ("sIi", ctypes.c_int64),
                ("rows", ctypes.c_int64), ("N", ctypes.c_int), ("out", ctypes.c_int64), ("sOi", ctypes.c_int64), ("loss", ctypes.c_int64), ("row_loss", ctypes.c_int64),
                ("L_all", ctypes.c_int), ("active_bits", ctypes.c_uint32 * 4)]


class _Softmax(ctypes.Structure):      # adpsgd::SoftmaxDesc
    _fields_ = [("precision", ctypes.c_int), ("L", ctypes.c_int), ("lmap", ctypes.c_uint8 * 128), ("status", ctypes.c_int64), ("rows", ctypes.c_int64), ("C", ctypes.c_int),
                ("logits", ctypes.c_int64), ("ldl", ctypes.c_int64), ("sLi", ctypes.c_int64), ("y", ctypes.c_int64), ("sYi", ctypes.c_int64),
                ("dlogits", ctypes.c_int64), ("ldd", ctypes.c_int64), ("sDi", ctypes.c_int64), ("row_loss", ctypes.c_int64)]


class _Products(ctypes.Structure):     # adpsgd::GradProducts
    _fields_ = [("has_dx", ctypes.c_bool), ("has_cs", ctypes.c_bool), ("dx", _Gemm), ("ndw", ctypes.c_int), ("dw", _Gemm * 2), ("cs", _Colsum)]


def _gemm_desc(M, N, K, groups, a_kc=0, b_kc=0, precision=Bd.FP32):
    lda, ldb = (K if a_kc else M), (K if b_kc else N)
    return _Gemm(precision=precision, a_kc=a_kc, b_kc=b_kc, M=M, N=N, K=K, lda=lda, sAi=M * K, ldb=ldb, sBi=N * K, ldc=N, sCi=M * N, groupsI=groups, groupsD=1, tile=-1)


@pytest.mark.parametrize("M,N,K,groups,want", [
    (672, 1024, 2560, 8, 14), (672, 1024, 2564, 8, 15),      # six rounds of 64x64 tiles against two of 128x128
    (672, 1024, 4096, 8, 15), (672, 1024, 9000, 8, 15), (1344, 1024, 3000, 8, 15), (640, 640, 9000, 8, 15),
    (2688, 2048, 4096, 8, 14),                               # 42 rounds of 14 against 11 of 53
    (2048, 2048, 4096, 1, 15), (2048, 2048, 2048, 1, 14),    # 4 rounds of 14 against one of 60; 4 of 12.8 against one of 43
])
def test_fp32_tile_follows_the_rates_of_the_kernels_that_run_it(M, N, K, groups, want):
    # ns per k: on the bf16 matrix units 12.8 a round (15.5 alone) in 64x64 tiles, 36 (43) in 128x128; on fp32 MFMAs, K > 2560, 14 (20) and 53 (60)
    dma = ctypes.c_bool()
    pick = ctypes.CDLL(Bd.LIB_PATH)["_ZN6adpsgd14gemm_pick_tileERKNS_8GemmDescERb"]
    assert pick(ctypes.byref(_gemm_desc(M, N, K, groups, a_kc=1)), ctypes.byref(dma)) == want and dma.value


@pytest.mark.parametrize("M,N,K,groups,want", [
    (168, 5000, 40, 12, 15), (1344, 3000, 64, 12, 15), (1344, 3000, 96, 12, 15), (1344, 3000, 116, 12, 14),      # rows of C that are no whole 64 bytes
    (1280, 1280, 80, 6, 14), (3360, 1280, 64, 8, 14), (512, 1024, 64, 8, 15), (2000, 320, 80, 6, 15),            # rows that are: few rounds of 128x128, or many
])
def test_fp32_tile_of_short_contractions(M, N, K, groups, want):
    dma = ctypes.c_bool()
    pick = ctypes.CDLL(Bd.LIB_PATH)["_ZN6adpsgd14gemm_pick_tileERKNS_8GemmDescERb"]
    for kc in (0, 1):
        assert pick(ctypes.byref(_gemm_desc(M, N, K, groups, a_kc=kc, b_kc=kc)), ctypes.byref(dma)) == want and dma.value


@pytest.mark.parametrize("rows,states,K,learners,want", [
    (168, 5000, 40, 12, 15), (336, 300, 64, 8, 15), (672, 1000, 64, 8, 15),                        # us, 128x128 / 64x64: 20 / 19; 9.4 / 5.4; 13.1 / 12.6
    (1344, 3000, 64, 12, 14), (1344, 3000, 96, 12, 14), (5120, 200, 80, 8, 14),                    # 55 / 81, 69 / 92, 18 / 23
])
def test_fp32_tile_of_short_output_layers_whose_rows_of_logits_are_whole_lines(rows, states, K, learners, want):
    dma = ctypes.c_bool()
    pick = ctypes.CDLL(Bd.LIB_PATH)["_ZN6adpsgd14gemm_pick_tileERKNS_8GemmDescERb"]
    g = _gemm_desc(rows, states, K, learners, a_kc=1, b_kc=1)
    g.ldc = (states + 31) // 32 * 32
    g.sCi = rows * g.ldc
    assert pick(ctypes.byref(g), ctypes.byref(dma)) == want and dma.value


@pytest.mark.parametrize("frames,before,want", [(2016, 1920, 1), (2688, 2560, 2), (2688, 2624, 1), (4200, 4000, 1)])
def test_fp32_weight_gradients_of_a_layer_share_a_launch_whatever_their_length(frames, before, want):
    # (one that is long and one that is not run on kernels of either kind)
    g = _Products(ndw=2)
    g.dw[0], g.dw[1] = _gemm_desc(1280, 320, frames, 6), _gemm_desc(1280, 320, before, 6)
    apart = ctypes.c_bool()
    launches = ctypes.CDLL(Bd.LIB_PATH)["_ZN6adpsgd21grad_product_launchesERKNS_12GradProductsERb"]
    assert launches(ctypes.byref(g), ctypes.byref(apart)) == want


@pytest.mark.parametrize("learners,states,width,rows,apart", [
    (8, 9000, 256, 2048, False), (8, 9000, 256, 2049, True),       # 288 tiles of dW; 128 blocks of 128 rows of dX, 136
    (4, 9000, 512, 3840, False), (4, 9000, 512, 4096, True),       # 240 tiles of dX; 128 of 256x256, which dX takes then
    (10, 10600, 256, 1600, True),                                  # 420 tiles of dW: no third of two rounds empty
    (8, 9000, 64, 2688, False),                                    # dX in 64x64 tiles
])
def test_bf16_output_layer_behind_a_bottleneck_shares_a_launch_where_dx_leaves_half_of_the_chip(learners, states, width, rows, apart):
    # (the column sums are apart unless dW runs in tiles of which two fit a compute unit)
    g = _Products(has_dx=True, has_cs=True, ndw=1)
    g.dx = _gemm_desc(rows, width, states, learners, a_kc=1, precision=Bd.BF16_GEMM)
    g.dw[0] = _gemm_desc(states, width, rows, learners, precision=Bd.BF16_GEMM)
    g.dw[0].lda = (states + 63) // 64 * 64                         # (k-rows padded to whole chunks, as the handle lays them out)
    g.cs = _Colsum(precision=1, L=learners, ld=states, rows=rows, N=states)
    got = ctypes.c_bool()
    assert ctypes.CDLL(Bd.LIB_PATH)["_ZN6adpsgd21grad_product_launchesERKNS_12GradProductsERb"](ctypes.byref(g), ctypes.byref(got)) == 1
    assert got.value == apart


class _Rec(ctypes.Structure):          # adpsgd::RecDesc
    _fields_ = [(n, ctypes.c_int) for n in ("precision", "L", "D", "B", "H", "T")] + [("lmap", ctypes.c_uint8 * 128), ("direct", ctypes.c_int), ("step", ctypes.c_int)] + \
               [(n, ctypes.c_int64) for n in "gates sGi c sCi y sYi wh sWi sWd dy sDYi da sDAi dc sDCi dbp sDBi".split()]


@pytest.mark.parametrize("prec,shape,L,members", ACROSS_XCDS)
def test_numbers_of_clusters_that_are_meant_to_exchange_through_memory_do(prec, shape, L, members):
    r = _Rec(precision=prec, L=L, D=2 if shape.bidirectional else 1, B=shape.batch, H=shape.hidden, T=shape.frames, direct=1)
    supported = ctypes.CDLL(Bd.LIB_PATH)["_ZN6adpsgd21rec_cluster_supportedERKNS_7RecDescEbi"]
    supported.restype = ctypes.c_bool
    assert supported(ctypes.byref(r), ctypes.c_bool(False), 256) and supported(ctypes.byref(r), ctypes.c_bool(True), 256)
    clusters, units = L * r.D * -(-shape.batch // 16), 64 if prec else 32
    assert members * units >= shape.hidden and (members - 2) * units < shape.hidden
    one_xcd, anywhere = 256 // 8 // members * 8, 256 // members
    assert -(-clusters // one_xcd) > -(-clusters // anywhere)


@pytest.mark.parametrize("precision,rows,classes,width,want", [
    (Bd.BF16_GEMM, 4096, 40, 768, True), (Bd.BF16_GEMM, 2049, 4, 768, True), (Bd.BF16_GEMM, 2049, 4, 776, False), (Bd.BF16_GEMM, 2048, 4, 776, True),      # 258 workgroups, 256
    (Bd.BF16_GEMM, 2048, 32, 1024, True), (Bd.BF16_GEMM, 80, 4, 1032, False), (Bd.BF16_GEMM, 2049, 32, 1024, False), (Bd.BF16_GEMM, 80, 16, 2048, False),
    (Bd.BF16_GEMM, 336, 4, 8192, False), (Bd.BF16_GEMM, 336, 500, 64, True), (Bd.BF16_GEMM, 336, 512, 72, False), (Bd.FP32, 336, 200, 80, True), (Bd.FP32, 336, 208, 80, False),
])
def test_output_layer_and_softmax_share_a_launch_where_w_o_is_small_and_its_rows_are_short(precision, rows, classes, width, want):
    learners = 2
    ldd = (classes + 63) // 64 * 64
    g = _gemm_desc(rows, classes, width, learners, a_kc=1, b_kc=1, precision=precision)
    g.bias = 64
    sm = _Softmax(precision=precision, L=learners, rows=rows, C=classes, ldl=ldd, sLi=rows * ldd, ldd=ldd, sDi=rows * ldd)
    supported = ctypes.CDLL(Bd.LIB_PATH)["_ZN6adpsgd22output_small_supportedERKNS_8GemmDescERKNS_11SoftmaxDescE"]
    supported.restype = ctypes.c_bool
    assert supported(ctypes.byref(g), ctypes.byref(sm)) == want


@pytest.mark.parametrize("learners,params,copies,want", [
    (4, 350_000, False, 2), (8, 800_000, False, 2), (8, 900_000, False, 0), (12, 500_000, False, 2), (10, 700_000, False, 0), (16, 700_000, False, 0),
    (24, 600_000, False, 0), (32, 600_000, False, 0), (24, 1_000_000, False, 0),                   # flat vectors and fp32 models: one walk is the shorter from there
    (16, 737_000, True, 2), (32, 737_000, True, 2), (16, 1_000_000, True, 0), (5, 958_000, True, 2), (8, 1_050_000, True, 0),      # models with a bf16 copy: later
    (33, 300_000, False, 0), (3, 300_000, False, 0), (12, 20_000, False, 2), (64, 100_000, False, 4), (4, 8_388_608, False, 2), (8, 3_000_000, False, 0),
])
def test_delayed_mean_takes_two_learners_to_a_thread_where_that_is_the_shorter(learners, params, copies, want):
    rule = ctypes.CDLL(Bd.LIB_PATH)["_ZN6adpsgd22mean_learners_a_threadEilbb"]
    assert rule(learners, ctypes.c_int64(params), ctypes.c_bool(False), ctypes.c_bool(copies)) == want


@pytest.mark.parametrize("learners,params,want", [(4, 4 << 20, 2), (3, 4 << 20, 0), (8, 400_000, 2), (8, 7 << 16, 0), (16, 100_000, 2), (7, 100_000, 0), (64, 250_000, 2), (64, 400_000, 0)])
def test_synchronous_mean_takes_two_learners_to_a_thread_where_that_is_the_shorter(learners, params, want):
    rule = ctypes.CDLL(Bd.LIB_PATH)["_ZN6adpsgd22mean_learners_a_threadEilbb"]
    assert rule(learners, ctypes.c_int64(params), ctypes.c_bool(True), ctypes.c_bool(False)) == want
