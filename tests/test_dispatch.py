"""CPU-only checks of the rules that choose between kernels: what a kernel cannot address must not reach it."""
import ctypes

import pytest

from paper_2110_11199_amd import binding as Bd

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
