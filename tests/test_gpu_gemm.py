"""GPU: the grouped MFMA GEMM against a float64 numpy product."""
import numpy as np
import pytest

from tests.gpu_util import rel_err, to_bf16_bits, from_bf16_bits

pytestmark = pytest.mark.gpu


def _run(prec, a_k, b_k, c_elem, M, N, K, groups, bias, pad=0, seed=0, tile=-1):
    import torch
    from paper_2110_11199_amd import binding as Bd
    r = np.random.default_rng(seed)
    dev = torch.device("cuda:0")
    r4 = lambda v: (v + 3) // 4 * 4
    lda = r4(K if a_k else M) + pad
    ldb = r4(K if b_k else N) + pad
    ldc = N + pad
    A = r.standard_normal((groups, M if a_k else K, lda)).astype(np.float32)
    B = r.standard_normal((groups, N if b_k else K, ldb)).astype(np.float32)
    bv = r.standard_normal((groups, N)).astype(np.float32) if bias else None
    if prec:
        A, B = from_bf16_bits(to_bf16_bits(A)), from_bf16_bits(to_bf16_bits(B))
        dA = torch.from_numpy(to_bf16_bits(A).view(np.int16)).to(dev)
        dB = torch.from_numpy(to_bf16_bits(B).view(np.int16)).to(dev)
    else:
        dA, dB = torch.from_numpy(A).to(dev), torch.from_numpy(B).to(dev)
    cdt = torch.int16 if (prec and c_elem) else torch.float32
    dC = torch.full((groups, M, ldc), 7, dtype=cdt, device=dev)
    dbias = torch.from_numpy(bv).to(dev) if bias else None
    Bd.adpsgd_gemm(prec, a_k, b_k, c_elem, M, N, K, dA.data_ptr(), lda, dA[0].numel(), dB.data_ptr(), ldb,
                   dB[0].numel(), dC.data_ptr(), ldc, M * ldc, dbias.data_ptr() if bias else None, N, groups,
                   torch.cuda.current_stream().cuda_stream, tile_config=tile)
    torch.cuda.synchronize()
    got = dC.cpu().numpy()
    if prec and c_elem:
        got = from_bf16_bits(got.view(np.uint16))
    Am = A[:, :, :K] if a_k else A[:, :, :M].transpose(0, 2, 1)
    Bm = B[:, :, :K] if b_k else B[:, :, :N].transpose(0, 2, 1)
    ref = np.einsum("gmk,gnk->gmn", Am.astype(np.float64), Bm.astype(np.float64))
    if bias:
        ref += bv[:, None, :]
    if pad:
        assert (got[:, :, N:] == (from_bf16_bits(np.array([7], np.uint16))[0] if (prec and c_elem) else 7)).all()
    return rel_err(got[:, :, :N], ref)


LAYOUTS = [(1, 1), (1, 0), (0, 0), (0, 1)]


@pytest.mark.parametrize("a_k,b_k", LAYOUTS)
@pytest.mark.parametrize("M,N,K", [(128, 128, 64), (200, 136, 100), (80, 256, 40), (257, 129, 260), (4, 4, 4)])
def test_gemm_fp32(a_k, b_k, M, N, K):
    print("gemm fp32", a_k, b_k, M, N, K, flush=True)
    assert _run(0, a_k, b_k, 0, M, N, K, 3, True, pad=4) < 2e-6
    assert _run(0, a_k, b_k, 1, M, N, K, 1, False) < 2e-6


@pytest.mark.parametrize("a_k,b_k", LAYOUTS)
@pytest.mark.parametrize("M,N,K", [(128, 128, 64), (200, 136, 100), (80, 256, 40), (257, 132, 260), (4, 8, 12)])
def test_gemm_bf16(a_k, b_k, M, N, K):
    print("gemm bf16", a_k, b_k, M, N, K, flush=True)
    # operands are exactly representable in bf16, so only the fp32 accumulation differs
    assert _run(1, a_k, b_k, 0, M, N, K, 3, True, pad=8) < 2e-6
    assert _run(1, a_k, b_k, 0, M, N, K, 2, False, pad=4) < 2e-6      # 8-byte aligned rows only
    assert _run(1, a_k, b_k, 1, M, N, K, 1, True) < 6e-3             # bf16 output rounding


@pytest.mark.parametrize("a_k,b_k", LAYOUTS)
@pytest.mark.parametrize("M,N,K,pad", [(520, 520, 192, 0), (520, 520, 192, 8), (516, 524, 128, 0), (516, 524, 128, 4),
                                         (264, 776, 100, 0), (520, 520, 64, 0), (520, 516, 448, 8)])
def test_gemm_bf16_large_tiles(a_k, b_k, M, N, K, pad):
    # enough 256x256 tiles (>= 128 over the groups) for the large-tile kernels: direct-to-LDS loads
    # when K is a multiple of 64 and all rows are 16-byte aligned (row counts need not be multiples of 8: pad=4
    # makes the k-rows of a 516-row operand 520 long), else register staging; K = 64 ... 448 is 2 ... 14 stages of
    # the direct-to-LDS main loop (its first, steady-state and last stages are separate code)
    print("gemm bf16 large", a_k, b_k, M, N, K, pad, flush=True)
    groups = 16 if N < 600 else 22
    assert _run(1, a_k, b_k, 0, M, N, K, groups, True, pad=pad) < 2e-6
    assert _run(1, a_k, b_k, 1, M, N, K, groups, False, pad=pad) < 6e-3


@pytest.mark.parametrize("a_k,b_k", LAYOUTS)
@pytest.mark.parametrize("M,N,K,pad", [(520, 516, 512, 0), (776, 520, 576, 8)])
def test_gemm_bf16_long_k_loop(a_k, b_k, M, N, K, pad):
    # 16 and 18 K stages of the hand-pipelined main loop (its steady state)
    print("gemm bf16 long K", a_k, b_k, M, N, K, pad, flush=True)
    assert _run(1, a_k, b_k, 0, M, N, K, 16, True, pad=pad) < 2e-6
    assert _run(1, a_k, b_k, 1, M, N, K, 16, False, pad=pad) < 6e-3


@pytest.mark.parametrize("variant", [11, 12, 13])
@pytest.mark.parametrize("a_k,b_k", LAYOUTS)
@pytest.mark.parametrize("K", [64, 128, 192, 256])
def test_gemm_bf16_forced_large_tile_configurations(variant, a_k, b_k, K):
    # the pipelined main loops (11: 64-k stages, 12 and 13: 32-k stages) have separate code for their first
    # stages, their steady state and their last stages: 1 .. 4 and 2 .. 8 stages here, in every operand layout
    # (the automatic choice uses 11 and 13 for K-contiguous operands only, 12 for the others)
    print("gemm bf16 forced configuration", variant, a_k, b_k, K, flush=True)
    assert _run(1, a_k, b_k, 0, 300, 264, K, 3, True, pad=8, tile=variant) < 2e-6


def test_gemm_rejects_misaligned_rows():
    import torch
    from paper_2110_11199_amd import binding as Bd
    t = torch.zeros(64 * 66, device="cuda:0")
    with pytest.raises(Bd.AdpsgdError) as ei:
        Bd.adpsgd_gemm(0, 1, 1, 0, 8, 8, 8, t.data_ptr(), 10, 0, t.data_ptr(), 8, 0, t.data_ptr(), 8, 0, None, 0, 1, None)
    assert ei.value.code == Bd.EINVAL
    for bad_tile, groups in ((7, 1), (-1, 0), (-1, 129)):     # unknown tile configuration, group counts out of range
        with pytest.raises(Bd.AdpsgdError) as ei:
            Bd.adpsgd_gemm(0, 1, 1, 0, 8, 8, 8, t.data_ptr(), 8, 0, t.data_ptr(), 8, 0, t.data_ptr(), 8, 0, None, 0, groups, None,
                           tile_config=bad_tile)
        assert ei.value.code == Bd.EINVAL


@pytest.mark.parametrize("prec,tile", [(0, 14), (0, 15), (1, 11), (1, 12), (1, 13), (1, 14), (1, 15)])
@pytest.mark.parametrize("a_k,b_k", LAYOUTS)
@pytest.mark.parametrize("M,N,K", [(64, 128, 8), (68, 60, 72), (300, 264, 200), (132, 520, 333), (129, 65, 61), (72, 72, 1)])
def test_gemm_k_past_the_last_whole_stage(prec, tile, a_k, b_k, M, N, K):
    # the part of K past the last 32- or 64-element stage (alone, after one stage, after several), one element to a
    # whole stage less one; K-contiguous operands need whole 16-byte chunks of K, the others take any K
    epc = 8 if prec else 4
    if a_k or b_k:
        K = (K + epc - 1) // epc * epc
    print("gemm K tail", prec, tile, a_k, b_k, M, N, K, flush=True)
    lda_pad = 8 if K % 8 == 0 else 4
    assert _run(prec, a_k, b_k, 0, M, N, K, 3, True, pad=lda_pad, tile=tile) < 2e-6
    assert _run(prec, a_k, b_k, 1, M, N, K, 2, False, tile=tile) < (6e-3 if prec else 2e-6)


@pytest.mark.parametrize("tile,edge", [(14, 128), (15, 64)])
@pytest.mark.parametrize("a_k,b_k", LAYOUTS)
@pytest.mark.parametrize("K", [196, 224, 240, 256, 257])
def test_gemm_fp32_on_the_bf16_matrix_units(tile, edge, a_k, b_k, K):
    # past the sizes that stay on fp32 MFMAs: one tile more than a whole number in rows and less in columns; an odd and an even
    # number of 16- and 32-element stages, whole ones and a last one of 1 and 4 elements.  Sums of K products rounded
    # once each: sqrt(K) 2^-24 of the result's scale, 1e-6
    K = K if not (a_k or b_k) else (K + 3) // 4 * 4
    print("gemm fp32 split", tile, a_k, b_k, K, flush=True)
    assert _run(0, a_k, b_k, 0, 2 * edge + 1, edge - 3, K, 3, True, pad=4, tile=tile) < 1e-6
    assert _run(0, a_k, b_k, 1, edge - 4, 3 * edge, K, 2, False, tile=tile) < 1e-6


@pytest.mark.parametrize("a_k,b_k", LAYOUTS)
@pytest.mark.parametrize("K", [20, 77, 80, 81, 112, 113])
def test_gemm_fp32_of_short_contractions(a_k, b_k, K):
    # several rounds of 64x64 tiles, the last of a row and a column ragged; rows of C that are whole 64 bytes and rows that are not.  A sum of K products
    # with K roundings of at most 2^-24 of a partial sum: as in test_gemm_fp32_of_long_contractions
    K = K if not (a_k or b_k) else (K + 3) // 4 * 4
    bound = 4 * max(K / 3, 4) ** 0.5 * 2.0 ** -24
    print("gemm fp32 short", a_k, b_k, K, flush=True)
    assert _run(0, a_k, b_k, 0, 1092, 1040, K, 2, True) < bound
    assert _run(0, a_k, b_k, 1, 1028, 1092, K, 2, False, pad=4) < bound


@pytest.mark.parametrize("tile,edge", [(14, 128), (15, 64)])
@pytest.mark.parametrize("a_k,b_k", LAYOUTS)
@pytest.mark.parametrize("K", [2560, 2564, 2577, 4096])
def test_gemm_fp32_of_long_contractions(tile, edge, a_k, b_k, K):
    # the last that runs on the bf16 matrix units and the first on fp32 MFMAs, an odd one, a whole number of stages.  K additions, each rounded by up to
    # 2^-24 of a partial sum, none of them (statistically) above the largest result: four standard deviations of K such errors, evenly spread,
    # relative to that result (2.4e-6 of 7.0e-6 measured at K = 2564)
    K = K if not (a_k or b_k) else (K + 3) // 4 * 4
    bound = 4 * (K / 3) ** 0.5 * 2.0 ** -24
    print("gemm fp32 long", tile, a_k, b_k, K, flush=True)
    assert _run(0, a_k, b_k, 0, 2 * edge + 1, edge - 3, K, 2, True, pad=4, tile=tile) < bound
    assert _run(0, a_k, b_k, 1, edge, 2 * edge, K, 2, False, tile=tile) < bound


@pytest.mark.parametrize("tile", [14, 15])
@pytest.mark.parametrize("a_k,b_k", LAYOUTS)
def test_gemm_fp32_of_values_that_have_no_finite_bf16_part(tile, a_k, b_k):
    # an infinity, a NaN and the largest fp32 value among ordinary ones: what the fp32 sums give, in their rows and nowhere else
    import torch
    from paper_2110_11199_amd import binding as Bd
    print("gemm fp32 non-finite", tile, a_k, b_k, flush=True)
    M, N, K = 260, 136, 256
    r = np.random.default_rng(3)
    A, B = r.standard_normal((M, K)).astype(np.float32), r.standard_normal((N, K)).astype(np.float32)
    B[:, :16] = 0.5                                        # (its second and third parts are 0)
    B[:, 5] = 0.0
    A[3, 4], A[140, 7], A[259, 9], A[200, 5] = np.inf, -np.inf, np.nan, np.float32(3.4028235e38)
    A[201, 6] = np.float32(3.4e38)
    dA = torch.from_numpy(np.ascontiguousarray(A if a_k else A.T)).cuda()
    dB = torch.from_numpy(np.ascontiguousarray(B if b_k else B.T)).cuda()
    dC = torch.empty(M, N, device="cuda")
    Bd.adpsgd_gemm(0, a_k, b_k, 0, M, N, K, dA.data_ptr(), K if a_k else M, 0, dB.data_ptr(), K if b_k else N, 0, dC.data_ptr(), N, 0,
                   None, 0, 1, torch.cuda.current_stream().cuda_stream, tile_config=tile)
    got = dC.cpu().numpy()
    assert (got[3] == np.inf).all() and (got[140] == -np.inf).all() and np.isnan(got[259]).all()
    ref = A.astype(np.float64) @ B.astype(np.float64).T
    rest = np.isfinite(ref).all(axis=1)
    assert rest.sum() == M - 3 and np.isfinite(got[rest]).all()
    assert (np.abs(got[rest] - ref[rest]) <= 2e-6 * np.abs(ref[rest]).max(axis=1, keepdims=True)).all()


@pytest.mark.parametrize("tile", [14, 15])
@pytest.mark.parametrize("a_k,b_k", LAYOUTS)
@pytest.mark.parametrize("scale_a,scale_b", [(-108, 0), (0, -108), (-108, 60), (-55, -55), (85, -85), (85, 30)])
def test_gemm_fp32_of_small_and_large_values(tile, a_k, b_k, scale_a, scale_b):
    # operands times powers of two, down to the values whose three bf16 parts still hold all 24 bits (2^-110; the largest of the distribution lie a little
    # above the scale, and those below it are a small share of a sum) and up to those whose check overflows: the same error as without
    import torch
    from paper_2110_11199_amd import binding as Bd
    print("gemm fp32 scaled", tile, a_k, b_k, scale_a, scale_b, flush=True)
    M, N, K = 136, 132, 256
    r = np.random.default_rng(5)
    A = (r.standard_normal((M, K)) * 2.0 ** scale_a).astype(np.float32)
    B = (r.standard_normal((N, K)) * 2.0 ** scale_b).astype(np.float32)
    dA = torch.from_numpy(np.ascontiguousarray(A if a_k else A.T)).cuda()
    dB = torch.from_numpy(np.ascontiguousarray(B if b_k else B.T)).cuda()
    dC = torch.empty(M, N, device="cuda")
    Bd.adpsgd_gemm(0, a_k, b_k, 0, M, N, K, dA.data_ptr(), K if a_k else M, 0, dB.data_ptr(), K if b_k else N, 0, dC.data_ptr(), N, 0,
                   None, 0, 1, torch.cuda.current_stream().cuda_stream, tile_config=tile)
    ref = A.astype(np.float64) @ B.astype(np.float64).T
    # (as test_gemm_fp32_of_long_contractions: four standard deviations of K roundings of 2^-24)
    assert np.abs(dC.cpu().numpy() - ref).max() < 4 * (K / 3) ** 0.5 * 2.0 ** -24 * np.abs(ref).max()
