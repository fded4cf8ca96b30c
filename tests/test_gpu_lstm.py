"""GPU: LSTM gradient and full ADPSGD iterations against the CPU oracle.

Tolerances (per tensor, max|diff| / max|ref|): 1e-4 with fp32 GEMM operands,
2e-2 with bf16 GEMM operands; the schedule is compared exactly."""
import numpy as np
import pytest

from oracle import lstm, schedule as S, adpsgd as A
from oracle.lstm import Shape
from paper_2110_11199_amd import synth
from tests.gpu_util import rel_err

pytestmark = pytest.mark.gpu

TOL = {0: 1e-4, 1: 2e-2}
# bf16 mode against the oracle run with its GEMM operands rounded to bf16 as well: what is
# left is summation order and values that land on
# the other side of a bf16 rounding boundary (one bf16 ulp = 2^-8 relative).
TOL_EMULATED = 1e-2


def _engine(shape, L, pattern, prec, seed=0, **kw):
    from paper_2110_11199_amd import binding as Bd
    cfg = Bd.make_config(L, pattern, seed=seed, input_dim=shape.input_dim, hidden=shape.hidden,
                         layers=shape.layers, bidirectional=shape.bidirectional, bottleneck=shape.bottleneck,
                         classes=shape.classes, batch=shape.batch, frames=shape.frames, precision=prec, **kw)
    return Bd.Adpsgd(cfg)


def _batches(shape, L, k, seed=0):
    return [(synth.features(seed, k, i, shape.frames, shape.batch, shape.input_dim),
             synth.labels(seed, k, i, shape.frames, shape.batch, shape.classes)) for i in range(L)]


def _to_dev(batches):
    import torch
    return [(torch.from_numpy(f).cuda(), torch.from_numpy(y).cuda()) for f, y in batches]


def _per_tensor_err(shape, got, ref):
    worst = 0.0
    for name, off, r, c in lstm.layout(shape)[0]:
        worst = max(worst, rel_err(got[off:off + r * c], ref[off:off + r * c]))
    return worst


SHAPES = [
    Shape(40, 64, 1, 0, 0, 100, 4, 20),       # the tiny benchmark shape
    Shape(12, 32, 2, 1, 0, 52, 5, 7),         # bidirectional, ragged batch
    Shape(24, 36, 2, 1, 16, 40, 33, 3),       # bottleneck, hidden not a multiple of 8/32, batch 33
    Shape(20, 64, 1, 1, 0, 300, 70, 4),       # batch 70 (64-row tiles + tail), several class tiles
    Shape(16, 32, 3, 0, 8, 36, 130, 2),       # batch 130 (128-row tiles + tail), unidirectional
    Shape(8, 8, 1, 1, 4, 8, 9, 1),            # one frame: no recurrence (9 rows: with 2 the bf16 rounding of a single
                                              # operand shows up as 2.2e-2 in a bias gradient, in the oracle's own bf16 run too)
    Shape(24, 192, 2, 1, 16, 64, 130, 3),     # hidden 192: ragged unit tiles of the direct-to-LDS kernels, batch 130
    Shape(16, 128, 1, 1, 0, 40, 48, 4),       # batch 48: the 64-row recurrent tile configuration
    Shape(8, 32, 1, 0, 0, 1500, 3, 2),        # 1500 classes: softmax rows of 4 float4 per thread
    Shape(8, 32, 1, 0, 0, 5000, 3, 2),        # 5000 classes: softmax rows on 512 threads
    Shape(16, 72, 2, 1, 0, 32, 20, 5),        # small-batch recurrent kernels: three unit tiles, the last one ragged
    Shape(12, 20, 1, 1, 0, 24, 32, 3),        # batch 32, hidden 20: half-empty last k-chunk (fp32); staged kernels (bf16)
    Shape(12, 264, 1, 1, 0, 20, 7, 4),        # hidden 264: more k-chunks than one pass of a workgroup's waves takes
]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("shape", SHAPES)
def test_gradient_matches_oracle(shape, prec):
    _check_gradient(shape, 2, prec)


# Enough learners for the direct-to-LDS step kernels (more split-contraction workgroups than the chip takes at once), at
# hidden sizes that are no multiple of their K stage: below one stage, one stage and a remainder, several.
DIRECT_SHAPES = [
    (Shape(8, 40, 1, 1, 0, 12, 130, 3), 26),      # 130 rows: five 32-row backward tiles, two 128-row forward tiles
    (Shape(8, 72, 1, 1, 0, 12, 70, 3), 30),       # 70 rows: 32-row backward tiles, ragged
    (Shape(8, 40, 1, 1, 0, 12, 70, 3), 97),       # the 128-row backward tile, partly filled
    (Shape(8, 136, 1, 0, 0, 12, 40, 3), 55),      # one direction, batch 40: the 64-row forward tile
    (Shape(8, 104, 1, 1, 0, 12, 20, 2), 66),      # a batch below 32 rows with many learners
]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("shape,L", DIRECT_SHAPES)
def test_gradient_on_the_direct_step_kernels(shape, L, prec):
    from paper_2110_11199_amd import binding as Bd
    _check_gradient(shape, L, prec, tune=[(Bd.TUNE_REC_PERSISTENT, 0)])


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[1], SHAPES[4], SHAPES[7], SHAPES[10], SHAPES[11]])
def test_gradient_frame_by_frame(shape, prec):
    # hidden sizes up to 128 run all frames in one launch unless told otherwise: here the kernels that take one frame each
    from paper_2110_11199_amd import binding as Bd
    _check_gradient(shape, 2, prec, tune=[(Bd.TUNE_REC_PERSISTENT, 0)])


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("classes", [4, 28, 32, 36, 60, 64, 68, 132])
def test_gradient_with_padded_rows_of_logits(classes, prec):
    # rows of logits are 32 elements apart and multiples of it, those of their gradient 64 (bf16): one column less, none, one more
    _check_gradient(Shape(8, 16, 1, 0, 0, classes, 9, 3), 2, prec)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("classes", [4, 16, 20, 128, 132, 256, 260, 512])
@pytest.mark.parametrize("hidden,batch,frames", [(8, 9, 1), (24, 5, 3), (16, 16, 2), (32, 11, 3)])
def test_gradient_with_the_output_layer_and_softmax_in_one_launch(hidden, batch, frames, classes, prec):
    # class tiles of 16 over the waves: one, a part of one, whole rounds, one more; 9, 15, 32 and 33 frames of blocks of 16; a contraction of part of a
    # chunk, of one and a part, of more than are in flight
    _check_gradient(Shape(8, hidden, 1, 1, 0, classes, batch, frames), 3, prec)


def _softmax_launches(shape, L, prec, tune=()):
    import torch
    from paper_2110_11199_amd import binding as Bd
    eng = _engine(shape, L, S.FIXED_RING, prec)
    for key, value in tune:
        eng.tune(key, value)
    eng.set_params(-1, torch.from_numpy(synth.initial_model(1, eng.P, 0.2)).cuda())
    b = _to_dev(_batches(shape, L, 0))
    eng.step(b, 0.0)
    Bd.adpsgd_set_profiling(eng.h, 1)
    eng.step(b, 0.0)
    launches = Bd.adpsgd_profile(eng.h)["softmax_ce"]["launches"]
    eng.close()
    return launches


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("tile,classes", [(15, 4), (15, 8), (15, 12), (0, 16), (15, 20), (0, 28), (15, 32), (15, 36), (0, 60), (15, 64), (14, 68), (14, 132), (-1, 516), (-1, 540), (-1, 544), (-1, 548)])
def test_gradient_with_logits_in_memory(tile, classes, prec):
    # The output layer's product stores the logits and the softmax reads them (a tile configuration that the caller sets means two launches; from 516
    # classes x 72 on W_o is past one launch by itself).  Their rows are 4, 8, 16 or 32 elements and multiples of 32 apart, those of their gradient up to 64 (bf16): a few
    # columns less, none, four more.
    from paper_2110_11199_amd import binding as Bd
    shape, tune = Shape(8, 16 if tile >= 0 else 72, 1, 0, 0, classes, 9, 3), [(Bd.TUNE_GEMM_TILE, tile)]
    assert _softmax_launches(shape, 2, prec, tune) == 1
    _check_gradient(shape, 2, prec, tune=tune)


@pytest.mark.parametrize("prec,width,classes", [(1, 88, 128), (1, 104, 260), (1, 120, 256), (1, 88, 340), (1, 96, 340), (1, 768, 40), (1, 392, 20),
                                                (0, 64, 128), (0, 72, 132), (0, 44, 260), (0, 52, 312), (0, 188, 20)])
def test_gradient_with_the_output_layer_and_softmax_in_one_launch_over_more_chunks_than_are_in_flight(prec, width, classes):
    # each number of waves and of class tiles to a wave, a contraction of three chunks and more (32 of k in bf16, 16 in fp32; two are in flight), some ending in part of
    # one; fp32 up to 192 in one round of tiles
    shape = Shape(8, 16, 1, 0, width, classes, 11, 3)
    assert _softmax_launches(shape, 2, prec) == 0
    _check_gradient(shape, 2, prec)


@pytest.mark.parametrize("hidden", [64, 100])
@pytest.mark.parametrize("frames", [2, 3, 4, 6, 7, 8, 9])
def test_gradient_with_inputs_requested_some_frames_ahead(hidden, frames):
    # backward in fp32 on one compute unit: fewer frames than are requested ahead, whole rounds of the four sets of inputs, one to three more
    _check_gradient(Shape(8, hidden, 1, 1, 0, 8, 6, frames), 2, 0)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("hidden", [16, 48, 100, 128])
@pytest.mark.parametrize("batch,frames", [(1, 2), (16, 5), (17, 1)])
def test_gradient_with_all_frames_on_one_compute_unit(hidden, batch, frames, prec):
    # one wave to eight, each register size; one row, a whole tile and one row more; an even, an odd and a single frame (which
    # runs as a launch of its own where the rows of W_h are aligned)
    _check_gradient(Shape(12, hidden, 2, 1, 0, 24, batch, frames), 2, prec)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("hidden", [16, 72, 128])
def test_gradient_with_all_frames_on_one_compute_unit_sixteen_rows_at_a_time(hidden, prec):
    # more blocks of four rows than three per compute unit: the kernels that take 16, the last block ragged
    _check_gradient(Shape(12, hidden, 1, 1, 0, 8, 77, 3), 20, prec)


@pytest.mark.parametrize("prec,hidden", [(0, 132), (0, 256), (0, 260), (0, 384), (0, 512), (1, 132), (1, 136), (1, 256), (1, 300), (1, 360), (1, 508), (1, 512), (1, 640)])
@pytest.mark.parametrize("batch,frames", [(1, 2), (17, 5), (32, 3)])
def test_gradient_with_all_frames_on_clusters_of_compute_units(prec, hidden, batch, frames):
    # every cluster size, whole and with units past the hidden size; one row, one row more than a block, whole blocks (2 and 3
    # frames are too few for some sizes: the next test has numbers that both passes of all of them run on clusters for)
    _check_gradient(Shape(12, hidden, 2, 1, 0, 24, batch, frames), 2, prec)


@pytest.mark.parametrize("prec,hidden", [(0, 132), (0, 260), (0, 384), (0, 512), (1, 136), (1, 360), (1, 508), (1, 512), (1, 640)])
@pytest.mark.parametrize("batch,frames", [(1, 7), (17, 8), (32, 7)])
def test_gradient_on_clusters_of_compute_units_from_few_frames_on(prec, hidden, batch, frames):
    # every cluster size, both passes; one row, one row more than a block, whole blocks
    _check_gradient(Shape(12, hidden, 1, 1, 0, 24, batch, frames), 2, prec)


# Numbers of clusters that would take a round of the chip more on one XCD each, so that their members lie on several and exchange through memory:
# 18 and 36 of 12 members (21 fit the 256 compute units anywhere, 16 on one XCD each), 42 and 84 of 6 (42, 40), 25 and 50 of 10 (25, 24).
ACROSS_XCDS = [
    (0, Shape(12, 348, 1, 1, 0, 24, 48, 7), 3, 12), (0, Shape(12, 384, 1, 1, 0, 24, 40, 7), 6, 12),
    (0, Shape(12, 320, 1, 0, 0, 24, 65, 7), 5, 10), (0, Shape(12, 260, 1, 1, 0, 24, 80, 7), 5, 10),
    (1, Shape(12, 360, 1, 1, 0, 24, 48, 7), 7, 6), (1, Shape(12, 264, 1, 1, 0, 24, 48, 7), 14, 6),
    (1, Shape(12, 640, 1, 0, 0, 24, 80, 7), 5, 10), (1, Shape(12, 516, 1, 1, 0, 24, 80, 7), 5, 10),
]


@pytest.mark.parametrize("prec,shape,L,members", ACROSS_XCDS)
def test_gradient_on_clusters_that_exchange_through_memory(prec, shape, L, members):
    from paper_2110_11199_amd import binding as Bd
    _check_gradient(shape, L, prec)
    for a, b in zip(_one_step(shape, L, prec, ()), _one_step(shape, L, prec, ((Bd.TUNE_REC_JOIN_US, 0),))):
        assert (a == b).all()


@pytest.mark.parametrize("shape,L", [(Shape(12, 360, 1, 1, 0, 24, 48, 21), 7), (Shape(12, 640, 1, 0, 0, 24, 80, 21), 5)])
def test_backward_on_clusters_that_exchange_through_memory_keeps_up_with_forward(shape, L):
    # Both passes exchange H words a row and member and multiply as much.  Partial sums in whole lines: backward 1.67 and 1.89 times as long as forward; in half
    # lines 2.55 and 3.0.
    import torch
    from paper_2110_11199_amd import binding as Bd
    print("backward against forward through memory", shape, L, flush=True)
    eng = _engine(shape, L, S.FIXED_RING, 1)
    eng.set_params(-1, torch.from_numpy(synth.initial_model(1, eng.P, 0.1)).cuda())
    b = _to_dev(_batches(shape, L, 0))
    ratios = []
    for _ in range(5):
        eng.step(b, 0.0)
        Bd.adpsgd_set_profiling(eng.h, 1)
        for _ in range(10):
            eng.step(b, 0.0)
        prof = Bd.adpsgd_profile(eng.h)
        Bd.adpsgd_set_profiling(eng.h, 0)
        assert prof["recurrent_fwd"]["launches"] == 10 and prof["recurrent_bwd"]["launches"] == 10
        ratios.append(prof["recurrent_bwd"]["ms"] / prof["recurrent_fwd"]["ms"])
    eng.close()
    assert sorted(ratios)[2] < 2.2, ratios


@pytest.mark.parametrize("shape,L", [
    (Shape(12, 20, 1, 0, 132, 4104, 193, 8), 16),  # 272 tiles of 256x256 of dW_o, two rounds with a third empty, beside 208 blocks of rows of dz: launches of their own
    (Shape(12, 20, 1, 0, 132, 8200, 193, 8), 8),   # 264 tiles and 104 blocks: dW_o in 128x256 tiles in the launch of dz
    (Shape(12, 20, 1, 1, 0, 1000, 5, 3), 2),       # more workgroups of column sums than of products
])
def test_gradient_of_output_layers_that_share_a_launch(shape, L):
    _check_gradient(shape, L, 1)


@pytest.mark.parametrize("shape", [
    Shape(12, 20, 2, 1, 0, 24, 330, 9),            # 2970 frames, 2640 with a predecessor: both weight gradients long, in one launch
    Shape(12, 20, 2, 1, 0, 24, 440, 6),            # 2640 and 2200: one long
    Shape(12, 20, 1, 1, 8, 2564, 5, 3),            # the gradient of a bottleneck over 2564 states
])
def test_gradient_with_long_fp32_contractions(shape):
    _check_gradient(shape, 2, 0)


def _check_gradient(shape, L, prec, tune=()):
    import torch
    print("lstm grad", shape, L, prec, flush=True)
    P = lstm.param_count(shape)
    w0 = synth.initial_model(1, P, 0.2)
    eng = _engine(shape, L, S.FIXED_RING, prec)
    assert eng.P == P
    from paper_2110_11199_amd import binding as Bd
    assert [(o, r, c) for _, o, r, c in lstm.layout(shape)[0]] == Bd.adpsgd_layout(eng.h)
    for key, value in tune:
        eng.tune(key, value)
    eng.set_params(-1, torch.from_numpy(w0).cuda())
    b = _batches(shape, L, 0)
    eng.step(_to_dev(b), 0.0)
    losses = eng.losses()
    for i in range(L):
        loss, g = lstm.loss_and_grad(shape, w0, b[i][0], b[i][1], np.float32)
        got = eng.grads(i).cpu().numpy()
        assert np.isfinite(got).all()
        assert _per_tensor_err(shape, got, g) < TOL[prec], (i, _per_tensor_err(shape, got, g))
        assert abs(losses[i] - loss) < TOL[prec] * abs(loss)
        if prec:
            _, ge = lstm.loss_and_grad(shape, w0, b[i][0], b[i][1], np.float32, bf16_gemm=True)
            assert _per_tensor_err(shape, got, ge) < TOL_EMULATED, (i, _per_tensor_err(shape, got, ge))
    eng.close()


def _run_recurrence(shape, L, pattern, prec, steps, lr, seed=0, scale=0.1, tune=(), drop_straggler_batches=False, **kw):
    import torch
    P = lstm.param_count(shape)
    w0 = synth.initial_model(seed, P, scale)
    eng = _engine(shape, L, pattern, prec, seed=seed, **kw)
    for key, value in tune:
        eng.tune(key, value)
    eng.set_params(-1, torch.from_numpy(w0).cuda())
    ora = A.Oracle(L, pattern, seed, shape=shape, w0=w0, straggler_p=kw.get("straggler_p", 0.0), mix=kw.get("mix"),
                   group_size=max(kw.get("group_size", 1), 1))
    emu = A.Oracle(L, pattern, seed, shape=shape, w0=w0, bf16_gemm=True, mix=kw.get("mix"),
                   straggler_p=kw.get("straggler_p", 0.0), group_size=max(kw.get("group_size", 1), 1)) if prec else None
    for k in range(steps):
        b = _batches(shape, L, k, seed)
        db = _to_dev(b)
        if drop_straggler_batches:      # a straggler's minibatch is not read: hand over no pointers for it
            act_k = S.schedule(pattern, seed, k, L, kw.get("straggler_p", 0.0))[2]
            db = [db[i] if act_k[i] else (None, None) for i in range(L)]
        eng.step(db, lr)
        ora.step(b, lr)
        G = L // kw["group_size"] if kw.get("group_size") else L
        assert tuple(v[:G] for v in eng.schedule(k)) == tuple(ora.last_schedule)
        active = ora.last_schedule[2] if G == L else [1] * L
        np.testing.assert_allclose(eng.losses(), ora.last_losses, rtol=TOL[prec])      # a straggler reports 0 on both sides
        for i in range(L):
            got_x = eng.params(i).cpu().numpy()
            if active[i]:
                got_g = eng.grads(i).cpu().numpy()
                assert _per_tensor_err(shape, got_g, ora.last_grads[i]) < TOL[prec], (k, i)
            assert _per_tensor_err(shape, got_x, ora.x[i]) < TOL[prec], (k, i)
        if emu is not None:
            emu.step(b, lr)
            for i in range(L):
                if active[i]:
                    assert _per_tensor_err(shape, eng.grads(i).cpu().numpy(), emu.last_grads[i]) < TOL_EMULATED, (k, i)
    eng.close()
    return ora


def test_tiny_config_five_steps_fixed_ring():
    print("cfg1 recurrence", flush=True)
    wl = synth.WORKLOADS["cfg1"]
    shape = Shape(wl.input_dim, wl.hidden, wl.layers, wl.bidirectional, wl.bottleneck, wl.classes, wl.batch, wl.frames)
    _run_recurrence(shape, wl.L, wl.pattern, 0, wl.steps, wl.lr, scale=wl.init_scale)


def test_random_ring_with_stragglers_small_model():
    print("random ring + stragglers", flush=True)
    _run_recurrence(Shape(12, 16, 1, 1, 0, 20, 3, 4), 6, S.RANDOM_RING, 0, 5, 0.2, seed=4, straggler_p=0.3)
    _run_recurrence(Shape(12, 16, 1, 1, 0, 20, 3, 4), 6, S.RANDOM_RING, 0, 5, 0.2, seed=4, straggler_p=0.3,
                    drop_straggler_batches=True)


@pytest.mark.parametrize("prec", [0, 1])
def test_random_ring_with_stragglers_at_a_real_size(prec):
    # stragglers on a model whose GEMMs run on the large-tile and direct-to-LDS kernels (hidden 256, batch 96,
    # 8 learners): the gradient phase runs on the compacted list of active learners
    print("random ring + stragglers, hidden 256", prec, flush=True)
    seed = 9
    assert any(0 < sum(S.schedule(S.RANDOM_RING, seed, k, 8, 0.3)[2]) < 8 for k in range(3))
    _run_recurrence(Shape(64, 256, 2, 1, 64, 512, 96, 5), 8, S.RANDOM_RING, prec, 3, 0.2, seed=seed, scale=0.05,
                    straggler_p=0.3, drop_straggler_batches=True)


def test_every_learner_a_straggler_leaves_everything_unchanged():
    import torch
    shape = Shape(12, 16, 1, 1, 0, 20, 3, 4)
    L, seed, p = 3, 0, 0.97
    ks = [k for k in range(40) if sum(S.schedule(S.FIXED_RING, seed, k, L, p)[2]) == 0]
    assert ks and ks[0] == 0, ks[:3]     # iteration 0 has no active learner with this seed
    eng = _engine(shape, L, S.FIXED_RING, 0, seed=seed, straggler_p=p)
    w0 = synth.initial_model(seed, eng.P, 0.1)
    eng.set_params(-1, torch.from_numpy(w0).cuda())
    eng.step([(None, None)] * L, 0.5)
    assert (eng.losses() == 0).all()
    for i in range(L):
        assert (eng.params(i).cpu().numpy().view(np.uint32) == w0.view(np.uint32)).all()
    eng.close()


def test_label_out_of_range_is_reported_not_repaired_silently():
    import torch
    from paper_2110_11199_amd import binding as Bd
    shape = Shape(12, 16, 1, 1, 0, 20, 3, 4)
    for bad in (-1, shape.classes, 1 << 30):
        eng = _engine(shape, 2, S.FIXED_RING, 0)
        eng.set_params(-1, torch.from_numpy(synth.initial_model(0, eng.P, 0.1)).cuda())
        b = _batches(shape, 2, 0)
        eng.step(_to_dev(b), 0.1)
        eng.status()                                   # clean so far
        b[1][1][2, 1] = bad
        eng.step(_to_dev(b), 0.1)
        with pytest.raises(Bd.AdpsgdError) as ei:
            eng.losses()
        assert ei.value.code == Bd.EINVAL and "label" in str(ei.value)
        with pytest.raises(Bd.AdpsgdError) as ei:      # sticky: the step after the flag has reached the host is refused
            eng.step(_to_dev(_batches(shape, 2, 1)), 0.1)
        assert ei.value.code == Bd.EINVAL
        with pytest.raises(Bd.AdpsgdError):
            eng.status()
        eng.close()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("classes", [20, 1500, 5000, 32772])
def test_label_out_of_range_is_reported_by_every_kind_of_softmax(classes, prec):
    # in one launch with the output layer, rows in registers of 256 and of 512 threads, and rows longer than those
    import torch
    from paper_2110_11199_amd import binding as Bd
    print("bad label", classes, prec, flush=True)
    shape = Shape(8, 32, 1, 0, 0, classes, 3, 2)
    assert _softmax_launches(shape, 2, prec) == (0 if classes == 20 else 1)
    for bad in (-1, classes, 1 << 30):
        eng = _engine(shape, 2, S.FIXED_RING, prec)
        eng.set_params(-1, torch.from_numpy(synth.initial_model(0, eng.P, 0.1)).cuda())
        b = _batches(shape, 2, 0)
        b[1][1].reshape(-1)[:] = classes - 1               # (the largest label is one)
        eng.step(_to_dev(b), 0.1)
        eng.status()
        b[1][1][1, 2] = bad
        eng.step(_to_dev(b), 0.1)
        with pytest.raises(Bd.AdpsgdError) as ei:
            eng.losses()
        assert ei.value.code == Bd.EINVAL and "label" in str(ei.value)
        eng.close()


@pytest.mark.parametrize("prec", [0, 1])
def test_delay_by_one_small_model(prec):
    print("d1d small", prec, flush=True)
    # weights U(-0.1, 0.1): with 12 frames per minibatch and weights of 0.3 the bf16 operand rounding
    # alone reaches 2.2e-2 on the smallest tensors
    ora = _run_recurrence(Shape(12, 16, 2, 1, 8, 20, 3, 4), 4, S.D1D, prec, 4, 0.3, seed=2, scale=0.1)
    assert ora.tau == 1


@pytest.mark.parametrize("prec", [0, 1])
def test_ring_neighbour_mixing_small_model(prec):
    print("ring neighbours (weights 1/3), model-bearing", prec, flush=True)
    ora = _run_recurrence(Shape(12, 16, 2, 1, 8, 20, 5, 4), 5, S.RANDOM_RING, prec, 4, 0.3, seed=5, scale=0.1, mix=S.MIX_TRI)
    assert ora.mix == S.MIX_TRI


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("mix", [S.MIX_HYBRID_PAIR, S.MIX_HYBRID_TRI])
def test_hybrid_super_learners_small_model(prec, mix):
    print("hybrid super-learners, model-bearing", prec, mix, flush=True)
    ora = _run_recurrence(Shape(12, 16, 2, 1, 8, 20, 5, 4), 6, S.RANDOM_RING, prec, 4, 0.3, seed=5, scale=0.1, mix=mix, group_size=2)
    assert ora.hybrid and ora.ring_size == 3


@pytest.mark.parametrize("prec", [0, 1])
def test_synchronous_baseline_small_model(prec):
    print("sdpsgd small, model-bearing", prec, flush=True)
    ora = _run_recurrence(Shape(12, 16, 2, 1, 8, 20, 5, 4), 4, S.SDPSGD, prec, 4, 0.3, seed=6, scale=0.1)
    assert ora.update_first and ora.consensus() == 0.0


@pytest.mark.parametrize("case", ["pair", "tri", "tri_d1d", "mean", "sync"])
def test_segmented_update_kernels_write_the_bf16_copy_of_a_small_model(case):
    # the update kernels that large models take by default (one member of a pair per thread; the ring or the learners in
    # segments), forced on a small bf16 model: the bf16 copy of the next gradient point they write feeds the next iteration
    from paper_2110_11199_amd import binding as Bd
    print("segmented update kernels, bf16 model", case, flush=True)
    shape = Shape(12, 32, 2, 1, 0, 52, 5, 7)
    if case == "pair":
        _run_recurrence(shape, 5, S.RANDOM_RING, 1, 3, 0.1, tune=((Bd.TUNE_PAIR_SPLIT, 64),), straggler_p=0.2)
    elif case == "tri":
        _run_recurrence(shape, 5, S.RANDOM_RING, 1, 3, 0.1, tune=((Bd.TUNE_TRI_SEGMENT, 2),), mix=S.MIX_TRI)
    elif case == "tri_d1d":
        _run_recurrence(shape, 5, S.D1D, 1, 3, 0.1, tune=((Bd.TUNE_TRI_SEGMENT, 2),), mix=S.MIX_TRI)
    elif case == "mean":
        _run_recurrence(shape, 5, S.D1D, 1, 3, 0.1, tune=((Bd.TUNE_SYNC_SEGMENT, 2),))
        _run_recurrence(shape, 5, S.FIXED_RING, 1, 3, 0.1, tune=((Bd.TUNE_SYNC_SEGMENT, 4),), mix=S.MIX_ALL)
    else:
        _run_recurrence(shape, 5, S.SDPSGD, 1, 3, 0.1, tune=((Bd.TUNE_SYNC_SEGMENT, 2),))


@pytest.mark.parametrize("groups", [2, 3, 5])
def test_forward_recurrence_in_learner_groups(groups):
    # large models run the forward recurrence group of learners by group of learners (all frames of a group
    # first); forced here on a small one, 5 learners in 2 + 3, 1 + 1 + 3 and 1 + 1 + 1 + 1 + 1
    from paper_2110_11199_amd import binding as Bd
    print("forward recurrence in learner groups", groups, flush=True)
    for prec in (0, 1):
        _run_recurrence(Shape(12, 64, 2, 1, 0, 20, 40, 3), 5, S.RANDOM_RING, prec, 2, 0.2, seed=7, scale=0.1,
                        tune=[(Bd.TUNE_REC_FWD_GROUPS, groups)])


@pytest.mark.parametrize("prec,hidden", [(0, 64), (1, 128), (0, 256), (1, 256)])
def test_learner_groups_are_taken_where_all_frames_would_run_in_one_launch(prec, hidden):
    import torch
    from paper_2110_11199_amd import binding as Bd
    shape = Shape(12, hidden, 2, 1, 0, 20, 8, 10)
    for groups in (0, 1, 3):
        e = _engine(shape, 5, S.FIXED_RING, prec)
        e.tune(Bd.TUNE_REC_FWD_GROUPS, groups)
        e.set_params(-1, torch.from_numpy(synth.initial_model(0, e.P, 0.1)).cuda())
        Bd.adpsgd_set_profiling(e.h, 1)
        e.step(_to_dev(_batches(shape, 5, 0)), 0.1)
        e.status()
        launches = Bd.adpsgd_profile(e.h)["recurrent_fwd"]["launches"]
        e.close()
        assert launches == shape.layers * (groups * shape.frames if groups else 1), (groups, launches)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[1], SHAPES[10]])
def test_small_batches_on_the_staged_kernels_too(shape, prec):
    # batches of at most 32 rows normally take the small-batch kernels; switched off, the register-staged
    # kernels with their 32-row tiles run the same recurrence
    from paper_2110_11199_amd import binding as Bd
    print("staged kernels, small batch", shape, prec, flush=True)
    _run_recurrence(shape, 2, S.FIXED_RING, prec, 2, 0.1, tune=((Bd.TUNE_REC_DIRECT, 0),))


def test_profile_counts_two_weight_gradients_in_one_launch_once():
    # input projection, output layer, its two gradient products and one launch for both weight gradients of the layer; with a
    # tile that cannot take two problems at once, two
    import torch
    from paper_2110_11199_amd import binding as Bd
    shape = Shape(40, 64, 1, 0, 0, 100, 4, 20)
    for tile, want in ((-1, 5), (0, 6)):
        e = _engine(shape, 4, S.FIXED_RING, 0)
        e.tune(Bd.TUNE_GEMM_TILE, tile)
        e.set_params(-1, torch.from_numpy(synth.initial_model(0, e.P, 0.1)).cuda())
        Bd.adpsgd_set_profiling(e.h, 1)
        e.step(_to_dev(_batches(shape, 4, 0)), 0.1)
        e.status()
        assert Bd.adpsgd_profile(e.h)["batched_gemm"]["launches"] == want
        e.close()


def test_tuning_is_per_handle():
    # two handles in one process: forcing the register-staged kernels on one must not change the other
    import torch
    from paper_2110_11199_amd import binding as Bd
    shape = Shape(64, 64, 1, 1, 0, 64, 40, 3)
    w0 = synth.initial_model(3, lstm.param_count(shape), 0.1)
    b = _batches(shape, 2, 0)
    out = []
    for forced in (False, True, False):
        a = _engine(shape, 2, S.FIXED_RING, 1)
        other = _engine(shape, 2, S.FIXED_RING, 1)
        if forced:
            other.tune(Bd.TUNE_REC_DIRECT, 0)
            other.tune(Bd.TUNE_GEMM_TILE, 0)
        for e in (a, other):
            e.set_params(-1, torch.from_numpy(w0).cuda())
            e.step(_to_dev(b), 0.1)
        out.append(a.grads(0).cpu().numpy().copy())
        a.close(); other.close()
    assert (out[0].view(np.uint32) == out[1].view(np.uint32)).all() and (out[0].view(np.uint32) == out[2].view(np.uint32)).all()
    with pytest.raises(Bd.AdpsgdError):
        e = _engine(shape, 2, S.FIXED_RING, 1)
        try:
            e.tune(Bd.TUNE_GEMM_TILE, 7)
        finally:
            e.close()


def test_library_initial_model_matches_generator_spec():
    import torch
    shape = Shape(8, 8, 1, 0, 0, 8, 2, 2)
    eng = _engine(shape, 3, S.FIXED_RING, 0, seed=77, init_scale=0.1)
    ref = A.init_model(77, eng.P, 0.1)
    for i in range(3):
        assert (eng.params(i).cpu().numpy() == ref).all()      # same w_0 on every learner
    eng.close()


PERSIST_SHAPES = [
    Shape(64, 128, 2, 1, 0, 64, 40, 5),       # hidden 128, batch 40: two row tiles, ragged
    Shape(64, 128, 1, 0, 0, 64, 128, 3),      # one direction, batch 128: four row tiles
    Shape(64, 256, 2, 1, 32, 96, 100, 4),     # hidden 256, batch 100: four row tiles, ragged; bottleneck
    Shape(32, 256, 1, 1, 0, 64, 64, 6),       # batch 64: two full row tiles
    Shape(32, 128, 1, 1, 0, 64, 9, 1),        # a single frame: no recurrent product at all
]


@pytest.mark.parametrize("shape", PERSIST_SHAPES)
def test_persistent_recurrent_kernels_match_oracle(shape):
    # all frames of a layer in one launch, W_h resident in registers, workgroups of a (learner, direction) pair
    # synchronised once per frame: forced on small shapes; 3 learners, stragglers in some iterations
    from paper_2110_11199_amd import binding as Bd
    print("persistent recurrent kernels", shape, flush=True)
    _run_recurrence(shape, 3, S.RANDOM_RING, 1, 3, 0.2, seed=11, scale=0.08, straggler_p=0.25,
                    tune=[(Bd.TUNE_REC_PERSISTENT, 1)])


def test_persistent_recurrent_kernels_in_several_launches():
    # hidden 256: 8 workgroups per (learner, direction) pair, 32 pairs per launch on 256 compute units;
    # 20 learners x 2 directions = 40 pairs run as 32 + 8
    from paper_2110_11199_amd import binding as Bd
    print("persistent recurrent kernels, 40 pairs", flush=True)
    _run_recurrence(Shape(32, 256, 1, 1, 0, 32, 33, 3), 20, S.D1D, 1, 2, 0.2, seed=12, scale=0.08,
                    tune=[(Bd.TUNE_REC_PERSISTENT, 1)])


def test_persistent_and_per_frame_kernels_agree_closely():
    # same arithmetic up to the summation order of the recurrent products: far inside the tolerance against the oracle
    import torch
    from paper_2110_11199_amd import binding as Bd
    shape = Shape(64, 256, 2, 1, 0, 64, 72, 5)
    w0 = synth.initial_model(3, lstm.param_count(shape), 0.08)
    b = _batches(shape, 2, 0)
    out = []
    for persistent in (0, 1):
        e = _engine(shape, 2, S.FIXED_RING, 1)
        e.tune(Bd.TUNE_REC_PERSISTENT, persistent)
        e.set_params(-1, torch.from_numpy(w0).cuda())
        e.step(_to_dev(b), 0.1)
        e.status()
        out.append(e.grads(0).cpu().numpy().copy())
        e.close()
    assert _per_tensor_err(shape, out[1], out[0]) < 4e-3


def test_persistent_kernel_wait_runs_out_and_is_reported():
    # a wait bound of 0 microseconds: the first workgroup that has to wait for its pair gives up, the others
    # follow, every workgroup returns; the handle reports the failure and refuses further steps
    import torch
    from paper_2110_11199_amd import binding as Bd
    shape = Shape(32, 128, 1, 1, 0, 32, 16, 4)
    e = _engine(shape, 2, S.FIXED_RING, 1)
    e.tune(Bd.TUNE_REC_PERSISTENT, 1)
    e.tune(Bd.TUNE_REC_WAIT_US, 0)
    e.set_params(-1, torch.from_numpy(synth.initial_model(0, e.P, 0.1)).cuda())
    e.step(_to_dev(_batches(shape, 2, 0)), 0.1)
    with pytest.raises(Bd.AdpsgdError) as ei:
        e.status()
    assert ei.value.code == Bd.EHIP and "wait" in str(ei.value)
    with pytest.raises(Bd.AdpsgdError) as ei:
        e.step(_to_dev(_batches(shape, 2, 1)), 0.1)
    assert ei.value.code == Bd.EHIP
    e.close()


def test_cluster_wait_runs_out_and_is_reported():
    # a wait bound of 0 microseconds gives up at the first exchange; every workgroup returns and the handle reports it
    import torch
    from paper_2110_11199_amd import binding as Bd
    shape = Shape(8, 256, 1, 1, 0, 8, 20, 4)
    e = _engine(shape, 2, S.FIXED_RING, 1)
    e.tune(Bd.TUNE_REC_WAIT_US, 0)
    e.set_params(-1, torch.from_numpy(synth.initial_model(0, e.P, 0.1)).cuda())
    e.step(_to_dev(_batches(shape, 2, 0)), 0.1)
    with pytest.raises(Bd.AdpsgdError) as ei:
        e.status()
    assert ei.value.code == Bd.EHIP and "wait" in str(ei.value)
    e.close()


def _one_step(shape, L, prec, tune):
    import torch
    e = _engine(shape, L, S.FIXED_RING, prec)
    for key, value in tune:
        e.tune(key, value)
    e.set_params(-1, torch.from_numpy(synth.initial_model(0, e.P, 0.1)).cuda())
    e.step(_to_dev(_batches(shape, L, 0)), 0.1)
    e.status()
    out = [t.cpu().numpy().view(np.uint32).copy() for i in range(L) for t in (e.grads(i), e.params(i))]
    e.close()
    return out


@pytest.mark.parametrize("prec,hidden", [(0, 132), (0, 260), (0, 384), (0, 512), (1, 136), (1, 300), (1, 360), (1, 512), (1, 640)])
def test_cluster_left_to_one_workgroup_gives_the_same_bits(prec, hidden):
    # every cluster size; two blocks of rows, the second of one row; a bound of 0 lets one workgroup do each cluster's work
    from paper_2110_11199_amd import binding as Bd
    print("clusters left to one workgroup", prec, hidden, flush=True)
    shape = Shape(12, hidden, 2, 1, 0, 24, 17, 8)
    for a, b in zip(_one_step(shape, 2, prec, ()), _one_step(shape, 2, prec, ((Bd.TUNE_REC_JOIN_US, 0),))):
        assert (a == b).all()


def test_cluster_waits_for_workgroups_that_have_not_started():
    # 64 clusters of 6 workgroups on 256 compute units: the cluster that is short of workgroups at first waits for one of the 40
    # before it (five to an XCD) to end (100 frames, some hundreds of microseconds).  That is no expiry of the bound on the exchange, nor
    # does it matter whether the cluster is left to one of its workgroups instead (bound of 20 microseconds)
    from paper_2110_11199_amd import binding as Bd
    print("cluster short of workgroups", flush=True)
    shape = Shape(12, 360, 1, 1, 0, 24, 64, 100)
    for a, b in zip(_one_step(shape, 8, 1, ((Bd.TUNE_REC_WAIT_US, 300),)), _one_step(shape, 8, 1, ((Bd.TUNE_REC_JOIN_US, 20),))):
        assert (a == b).all()


def test_batch_beyond_the_second_dimension_of_a_grid():
    # 1 100 000 segments are 68 750 blocks of 16 rows: more than a grid's second dimension holds, so every frame is a launch
    from paper_2110_11199_amd import binding as Bd
    print("batch of 1.1 million", flush=True)
    import torch
    T, B = 3, 1_100_000
    out = []
    for persistent in (-1, 0):
        e = _engine(Shape(4, 4, 1, 0, 0, 4, B, T), 1, S.FIXED_RING, 0)
        e.tune(Bd.TUNE_REC_PERSISTENT, persistent)
        e.set_params(-1, torch.from_numpy(synth.initial_model(0, e.P, 0.1)).cuda())
        x = torch.arange(T * B * 4, device="cuda", dtype=torch.float32).remainder_(7.0)
        e.step([(x, torch.zeros(T * B, dtype=torch.int32, device="cuda"))], 0.1)
        e.status()
        out.append(e.grads(0).cpu().numpy().view(np.uint32).copy())
        e.close()
    assert np.isfinite(out[0].view(np.float32)).all() and (out[0] == out[1]).all()


@pytest.mark.parametrize("hidden", [132, 256, 320])
def test_clusters_in_fp32_with_weights_that_no_bf16_parts_hold(hidden):
    # an infinite recurrent weight: the forward pass saturates a gate, and backward 0 x inf makes all gradients of the first direction NaN, frame by frame
    # as on clusters.  What is finite and compared - the output layer and the second direction - shows that forward pass and nothing of the backward
    # products of the first direction: those are compared with finite weights, below
    import torch
    from paper_2110_11199_amd import binding as Bd
    print("clusters, weights without finite parts", hidden, flush=True)
    shape = Shape(12, hidden, 1, 1, 0, 24, 5, 8)
    out = []
    for persistent in (-1, 0):
        e = _engine(shape, 2, S.FIXED_RING, 0)
        e.tune(Bd.TUNE_REC_PERSISTENT, persistent)
        w = synth.initial_model(0, e.P, 0.1)
        names = {n: (o, r, c) for n, o, r, c in lstm.layout(shape)[0]}
        o, rows, cols = [v for k, v in names.items() if v[1] == 8 * hidden and v[2] == hidden][0]
        wh = w[o:o + rows * cols].reshape(rows, cols)
        wh[3, :] = 0.0
        wh[3, 7] = np.inf                                  # the input gate of cell 3, first direction
        wh[hidden + 9, 11] = np.float32(3.4028235e38)      # the forget gate of cell 9
        e.set_params(-1, torch.from_numpy(w).cuda())
        e.step(_to_dev(_batches(shape, 2, 0)), 0.0)
        e.status()
        out.append(e.grads(0).cpu().numpy().copy())
        e.close()
    a, b = out
    assert (np.isnan(a) == np.isnan(b)).mean() > 0.999
    both = np.isfinite(a) & np.isfinite(b)
    assert both.sum() > 0 and np.abs(a[both] - b[both]).max() <= 1e-4 * np.abs(b[both]).max()


def _one_gradient(shape, L, w, batches, tune):
    import torch
    e = _engine(shape, L, S.FIXED_RING, 0)
    for key, value in tune:
        e.tune(key, value)
    e.set_params(-1, torch.from_numpy(w).cuda())
    e.step(_to_dev(batches), 0.0)
    e.status()
    out = [e.grads(i).cpu().numpy().copy() for i in range(L)]
    e.close()
    return out


def _tensor(shape, w, name):
    off, r, c = {n: (o, r, c) for n, o, r, c in lstm.layout(shape)[0]}[name]
    return w[off:off + r * c].reshape(r, c)


def _check_cluster_against_alone_and_frames(shape, L, w, batches):
    # a cluster, one workgroup for a cluster: the same bits; frame by frame: the same sums in another order (1e-5 of a tensor's largest value, as for
    # other sums of this length)
    from paper_2110_11199_amd import binding as Bd
    together = _one_gradient(shape, L, w, batches, ())
    alone = _one_gradient(shape, L, w, batches, ((Bd.TUNE_REC_JOIN_US, 0),))
    frames = _one_gradient(shape, L, w, batches, ((Bd.TUNE_REC_PERSISTENT, 0),))
    for a, b, f in zip(together, alone, frames):
        assert np.isfinite(f).all() and np.isfinite(a).all()
        assert _per_tensor_err(shape, a, f) < 1e-5, _per_tensor_err(shape, a, f)
        assert (a.view(np.uint32) == b.view(np.uint32)).all(), (a.view(np.uint32) != b.view(np.uint32)).sum()
    return frames


@pytest.mark.parametrize("hidden", [132, 256, 320])
def test_clusters_in_fp32_with_finite_weights_that_no_bf16_parts_hold(hidden):
    # the largest fp32 value, whose first bf16 part is infinite, in a gate of one unit in either direction: times any h it saturates the gate, so
    # that the da of the gate is 0 in every frame that hands one on, and all gradients are finite.  The unit's member multiplies in fp32, the others in parts
    print("clusters, finite weights without finite parts", hidden, flush=True)
    shape = Shape(12, hidden, 1, 1, 0, 24, 17, 8)
    w = synth.initial_model(0, lstm.param_count(shape), 0.1)
    wh = _tensor(shape, w, "Wh0")
    big = np.float32(3.4028235e38)
    wh[3, 7] = big                                         # input gate of cell 3, first direction: the first member
    wh[hidden + hidden - 2, hidden - 3] = -big             # forget gate of the last but one: the last member that has units
    wh[4 * hidden + 3 * hidden + 70, 1] = big              # output gate of cell 70, second direction
    grads = _check_cluster_against_alone_and_frames(shape, 2, w, _batches(shape, 2, 0))
    g = _tensor(shape, grads[0], "Wh0")
    assert (g[3] == 0).all() and (g[4 * hidden + 3 * hidden + 70] == 0).all()      # (the saturated gates)
    assert (np.abs(g).max(axis=1) > 0).sum() >= 8 * hidden - 3                     # (and no others)


@pytest.mark.parametrize("hidden", [132, 256, 320])
def test_clusters_in_fp32_with_gradients_that_become_ordinary_again(hidden):
    # a loss in the last frame only, whose gradient is so large (2^93) that the check of the parts overflows there, and halves from frame to
    # frame: the first frames multiply in fp32, later ones in parts
    print("clusters, large gradients", hidden, flush=True)
    frames, batch = 40, 17
    shape = Shape(12, hidden, 1, 0, 0, 8, batch, frames)
    w = synth.initial_model(0, lstm.param_count(shape), 0.02)
    wo, bo = _tensor(shape, w, "Wo"), _tensor(shape, w, "bo")
    wo *= np.float32(2.0 ** 108)                           # 0.02 x 2^108: about 2^102, divided by the 680 rows of the minibatch
    bo[:] = 0.0
    bo[0, 0] = 2.0 ** 120                                  # state 0 has all the probability, whatever h
    y = np.zeros((frames, batch), np.int32)
    y[-1] = 1
    b = [(f, y.reshape(l.shape)) for f, l in _batches(shape, 2, 0)]
    _check_cluster_against_alone_and_frames(shape, 2, w, b)
