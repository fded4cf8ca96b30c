"""CPU-only checks of the C ABI: the library loads, exports what the header
declares, validates configurations, and its host-side schedule (a second,
independent implementation) is bit-identical to the oracle's."""
import os
import re
import ctypes
import pytest

from oracle import schedule as S
from paper_2110_11199_amd import binding as Bd

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    hdr = open(os.path.join(ROOT, "include", "adpsgd.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    declared = set(re.findall(r"\b(adpsgd_[a-z_0-9]+)\s*\(", hdr))
    assert len(declared) >= 15
    lib = ctypes.CDLL(Bd.LIB_PATH)
    for name in sorted(declared):
        assert hasattr(lib, name), name
    assert declared == set(Bd.EXPORTS)


@pytest.mark.parametrize("pattern", [0, 1, 2])
@pytest.mark.parametrize("L", [1, 2, 3, 4, 7, 8, 16, 64, 128])
@pytest.mark.parametrize("p", [0.0, 0.1, 0.5])
def test_schedule_is_bit_identical_to_the_oracle(pattern, L, p):
    for seed in (0, 12345, 2**63 + 11, 2**64 - 1):
        for k in (0, 1, 2, 3, 49, 1000003):
            assert Bd.adpsgd_schedule_of(pattern, seed, p, L, k) == S.schedule(pattern, seed, k, L, p)


def test_schedule_matches_stored_vectors():
    with open(os.path.join(ROOT, "tests", "golden", "schedule_vectors.txt")) as fh:
        rows = [ln.split() for ln in fh if ln.strip() and not ln.startswith("#")]
    for row in rows:
        pattern, seed, k, L, p = int(row[0]), int(row[1]), int(row[2]), int(row[3]), float(row[4])
        o, pa, a = Bd.adpsgd_schedule_of(pattern, seed, p, L, k)
        assert list(map(int, row[5:])) == o + pa + a


def test_config_validation_and_workspace_size():
    ok = Bd.make_config(4, Bd.FIXED_RING, input_dim=40, hidden=64, layers=1, classes=100, batch=4, frames=20)
    n = Bd.adpsgd_workspace_bytes(ok)
    assert n > 4 * 33380 * 4 * 2 and n % 256 == 0
    flat = Bd.make_config(64, Bd.RANDOM_RING, flat_params=135_000_000, straggler_p=0.1)
    scratch = 16640 + 256               # 2049 doubles of the consensus-distance reduction, rounded to 256 bytes; the status word
    assert Bd.adpsgd_workspace_bytes(flat) == 64 * 135_000_000 * 4 + scratch
    d1d = Bd.make_config(64, Bd.D1D, flat_params=1000)
    mean = 1024 * 4                     # chunk buffer of the global-mean update: min(16M, P rounded up to 1024) floats
    assert Bd.adpsgd_workspace_bytes(d1d) == 2 * 64 * 1024 * 4 + scratch + mean     # two model buffers, padded stride
    bad = [Bd.make_config(0, 0, flat_params=8), Bd.make_config(129, 0, flat_params=8),
           Bd.make_config(4, 4, flat_params=8), Bd.make_config(4, Bd.D1D, flat_params=8, straggler_p=0.1),
           Bd.make_config(4, Bd.SDPSGD, flat_params=8, straggler_p=0.1), Bd.make_config(4, Bd.SDPSGD, flat_params=8, tau=1),
           Bd.make_config(4, Bd.SDPSGD, flat_params=8, mix=Bd.MIX_PAIR),
           Bd.make_config(4, 0, flat_params=8, tau=1, straggler_p=0.1),
           Bd.make_config(4, 0, input_dim=39, hidden=64, layers=1, classes=100, batch=4, frames=20),
           Bd.make_config(4, 0, input_dim=40, hidden=64, layers=0, classes=100, batch=4, frames=20),
           Bd.make_config(4, 0, flat_params=8, precision=2), Bd.make_config(4, 0, flat_params=8, mix=3),
           Bd.make_config(4, 1, flat_params=8, mix=Bd.MIX_TRI, straggler_p=0.1),
           Bd.make_config(1, 0, flat_params=8, mix=Bd.MIX_TRI), Bd.make_config(2, 1, flat_params=8, mix=Bd.MIX_TRI)]
    assert Bd.adpsgd_workspace_bytes(Bd.make_config(4, 0, flat_params=8, mix=Bd.MIX_TRI)) > 0     # ring neighbours, weights 1/3
    # the synchronous baseline: one model buffer, the all-learner mean by default
    assert Bd.adpsgd_workspace_bytes(Bd.make_config(64, Bd.SDPSGD, flat_params=1000)) == 64 * 1024 * 4 + scratch + mean
    assert Bd.adpsgd_workspace_bytes(Bd.make_config(4, Bd.SDPSGD, flat_params=8, mix=Bd.MIX_ALL, tau=0)) > 0
    for cfg in bad:
        with pytest.raises(Bd.AdpsgdError) as ei:
            Bd.adpsgd_workspace_bytes(cfg)
        assert ei.value.code == Bd.EINVAL and Bd.adpsgd_last_error()


def test_hybrid_mixing_configurations():
    ok = [Bd.make_config(8, Bd.FIXED_RING, flat_params=8, mix=Bd.MIX_HYBRID_PAIR, group_size=2),
          Bd.make_config(8, Bd.RANDOM_RING, flat_params=8, mix=Bd.MIX_HYBRID_PAIR, group_size=8),
          Bd.make_config(12, Bd.RANDOM_RING, flat_params=8, mix=Bd.MIX_HYBRID_TRI, group_size=4),
          Bd.make_config(12, Bd.FIXED_RING, flat_params=8, mix=Bd.MIX_HYBRID_TRI, group_size=12),
          Bd.make_config(12, Bd.FIXED_RING, flat_params=8, mix=Bd.MIX_HYBRID_TRI, group_size=1, tau=1)]
    for cfg in ok:
        assert Bd.adpsgd_workspace_bytes(cfg) > 0
    bad = [Bd.make_config(8, Bd.FIXED_RING, flat_params=8, mix=Bd.MIX_HYBRID_PAIR, group_size=3),      # 8 is not a multiple of 3
           Bd.make_config(8, Bd.FIXED_RING, flat_params=8, mix=Bd.MIX_HYBRID_PAIR, group_size=0),
           Bd.make_config(8, Bd.FIXED_RING, flat_params=8, mix=Bd.MIX_HYBRID_TRI, group_size=4),       # a ring of two super-learners
           Bd.make_config(8, Bd.D1D, flat_params=8, mix=Bd.MIX_HYBRID_PAIR, group_size=2),
           Bd.make_config(8, Bd.SDPSGD, flat_params=8, mix=Bd.MIX_HYBRID_PAIR, group_size=2),
           Bd.make_config(8, Bd.RANDOM_RING, flat_params=8, mix=Bd.MIX_HYBRID_PAIR, group_size=2, straggler_p=0.1),
           Bd.make_config(8, Bd.RANDOM_RING, flat_params=8, mix=Bd.MIX_PAIR, group_size=2),            # group_size without a hybrid mix
           Bd.make_config(8, Bd.RANDOM_RING, flat_params=8, mix=5, group_size=2)]
    for cfg in bad:
        with pytest.raises(Bd.AdpsgdError) as ei:
            Bd.adpsgd_workspace_bytes(cfg)
        assert ei.value.code == Bd.EINVAL and Bd.adpsgd_last_error()


def test_learning_rate_helper_matches_the_oracle_and_the_papers_figures():
    from oracle import lr as LR
    with open(os.path.join(ROOT, "tests", "golden", "lr_schedule_paper.txt")) as fh:
        rows = [ln.split() for ln in fh if ln.strip() and not ln.startswith("#")]
    for name, epoch, rate in rows:
        args = (0.1, 0.0, 0, 10) if name == "baseline" else (3.2, 0.32, 10, 10)
        got = Bd.adpsgd_lr_at_epoch(int(epoch), *args)
        assert abs(got - float(rate)) <= 1.2e-7 * float(rate), (name, epoch, got)
    import numpy as np
    for epoch in range(1, 21):
        for peak, start, warm, hold in ((0.1, 0.0, 0, 10), (3.2, 0.32, 10, 10), (1.5, 0.5, 3, 7), (0.7, 0.1, 1, 1)):
            # float arguments reach the library as float32: feed the oracle the same rounded values
            ref = LR.lr_at_epoch(epoch, float(np.float32(peak)), start=float(np.float32(start)), warmup_epochs=warm, hold_until=hold)
            assert Bd.adpsgd_lr_at_epoch(epoch, peak, start, warm, hold) == np.float32(ref)
    for bad in ((0, 0.1, 0.0, 0, 10), (1, 0.1, 0.0, -1, 10)):
        with pytest.raises(Bd.AdpsgdError):
            Bd.adpsgd_lr_at_epoch(*bad)


@pytest.mark.parametrize("precision,logits,dlogits", [(Bd.FP32, 4 * 4, 4 * 4), (Bd.BF16_GEMM, 4 * 4, 8 * 2)])
def test_rows_of_few_classes_are_no_whole_lines(precision, logits, dlogits):
    # bytes of a frame's logits and of their gradient: 4 classes against 64, whose rows are whole lines of 128 bytes
    shape = dict(input_dim=8, hidden=16, layers=1, batch=64, frames=1024, precision=precision)
    few, many = (Bd.adpsgd_workspace_bytes(Bd.make_config(3, Bd.FIXED_RING, classes=c, **shape)) for c in (4, 64))
    saved = 3 * 64 * 1024 * (64 * 4 + 64 * (2 if precision else 4) - logits - dlogits)
    assert saved <= many - few < saved + 3 * 64 * 32 * 16          # (and the models, 1020 parameters apart)


def test_create_rejects_a_missing_workspace():
    cfg = Bd.make_config(2, 0, flat_params=8)
    with pytest.raises(Bd.AdpsgdError) as ei:
        Bd.adpsgd_create(cfg, None, 0, None)
    assert ei.value.code == Bd.ENOMEM


def test_argument_checks_that_need_no_gpu():
    # every rejection below happens before any HIP call
    for call in (lambda: Bd.adpsgd_set_tuning(None, Bd.TUNE_GEMM_TILE, 12), lambda: Bd.adpsgd_status(None),
                 lambda: Bd.adpsgd_delay(10_000_001, None), lambda: Bd.adpsgd_step_masked(None, [None], 0.1, [1]),
                 lambda: Bd.adpsgd_probe_mfma(None, 1, 1, None), lambda: Bd.adpsgd_probe_stream(3, 1, 0, 0x10000, 64, 16, None),
                 lambda: Bd.adpsgd_probe_stream(2, 1, 0, 0x10000, 60, 16, None),
                 lambda: Bd.adpsgd_capture_begin(None), lambda: Bd.adpsgd_capture_end(None), lambda: Bd.adpsgd_graph_replay(None)):
        with pytest.raises(Bd.AdpsgdError) as ei:
            call()
        assert ei.value.code == Bd.EINVAL
    assert Bd.adpsgd_graph_steps(None) == -1
    Bd.adpsgd_graph_destroy(None)       # a no-op
    fake = 0x10000      # never dereferenced: the size checks come first
    for ptr, stride, L, P, out in ((None, 8, 2, 8, fake), (fake, 8, 2, 8, None), (fake, 8, 0, 8, fake), (fake, 8, 129, 8, fake),
                                   (fake, 4, 2, 8, fake), (fake, 8, 2, 0, fake), (fake, 8, 2, 8, fake + 4),
                                   (fake, 1 << 40, 128, (Bd.STATIC_MAX_ELEMENTS >> 7) + 1, fake)):
        with pytest.raises(Bd.AdpsgdError) as ei:
            Bd.adpsgd_consensus_static(ptr, stride, L, P, out, None)
        assert ei.value.code == Bd.EINVAL and Bd.adpsgd_last_error()
