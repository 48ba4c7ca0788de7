"""How many workgroups share a group (the library's own rule, asked on the
host), and that a tuned launch shape splits few groups as a default one does
while a shape that the caller set does not."""

import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1712_07070_amd import hydro  # noqa: E402

LATTICES = [(1, 1, 1), (3, 2, 1), (4, 4, 2), (5, 3, 3), (8, 4, 3), (8, 6, 4), (7, 7, 4), (8, 8, 8)]


@pytest.fixture
def host(monkeypatch):
    """Host tensors in place of device ones: nothing is launched."""
    monkeypatch.setattr(hydro, "_dev", lambda t, name: t.data_ptr())


def entries(lattices, dtype, cfl=None):
    out = []
    for ng in lattices:
        G = int(np.prod(ng))
        U = torch.empty((G, 5, 16, 16, 16), dtype=dtype)
        out.append((U, torch.empty_like(U), ng, (0,) * 6, 1e-3, 0.1, None, cfl))
    return out


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_every_split_occurs_and_large_batches_are_whole(dtype):
    """The lattices of the bitwise segment tests take every split, and the
    batches those tests compare with take none."""
    ctx = hydro.Context()
    splits = [hydro.level_segments(ng, dtype, ctx=ctx) for ng in LATTICES]
    assert set(splits) == {1, 2, 4, 8, 16} and splits == sorted(splits, reverse=True)
    assert hydro.padded_segments(0, dtype) == hydro.padded_segments(1024, dtype) == 1
    assert hydro.padded_segments(1400, dtype) == hydro.level_segments((16, 16, 16), dtype, ctx=ctx) == 1
    for ng in LATTICES:
        assert hydro.level_segments(ng, dtype, with_cfl=True, ctx=ctx) == hydro.level_segments(ng, dtype, ctx=ctx)
        # per-patch time-steps: no segment holds part of a patch
        assert hydro.level_segments(ng, dtype, True, True, ctx=ctx) == min(2, hydro.level_segments(ng, dtype, ctx=ctx))


def test_queries_refuse_bad_arguments():
    lib = hydro.load()
    assert lib.hydro_padded_segments(-1, 0) == lib.hydro_padded_segments(1, 2) == -1
    assert lib.hydro_level_segments(None, 0, 1, 1, 0, 0, 0) == lib.hydro_level_segments(None, 1, 1, 1, 2, 0, 0) == -1
    assert lib.hydro_batched_segments(None, None, 1, 0) == -1
    assert lib.hydro_set_batched_tuned(None, 0, 1) == lib.hydro_set_batched_tuned(None, 2, 1) == -1


def test_level_shape_set_by_the_caller_runs_whole_groups(tmp_path):
    path = tmp_path / "tune.json"
    path.write_text('{"version": 1, "entries": {"level/f64/plain/2x2x2": 3}}')
    ctx = hydro.Context(str(path))
    assert hydro.level_segments((2, 2, 2), torch.float64, ctx=ctx) == 16     # tuned
    hydro.set_level_variant(torch.float64, False, 6, ctx=ctx)
    assert hydro.level_segments((2, 2, 2), torch.float64, ctx=ctx) == 1
    assert hydro.level_segments((2, 2, 2), torch.float64, with_cfl=True, ctx=ctx) == 16


def test_batched_shape_chosen_by_timing_splits_few_groups(host, tmp_path):
    lv = entries([(2, 2, 2), (3, 1, 4)], torch.float64)
    ctx = hydro.Context()
    default = hydro.batched_segments(lv, ctx)
    assert default == hydro.padded_segments(20, torch.float64) > 1
    hydro.set_batched_variant(torch.float64, 5, ctx=ctx)
    assert hydro.batched_segments(lv, ctx) == 1
    assert hydro.batched_segments(entries([(2, 2, 2)], torch.float32), ctx) == 16
    hydro.set_batched_tuned(torch.float64, 4, ctx=ctx)
    assert hydro.batched_segments(lv, ctx) == default and hydro.get_batched_variant(torch.float64, ctx) == 4


def test_tuning_the_w_cycle_keeps_the_split(host, monkeypatch):
    """MultiLevel.autotune installs the shape of the best total time, and its
    few groups are split as in an untuned context."""
    ml = object.__new__(hydro.MultiLevel)
    ml.L, ml.adaptive, ml.gamma, ml.dtype, ml.ctx = 2, False, 1.4, torch.float64, hydro.Context()
    ml.work = torch.zeros(hydro.BATCH_WORK_WORDS, dtype=torch.int32)
    lv = entries([(2, 2, 2), (3, 1, 4)], torch.float64)
    monkeypatch.setattr(ml, "_entries", lambda lvls, s=0: [lv[l] for l in lvls], raising=False)
    times = [2.0] * hydro.BATCHED_VARIANTS
    times[7] = 1.0
    monkeypatch.setattr(hydro, "autotune_batched", lambda *a, **k: (7, times))
    before = hydro.batched_segments(lv, ml.ctx)
    assert ml.autotune()[0] == 7
    assert hydro.get_batched_variant(torch.float64, ml.ctx) == 7
    assert hydro.batched_segments(lv, ml.ctx) == before > 1


@pytest.mark.gpu
def test_batched_tuner_lifts_a_shape_set_before(tmp_path):
    """A shape that the caller set, then hydro_autotune_batched on the same
    levels: the tuned entry is used, and few groups are split under it."""
    print("batched tuner after a set shape", flush=True)
    ctx = hydro.Context()
    lv = [tuple(t.cuda() if isinstance(t, torch.Tensor) else t for t in e)
          for e in entries([(2, 2, 2), (3, 1, 4)], torch.float64)]
    for e in lv:
        e[0].copy_(torch.tensor([1.0, 0.1, 0.2, 0.3, 2.0], dtype=torch.float64, device="cuda").view(1, 5, 1, 1, 1))
    work = torch.zeros(hydro.BATCH_WORK_WORDS, dtype=torch.int32, device="cuda")
    hydro.set_batched_variant(torch.float64, 5, ctx=ctx)
    assert hydro.batched_segments(lv, ctx) == 1
    hydro.autotune_batched(lv, 1.4, work, reps=1, ctx=ctx)
    assert ctx.num_tuned() == 1 and hydro.batched_segments(lv, ctx) > 1
    assert hydro.batched_segments(lv[:1], ctx) == 1   # other levels: still as set


def test_batched_shape_set_by_the_caller_replaces_tuned_ones_of_both_forms(host, tmp_path):
    """hydro_set_batched_variant stands in place of the tuned entries of its dtype,
    also those of launches that reduce CFL time-steps."""
    path = tmp_path / "tune.json"
    path.write_text('{"version": 1, "entries": {"batched/f64/2x2x2": 3, "batched-cfl/f64/2x2x2": 4, '
                    '"batched-cfl/f32/2x2x2": 2}}')
    ctx = hydro.Context(str(path))
    dt = torch.zeros(1, dtype=torch.float64)
    cfl = entries([(2, 2, 2)], torch.float64, dict(c_cfl=0.5, dt_next=dt))
    assert ctx.num_tuned() == 3 and hydro.batched_segments(cfl, ctx) > 1
    hydro.set_batched_variant(torch.float64, 5, ctx=ctx)
    assert ctx.num_tuned() == 1
    assert hydro.batched_segments(cfl, ctx) == hydro.batched_segments(entries([(2, 2, 2)], torch.float64), ctx) == 1
