"""Host-side logic of the coupled AMR driver (no GPU): which buffers its
substeps read and write, with the library's launches replaced by recorders."""

import pytest

torch = pytest.importorskip("torch")

from paper_1712_07070_amd import hydro  # noqa: E402
from paper_1712_07070_amd import workloads as W  # noqa: E402


class Recorder:
    """Stands for the library: records the state buffers of every level step,
    and fails at the step `fail_at`."""

    def __init__(self):
        self.steps, self.fail_at = [], None

    def hydro_ext_workspace_bytes(self, *args):
        return 0

    def hydro_amr_advance(self, fine, *args):
        self.steps.append((fine._obj.U_dev, args[12]))   # old states, U_out_dev
        return -1 if len(self.steps) - 1 == self.fail_at else 0

    def hydro_strerror(self, status):
        return b"refused"

    def __getattr__(self, name):
        return lambda *args: 0


@pytest.fixture
def lib(monkeypatch):
    rec = Recorder()
    monkeypatch.setattr(hydro, "load", lambda: rec)
    monkeypatch.setattr(hydro, "_stream", lambda: 0)
    monkeypatch.setattr(hydro, "_dev", lambda t, name: t.data_ptr())
    return rec


def solver(scheme=hydro.SCHEME_MHM_PLM_HLLC, dtype=torch.float64, n0=3, boxes=(((2, 4),) * 3, ((5, 7),) * 3), **kw):
    pos = W.nested_positions(n0, boxes)
    U = [torch.zeros((len(p), 5, 16, 16, 16), dtype=dtype) for p in pos]
    return hydro.AmrSolver((n0,) * 3, pos, U, 1.0 / 48, 5.0 / 3.0, scheme=scheme, **kw)


@pytest.mark.parametrize("fail_at", range(7))
def test_failed_substep_leaves_the_solver_usable(lib, fail_at):
    """A step that raises in any of its substeps (levels 0 1 2 2 1 2 2) keeps no
    state behind: the next one starts every level from the caller's tensor and
    ends there."""
    s = solver()
    s.step(1e-3)
    clean, lib.steps = lib.steps, []
    assert len(clean) == 7
    for l, (first, second) in ((1, (1, 4)), (2, (2, 3)), (2, (5, 6))):
        mine = s.U[l].data_ptr()
        assert clean[first][0] == mine and clean[second] == (clean[first][1], mine)
    lib.fail_at = fail_at
    with pytest.raises(hydro.HydroError):
        s.step(1e-3)
    lib.steps, lib.fail_at = [], None
    s.step(1e-3)
    assert lib.steps == clean
