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


@pytest.mark.parametrize("ghost", [2, 3, 5])
@pytest.mark.parametrize("n0,boxes", [(2, ()), (3, (((2, 4),) * 3,)), (3, (((0, 6),) * 3, ((0, 12),) * 3)),
                                      (3, (((2, 4),) * 3, ((5, 7),) * 3))])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_direct_steps_take_no_more_memory_than_padded_ones(lib, dtype, n0, boxes, ghost):
    """The second state buffers of the direct step fit in what its scratch cells
    take less than padded blocks (which the other words hold, with old states
    for all levels but the finest): the largest hierarchy that fits the card is
    no smaller."""
    def held(s):
        return sum(t.numel() * t.element_size() for ts in (s.pad, s.work, s.flux, s.alt, s.reg) for t in ts
                   if t is not None)
    direct = solver(dtype=dtype, n0=n0, boxes=boxes, ghost=ghost)
    padded = solver(hydro.SCHEME_MHM_PLM_HLLC | hydro.RIEMANN_ROE, dtype=dtype, n0=n0, boxes=boxes, ghost=ghost)
    assert direct.direct and not padded.direct
    assert held(direct) <= held(padded)


# The scratch cells are addressed by arithmetic that runs only on the device; an
# index used twice or beyond the block would give wrong cells (or write outside
# the buffer).  The function is taken from the kernel header as written and
# compiled for the host.
_SHELL_CHECK = r"""
#include <cstdio>
#include <vector>
%s
int main() {
  std::vector<int> seen(kShellCells, 0);
  int cells = 0, bad = 0;
  for (int z = -2; z <= 17; ++z) for (int y = -2; y <= 17; ++y) for (int x = -2; x <= 17; ++x) {
    if (x >= 0 && x <= 15 && y >= 0 && y <= 15 && z >= 0 && z <= 15) continue;
    const unsigned i = shell_cell(x, y, z);
    ++cells;
    if (i >= unsigned(kShellCells)) ++bad;
    else ++seen[i];
  }
  for (int v : seen) bad += v != 1;
  printf("%%d %%d\n", cells, bad);
  return bad != 0;
}
"""


def test_scratch_cells_of_a_group_are_distinct(tmp_path):
    import os
    import re
    import shutil
    import subprocess
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    src = open(os.path.join(root, "paper_1712_07070_amd", "csrc", "kernels.h")).read()
    i = src.index("constexpr int kShellCells")
    j = src.index("}\n", src.index(" shell_cell(", i)) + 2
    body = re.sub(r"__host__ __device__ __forceinline__|__device__ __forceinline__", "inline", src[i:j])
    cpp, exe = tmp_path / "shell.cpp", tmp_path / "shell"
    cpp.write_text(_SHELL_CHECK % body)
    subprocess.run([gxx, "-O2", "-std=c++17", str(cpp), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.stdout.split() == [str(20 ** 3 - 16 ** 3), "0"]
