"""The ghost fill at the edges of its launch rule (padded planes dealt to the
XCDs in contiguous ranges; pairs of cells stored together where the
destination is aligned to a pair), bitwise against the oracle."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hydro():
    from paper_1712_07070_amd import hydro as h
    h.load()
    return h


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("ng,ghost,bc", [((1, 1, 1), 0, (0,) * 6), ((1, 1, 1), 16, (0, 0, 1, 1, 0, 0)),
                                         ((3, 1, 2), 2, (1,) * 6), ((1, 5, 1), 3, (0, 0, 1, 1, 0, 0))])
def test_fill_ghosts_edges_bitwise(hydro, dtype, shift, ng, ghost, bc):
    """Smallest lattices and ghost widths, plane counts that leave the XCDs'
    ranges uneven, and a destination off the pair alignment by one element."""
    print("fill_ghosts", dtype.__name__, shift, ng, ghost, flush=True)
    G, P = ng[0] * ng[1] * ng[2], 16 + 2 * ghost
    level = np.random.default_rng(7).normal(size=(G, 5, 16, 16, 16)).astype(dtype)
    ref = oracle.fill_ghosts(level.astype(np.float64), ng, ghost, bc).astype(dtype)
    flat = torch.zeros(G * 5 * P ** 3 + 2, dtype=torch.from_numpy(level).dtype, device="cuda")
    out = flat[shift:shift + G * 5 * P ** 3].view(G, 5, P, P, P)
    hydro.fill_ghosts(torch.from_numpy(level).cuda(), ng, ghost, bc, out=out)
    assert np.array_equal(out.cpu().numpy(), ref)
    assert float(flat[:shift].abs().sum() + flat[shift + out.numel():].abs().sum()) == 0.0   # nothing beside it
