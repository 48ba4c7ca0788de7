"""The step adjoint of few groups (each shared by several workgroups, one per z
segment) against whole groups, bitwise: the same groups in a batch too large to
be split, for batches that take 14, 7, 5, 4, 3, 2 segments and none."""

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

GAMMA, DT, DX = 5.0 / 3.0, 1e-3, 1.0 / 64


@pytest.fixture(scope="module")
def hydro():
    from paper_1712_07070_amd import hydro as h
    h.load()
    return h


def noise(G, P, dtype, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    u = lambda: torch.rand((G, P, P, P), generator=g, device="cuda", dtype=torch.float64)
    rho = 0.05 + 1.95 * u()
    v = [0.5 * torch.randn((G, P, P, P), generator=g, device="cuda", dtype=torch.float64) for _ in range(3)]
    p = 0.5 + 1.5 * u()
    E = p / (GAMMA - 1.0) + 0.5 * rho * (v[0] ** 2 + v[1] ** 2 + v[2] ** 2)
    return torch.stack([rho] + [rho * c for c in v] + [E], 1).to(dtype).contiguous()


LATTICES = [(1, 1, 1), (3, 2, 3), (4, 3, 3), (5, 5, 2), (4, 4, 4), (6, 4, 4), (8, 5, 2), (16, 4, 2), (8, 8, 4), (7, 6, 7)]
BC = (0, 0, 1, 1, 0, 0)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("ng", LATTICES)
@pytest.mark.parametrize("scheme", ["second", "first"])
def test_adjoint_segments_bitwise(hydro, dtype, ng, scheme):
    print("adjoint segments", dtype, ng, scheme, flush=True)
    G = ng[0] * ng[1] * ng[2]
    word = hydro.SCHEME_MHM_PLM_HLLC | (hydro.FIRST_ORDER if scheme == "first" else 0)
    level = noise(G, 16, dtype, 3)
    gout = torch.randn((G, 5, 16, 16, 16), generator=torch.Generator(device="cuda").manual_seed(4), device="cuda",
                       dtype=torch.float64).to(dtype)
    pad = hydro.fill_ghosts(level, ng, 3, BC)
    few = hydro.advance_adjoint(pad, gout, DT, DX, GAMMA, scheme=word)
    # the same groups over and over, in a batch that is not split
    n = max(1024, G)
    idx = torch.arange(n, device="cuda") % G
    many = hydro.advance_adjoint(pad[idx].contiguous(), gout[idx].contiguous(), DT, DX, GAMMA, scheme=word)
    assert bool(torch.isfinite(many).all()) and float(many.abs().max()) > 0
    assert torch.equal(many, few[idx])
    # the level form: the same cotangents, gathered
    work = hydro.adjoint_workspace(G, dtype, True)
    work.fill_(255)  # NaN in whatever is read without being written
    lev = hydro.advance_level_adjoint(level, gout, ng, BC, DT, DX, GAMMA, scheme=word, work=work)
    work.fill_(255)
    dt_dev = torch.full((1,), DT, dtype=torch.float64, device="cuda")
    assert torch.equal(lev, hydro.advance_level_adjoint(level, gout, ng, BC, 1.0, DX, GAMMA, scheme=word, work=work,
                                                        dt_dev=dt_dev))
    ref = hydro.gather_ghost_adjoint(many[:G].contiguous(), ng, 3, BC)
    # the two gathers add up to 8 terms per cell in the same order, the padded
    # one with the zeros of the cells that the step does not read in between
    assert torch.equal(lev, ref)
