"""Few groups shared by several workgroups, one per z segment, against whole
groups: the same bits, unphysical counts, face fluxes and CFL time-steps, for
lattices that take 16, 8, 4, 2 segments and none.  Whole groups run where the
caller sets the launch shape (level, batched) and in batches too large to be
split (padded)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

GAMMA, DX = 5.0 / 3.0, 1.0 / 64


@pytest.fixture(scope="module")
def hydro():
    from paper_1712_07070_amd import hydro as h
    h.load()
    return h


def noise(G, P, dtype, low=False, seed=5):
    """White noise; low: pressures down to 1e-3, so that items are unphysical."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    u = lambda: torch.rand((G, P, P, P), generator=g, device="cuda", dtype=torch.float64)
    rho = 0.05 + 1.95 * u()
    v = [0.5 * torch.randn((G, P, P, P), generator=g, device="cuda", dtype=torch.float64) for _ in range(3)]
    p = (1e-3 if low else 0.5) + 1.5 * u() ** (6 if low else 1)
    E = p / (GAMMA - 1.0) + 0.5 * rho * (v[0] ** 2 + v[1] ** 2 + v[2] ** 2)
    return torch.stack([rho] + [rho * c for c in v] + [E], 1).to(dtype).contiguous()


def same(a, b):
    return bool(((a == b) | (torch.isnan(a) & torch.isnan(b))).all())


LATTICES = [(1, 1, 1), (3, 2, 1), (4, 4, 2), (5, 3, 3), (8, 4, 3), (8, 6, 4), (7, 7, 4), (8, 8, 8)]
BC = (0, 0, 1, 1, 0, 0)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("ng", LATTICES)
@pytest.mark.parametrize("form", ["plain", "cfl", "patch"])
def test_level_segments_bitwise(hydro, dtype, ng, form):
    print("level segments", dtype, ng, form, flush=True)
    G = ng[0] * ng[1] * ng[2]
    whole = hydro.Context()
    hydro.set_variant(dtype, 6, ctx=whole)
    split = hydro.Context()
    for low in (False, True):
        U = noise(G, 16, dtype, low)
        got = []
        for ctx in (whole, split):
            n_bad = torch.zeros(1, dtype=torch.int32, device="cuda")
            dts = torch.full((3,), float("inf"), dtype=torch.float64, device="cuda")
            dts[0], dts[2] = 1e-4, 1.0
            patch = torch.zeros(8 * G, dtype=torch.float64, device="cuda") if form == "patch" else None
            kw = {} if form == "plain" else dict(dt_dev=dts[0:1], dt_next=dts[1:2], dt_reset=dts[2:3],
                                                 dt_patch_next=patch)
            out = hydro.advance_level(U, ng, BC, 1e-4, DX, GAMMA, n_bad=n_bad, ctx=ctx, **kw)
            got.append((out, n_bad, dts, torch.zeros(1, device="cuda") if patch is None else patch))
        for a, b in zip(*got):
            assert same(a, b)
        if form != "plain":
            assert float(got[1][2][2]) == float("inf")


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("G", [1, 6, 32, 45, 96, 196])
@pytest.mark.parametrize("word", ["advance", "davis", "first-order", "roe", "char-hlle"])
def test_padded_segments_bitwise(hydro, dtype, G, word):
    print("padded segments", dtype, G, word, flush=True)
    h, n_all = hydro, 1400   # enough groups that none is split
    sch = {"advance": h.SCHEME_MHM, "davis": h.SCHEME_MHM | h.WAVESPEED_DAVIS,
           "first-order": h.SCHEME_MHM | h.FIRST_ORDER, "roe": h.SCHEME_MHM | h.RIEMANN_ROE | h.LIMITER_VANLEER,
           "char-hlle": h.SCHEME_MHM | h.CHARACTERISTIC | h.RIEMANN_HLLE}[word]
    for low in (False, True):
        few = noise(G, 20, dtype, low)
        # the others hold a uniform state, which adds nothing to the count
        rest = torch.tensor([1.0, 0.1, 0.2, 0.3, 2.0], dtype=dtype, device="cuda").view(1, 5, 1, 1, 1)
        many = torch.cat([few, rest.expand(n_all - G, 5, 20, 20, 20)]).contiguous()
        got = []
        for U in (many, few):
            n_bad = torch.zeros(1, dtype=torch.int32, device="cuda")
            ff = torch.zeros((U.shape[0], 9, 5, 16, 16), dtype=dtype, device="cuda")
            if word == "advance":
                out = h.advance(U, 1e-4, DX, GAMMA, n_bad=n_bad)
            else:
                out = h.advance_ext(U, 1e-4, DX, GAMMA, sch, n_bad=n_bad, face_flux=ff)
            got.append((out[:G], n_bad, ff[:G]))
        for a, b in zip(*got):
            assert same(a, b)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("lattices", [[(2, 1, 1)], [(2, 2, 2), (3, 1, 4)], [(4, 4, 4), (5, 5, 5), (2, 3, 1)]])
@pytest.mark.parametrize("patch", [False, True])
def test_batched_segments_bitwise(hydro, dtype, noalloc, lattices, patch):
    print("batched segments", dtype, noalloc, lattices, patch, flush=True)
    whole = hydro.Context()
    hydro.set_batched_variant(dtype, 0, ctx=whole)
    got = []
    for ctx in (whole, hydro.Context()):
        n_bad = torch.zeros(1, dtype=torch.int32, device="cuda")
        work = torch.zeros(hydro.BATCH_WORK_WORDS, dtype=torch.int32, device="cuda")
        dts = torch.full((2 + len(lattices),), float("inf"), dtype=torch.float64, device="cuda")
        dts[0] = 2e-4
        entries, outs = [], []
        for l, ng in enumerate(lattices):
            G = ng[0] * ng[1] * ng[2]
            U = noise(G, 16, dtype, low=l == 1, seed=l)
            out = torch.zeros_like(U)
            pt = torch.zeros(8 * G, dtype=torch.float64, device="cuda")
            cfl = dict(dt_dev_scale=0.5 ** l, c_cfl=0.5, dt_next_scale=2.0 ** l, dt_next=dts[1:2])
            if patch:
                cfl["dt_patch"] = pt
            entries.append((U, out, ng, BC, 1e-4, DX, dts[0:1], cfl))
            outs += [out, pt]
        if noalloc:
            hydro.advance_batched_noalloc(entries, GAMMA, n_bad=n_bad, ctx=ctx)
        else:
            hydro.advance_batched(entries, GAMMA, work, n_bad=n_bad, ctx=ctx)
        assert int(work.abs().sum()) == 0
        got.append(outs + [n_bad, dts])
    for a, b in zip(*got):
        assert same(a, b)


def test_segment_counts_cover_the_rule():
    """The lattices above take every split of the rule (march_segments)."""
    def segments(G, slots, share):
        best, cost = 1, 0.0
        for s in (1, 2, 4, 8, 16):
            n = (G * s + 255) // 256
            full, rest = (n // slots) * (1 + share * (slots - 1)), n % slots
            c = (full + (1 + share * (rest - 1) if rest else 0)) * (16 // s + 2)
            if s == 1:
                cost = 0.9 * c
            elif c < cost:
                best, cost = s, c
        return best
    for slots, share in ((2, 0.5), (3, 0.22)):
        assert {segments(int(np.prod(ng)), slots, share) for ng in LATTICES} == {1, 2, 4, 8, 16}
