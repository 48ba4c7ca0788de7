"""Every limiter, projection and solver family of the PLM march (their own
kernel copies, hydro_advance_ext) and its first-order copies: whole groups, z
segments of every length the sizes give, with and without face fluxes, the
same bits; the step against the oracle at the bars of
test_gpu_ext_schemes.py."""

import numpy as np
import pytest

import oracle
from paper_1712_07070_amd import workloads as W
from tests.oracle_runs import assert_parity

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = {np.float64: 1e-12, np.float32: 1e-5}
LIMITERS = {"gminmod": 0, "vanleer": oracle.LIMITER_VANLEER, "vanalbada": oracle.LIMITER_VANALBADA,
            "hybrid": oracle.LIMITER_HYBRID}
WORDS = {"%s%s-%s" % (l, c, s): oracle.SCHEME_MHM | lw | cw | sw
         for l, lw in LIMITERS.items() for c, cw in (("", 0), ("-char", oracle.CHARACTERISTIC))
         for s, sw in (("hllc", 0), ("roe", oracle.RIEMANN_ROE)) if lw | cw | sw}
WORDS["first-hlle"] = oracle.SCHEME_MHM | oracle.FIRST_ORDER | oracle.RIEMANN_HLLE
WORDS["first-char-vanleer-roe"] = (oracle.SCHEME_MHM | oracle.FIRST_ORDER | oracle.RIEMANN_ROE |
                                   oracle.CHARACTERISTIC | oracle.LIMITER_VANLEER)


@pytest.fixture(scope="module")
def hydro():
    from paper_1712_07070_amd import hydro as h
    h.load()
    return h


def same(a, b):
    return bool(((a == b) | (torch.isnan(a) & torch.isnan(b))).all())


def low_pressure_groups(lv):
    """Eight padded groups of noise with pressures down to 1e-3."""
    rng = np.random.default_rng(7)
    P = 22
    rho = rng.uniform(0.05, 2.0, (8, P, P, P))
    v = 0.5 * rng.standard_normal((3, 8, P, P, P))
    p = 1e-3 * 2000.0 ** rng.uniform(0.0, 1.0, (8, P, P, P))
    E = p / (lv.gamma - 1.0) + 0.5 * rho * (v ** 2).sum(0)
    return np.ascontiguousarray(np.stack([rho, rho * v[0], rho * v[1], rho * v[2], E], 1))


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("name", list(WORDS))
def test_plm_word_copies(hydro, name, dtype):
    print("plm word", name, dtype.__name__, flush=True)
    word, tdt = WORDS[name], torch.float64 if dtype == np.float64 else torch.float32
    lv = W.white_noise(32)
    pad = oracle.fill_ghosts(lv.U.astype(dtype).astype(np.float64), lv.ng, 3, lv.bc)
    dt = float(oracle.dt_patch(pad, lv.dx, lv.gamma, 0.5).min())
    assert hydro.padded_segments(1400, tdt) == 1
    assert [hydro.padded_segments(8 * n, tdt) for n in (1, 5, 17)] == ([16, 4, 2] if tdt == torch.float64
                                                                       else [16, 16, 4])
    for blocks in (pad, low_pressure_groups(lv)):
        few = torch.from_numpy(blocks.astype(dtype)).cuda()
        res = []
        for n in (1, 5, 17, 175):
            U = few.repeat(n, 1, 1, 1, 1)
            n_bad = torch.zeros(2, dtype=torch.int32, device="cuda")
            ff = torch.zeros((8 * n, 9, 5, 16, 16), dtype=tdt, device="cuda")
            out = hydro.advance_ext(U, dt, lv.dx, lv.gamma, word, n_bad=n_bad[:1])
            with_flux = hydro.advance_ext(U, dt, lv.dx, lv.gamma, word, n_bad=n_bad[1:], face_flux=ff)
            assert same(out, with_flux) and int(n_bad[0]) == int(n_bad[1]) and int(n_bad[0]) % n == 0
            first = out[:8]
            assert same(out, first.repeat(n, 1, 1, 1, 1)) and same(ff, ff[:8].repeat(n, 1, 1, 1, 1))
            res.append((first.clone(), ff[:8].clone(), int(n_bad[0]) // n))
            del U, out, with_flux, ff
        for r in res[1:]:
            assert same(r[0], res[0][0]) and same(r[1], res[0][1]) and r[2] == res[0][2]
        if blocks is pad:
            ref, nb = oracle.step_any(pad, dt, lv.dx, lv.gamma, 1.5, word)
            assert_parity(res[0][0].cpu().numpy(), ref, TOL[dtype], name)
            assert res[0][2] == nb == 0
        else:
            assert res[0][2] > 0 or "first" in name
