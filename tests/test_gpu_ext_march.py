"""The march of the other schemes (PPM, CTU, dual energy) against the chain of
per-cell kernels, which takes calls of few groups: the same bits for every
split of a group into z segments (16, 8, 4, 2, 1 as the number of groups
grows), every mode, and the counts of unphysical items and face fluxes the
same.  The chain itself is checked against the oracle at those sizes in
test_gpu_ext_schemes.py."""

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hydro():
    from paper_1712_07070_amd import hydro as h
    h.load()
    return h


def noise(G, P, nf, dtype, p_low, seed=11):
    """White noise; with p_low = 1e-3 some faces and cells turn unphysical."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    u = lambda: torch.rand((G, P, P, P), generator=g, device="cuda", dtype=torch.float64)
    rho = 0.05 + 1.95 * u() if p_low < 0.1 else 0.5 + 1.5 * u()
    v = [0.5 * torch.randn((G, P, P, P), generator=g, device="cuda", dtype=torch.float64) for _ in range(3)]
    p = p_low * (2.0 / p_low) ** u()
    f = [rho] + [rho * c for c in v] + [1.5 * p + 0.5 * rho * (v[0] ** 2 + v[1] ** 2 + v[2] ** 2)]
    if nf == 6:
        f.append(p / rho ** (2.0 / 3.0))
    return torch.stack(f, 1).to(dtype).contiguous()


def words(h):
    return {
        "ppm-hllc-hybrid": (h.SCHEME_MHM | h.PPM | h.LIMITER_HYBRID, 3),
        "ppm-char-roe": (h.SCHEME_MHM | h.PPM | h.CHARACTERISTIC | h.RIEMANN_ROE, 4),
        "ppm-first-order": (h.SCHEME_MHM | h.PPM | h.FIRST_ORDER, 3),
        "ppm-hlle-davis-dual": (h.SCHEME_MHM | h.PPM | h.RIEMANN_HLLE | h.WAVESPEED_DAVIS | h.DUAL_ENERGY, 3),
        "plm-char-vanleer-dual": (h.SCHEME_MHM | h.CHARACTERISTIC | h.LIMITER_VANLEER | h.DUAL_ENERGY, 2),
        "ctu-roe": (h.SCHEME_CTU | h.RIEMANN_ROE, 2),
        "ctu-char-hlle-dual": (h.SCHEME_CTU | h.CHARACTERISTIC | h.RIEMANN_HLLE | h.DUAL_ENERGY, 3),
        "ctu-ppm-vanalbada": (h.SCHEME_CTU | h.PPM | h.LIMITER_VANALBADA, 3),
        "ctu-ppm-roe-dual": (h.SCHEME_CTU | h.PPM | h.RIEMANN_ROE | h.DUAL_ENERGY, 3),
    }


def same(a, b):
    return bool(((a == b) | (torch.isnan(a) & torch.isnan(b))).all())


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("name,G", [("ppm-hllc-hybrid", 3), ("ppm-hllc-hybrid", 35), ("ppm-hllc-hybrid", 70),
                                    ("ppm-hllc-hybrid", 100), ("ppm-hllc-hybrid", 200), ("ppm-hllc-hybrid", 515),
                                    ("ppm-char-roe", 9), ("ppm-char-roe", 130), ("ppm-first-order", 20),
                                    ("ppm-hlle-davis-dual", 6), ("ppm-hlle-davis-dual", 130),
                                    ("plm-char-vanleer-dual", 7), ("plm-char-vanleer-dual", 260), ("ctu-roe", 7),
                                    ("ctu-roe", 33), ("ctu-roe", 100), ("ctu-roe", 200), ("ctu-roe", 515),
                                    ("ctu-char-hlle-dual", 60), ("ctu-ppm-vanalbada", 41), ("ctu-ppm-vanalbada", 260),
                                    ("ctu-ppm-roe-dual", 90), ("ppm-hlle-davis-dual", 9), ("plm-char-vanleer-dual", 9),
                                    ("ctu-char-hlle-dual", 9), ("ctu-ppm-vanalbada", 49)])
def test_march_equals_chain_bitwise(hydro, dtype, name, G):
    word, ghost = words(hydro)[name]
    print("ext march", name, G, dtype, flush=True)
    nf = 6 if word & hydro.DUAL_ENERGY else 5
    for p_low in (0.5, 1e-3):
        pad = noise(G, 16 + 2 * ghost, nf, dtype, p_low)
        dt, dx = 2e-4, 1.0 / 64
        ff = torch.zeros((G, 9, 5, 16, 16), dtype=dtype, device="cuda") if nf == 5 else None
        n_bad = torch.zeros(1, dtype=torch.int32, device="cuda")
        got = hydro.advance_ext(pad, dt, dx, 5.0 / 3.0, word, n_bad=n_bad, face_flux=ff)
        ref, n_ref = torch.empty_like(got), torch.zeros_like(n_bad)
        ff_ref = None if ff is None else torch.empty_like(ff)
        work = hydro.ext_workspace(2, ghost, dtype, word)
        for g in range(0, G, 2):   # at most two groups a call: the chain
            e = min(g + 2, G)
            hydro.advance_ext(pad[g:e], dt, dx, 5.0 / 3.0, word, out=ref[g:e], n_bad=n_ref, work=work,
                              face_flux=None if ff is None else ff_ref[g:e])
        assert same(got, ref)
        assert int(n_bad) == int(n_ref)
        # the low-pressure noise is counted (the first-order step, without slopes, keeps it physical)
        assert p_low > 0.1 or int(n_ref) > 0 or word & hydro.FIRST_ORDER
        if ff is not None:
            assert same(ff, ff_ref)
