"""The march and the chain of kernels of the other schemes (PPM, CTU, dual
energy), told apart by the library's own rule: every pair of projection and
solver family that has its own march kernels, at sizes on the march's side of
the rule, bitwise against the chain."""

import pytest

torch = pytest.importorskip("torch")

from paper_1712_07070_amd import hydro as H  # noqa: E402

M, C, PPM, CHR, DE = H.SCHEME_MHM, H.SCHEME_CTU, H.PPM, H.CHARACTERISTIC, H.DUAL_ENERGY
VL, ROE = H.LIMITER_VANLEER, H.RIEMANN_ROE


def chain_sizes(word, dtype, n=200):
    ghost = 3 if word & PPM else 2
    return [G for G in range(1, n) if H.ext_uses_chain(G, ghost, dtype, word)]


@pytest.mark.parametrize("word,f64,f32", [
    (M | PPM, [(1, 5)], [(1, 7)]),
    (M | PPM | CHR | ROE, [(1, 5)], [(1, 7)]),
    (M | PPM | DE, [(1, 11)], [(1, 10)]),
    (M | DE, [], []),
    (M | DE | CHR | VL, [], []),
    (M | VL | ROE, [], []),                        # the default march's words
    (C, [(1, 4)], [(1, 6)]),
    (C | CHR, [(1, 4)], [(1, 8)]),
    (C | CHR | VL, [(1, 11), (17, 20)], [(1, 8)]),
    (C | DE, [(1, 14), (17, 20)], [(1, 6)]),
    (C | DE | CHR | VL, [(1, 14), (17, 20)], [(1, 6)]),
    (C | PPM, [(1, 52), (65, 80)], [(1, 52)]),
    (C | PPM | CHR | ROE, [(1, 52), (65, 80)], [(1, 52)]),
    (C | PPM | DE, [(1, 96)], [(1, 52), (65, 80)]),
])
def test_rule_between_march_and_chain(word, f64, f32):
    for dtype, ranges in ((torch.float64, f64), (torch.float32, f32)):
        assert chain_sizes(word, dtype) == [G for a, b in ranges for G in range(a, b + 1)]


def test_rule_refuses_what_the_step_refuses():
    lib = H.load()
    assert lib.hydro_ext_uses_chain(-1, 3, 0, M | PPM) == lib.hydro_ext_uses_chain(1, 2, 0, M | PPM) == -1
    assert lib.hydro_ext_uses_chain(1, 3, 2, M | PPM) == lib.hydro_ext_uses_chain(1, 3, 0, M | (3 << 16)) == -1


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


def same(a, b):
    return bool(((a == b) | (torch.isnan(a) & torch.isnan(b))).all())


# (word, groups): the first size past the chain and one of whole or half groups
MARCH = [
    (M | PPM, 8), (M | PPM | ROE, 130), (M | PPM | CHR, 12), (M | PPM | CHR | ROE | VL, 270),
    (M | PPM | DE | H.RIEMANN_HLLE, 12), (M | PPM | DE | ROE, 130), (M | PPM | CHR | DE, 40),
    (M | PPM | CHR | DE | ROE, 270),
    (C, 7), (C | ROE, 270), (C | CHR, 9), (C | CHR | VL, 23), (C | CHR | ROE, 130), (C | CHR | ROE | VL, 515),
    (C | DE, 23), (C | DE | ROE, 130), (C | CHR | DE, 270), (C | CHR | DE | ROE | VL, 23),
    (C | PPM, 53), (C | PPM | ROE, 130), (C | PPM | CHR, 97), (C | PPM | CHR | H.LIMITER_HYBRID, 270),
    (C | PPM | CHR | ROE, 130), (C | PPM | CHR | ROE | VL, 515),
    (C | PPM | DE, 97), (C | PPM | DE | ROE, 130), (C | PPM | CHR | DE, 130), (C | PPM | CHR | DE | ROE | VL, 270),
]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("word,G", MARCH)
def test_march_of_every_copy_equals_chain(dtype, word, G):
    print("march copy", hex(word), G, dtype, flush=True)
    ghost, nf = (3 if word & PPM else 2), (6 if word & DE else 5)
    assert not H.ext_uses_chain(G, ghost, dtype, word) and H.ext_uses_chain(2, ghost, dtype, word)
    for p_low in (0.5, 1e-3):
        pad = noise(G, 16 + 2 * ghost, nf, dtype, p_low)
        ff = torch.zeros((G, 9, 5, 16, 16), dtype=dtype, device="cuda") if nf == 5 else None
        n_bad = torch.zeros(1, dtype=torch.int32, device="cuda")
        got = H.advance_ext(pad, 2e-4, 1.0 / 64, 5.0 / 3.0, word, n_bad=n_bad, face_flux=ff)
        ref, n_ref = torch.empty_like(got), torch.zeros_like(n_bad)
        ff_ref = None if ff is None else torch.empty_like(ff)
        work = H.ext_workspace(2, ghost, dtype, word)
        for g in range(0, G, 2):
            e = min(g + 2, G)
            H.advance_ext(pad[g:e], 2e-4, 1.0 / 64, 5.0 / 3.0, word, out=ref[g:e], n_bad=n_ref, work=work,
                          face_flux=None if ff is None else ff_ref[g:e])
        assert same(got, ref) and int(n_bad) == int(n_ref) and (p_low > 0.1 or int(n_ref) > 0)
        assert ff is None or same(ff, ff_ref)
