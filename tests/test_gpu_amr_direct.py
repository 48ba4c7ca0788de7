"""hydro_amr_advance against hydro_amr_fill_ghosts + hydro_advance_ext on the
same levels: the new states and unphysical counts the same bits, the face
fluxes wherever the flux registers and the fix-up read them; lattices with
sides of every kind (siblings, missing siblings, periodic and outflow domain
faces), whole groups and z segments."""

import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hydro():
    from paper_1712_07070_amd import hydro as h
    h.load()
    return h


def boxes(n0, box):
    pos = [np.array([(x, y, z) for z in range(n0[2]) for y in range(n0[1]) for x in range(n0[0])], np.int32)]
    pos.append(np.array([(x, y, z) for z in range(*box[2]) for y in range(*box[1]) for x in range(*box[0])], np.int32))
    return pos


def flux_planes(n0, pos, l, bc, coupled):
    """[G, 9] bool: the planes of level l's groups read by hydro_amr_flux_accumulate
    (open sides) and, when coupled to the next level, by hydro_amr_fixup (a face
    between a refined patch and one that is not)."""
    def level(m):
        have = set(map(tuple, np.asarray(pos[m]).tolist()))
        n = [v << m for v in n0]

        def at(p):
            p = list(p)
            for d in range(3):
                if p[d] < 0 or p[d] >= n[d]:
                    if bc[2 * d + (p[d] >= n[d])] != 0:
                        return None   # beyond an outflow face
                    p[d] %= n[d]
            return tuple(p) in have
        return at
    own, fine = level(l), level(l + 1) if coupled else None
    need = np.zeros((len(pos[l]), 9), bool)
    for g, p in enumerate(np.asarray(pos[l]).tolist()):
        for d in range(3):
            for k in range(3):
                if k != 1:
                    q = list(p)
                    q[d] += k - 1
                    need[g, 3 * d + k] |= own(q) is False
                for a in range(2):
                    for b in range(2):
                        c = [2 * v for v in p]
                        c[d] += k
                        c[(d + 1) % 3] += a
                        c[(d + 2) % 3] += b
                        below = list(c)
                        below[d] -= 1
                        if coupled:
                            need[g, 3 * d + k] |= bool(fine(below)) != bool(fine(c))
    return need


CASES = {
    # (level-0 lattice, box of refined patches (x, y, z), domain faces)
    "one group": ((2, 2, 2), ((1, 2), (1, 2), (1, 2)), (0,) * 6),
    "periodic across x": ((2, 3, 3), ((0, 4), (2, 4), (2, 5)), (0,) * 6),
    "outflow corner": ((2, 3, 3), ((0, 2), (0, 3), (3, 6)), (1,) * 6),
    "L shape": ((3, 3, 2), None, (0, 0, 1, 1, 0, 0)),
    "whole groups": ((6, 6, 5), ((1, 11), (1, 11), (1, 9)), (1, 1, 0, 0, 1, 1)),
}


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("ghost", [2, 3])
def test_amr_advance_equals_fill_and_step(hydro, dtype, case, ghost):
    print("amr advance", dtype, case, ghost, flush=True)
    n0, box, bc = CASES[case]
    pos = boxes(n0, box or ((1, 5), (1, 5), (1, 3)))
    if box is None:   # take a corner out of the refined region
        pos[1] = pos[1][~((pos[1][:, 0] >= 3) & (pos[1][:, 1] >= 3))]
    g = torch.Generator(device="cuda").manual_seed(3)

    def states(G):
        r = lambda: torch.rand((G, 16, 16, 16), generator=g, device="cuda", dtype=torch.float64)
        rho, p, v = 0.5 + 1.5 * r(), 0.5 + 1.5 * r(), [0.6 * (r() - 0.5) for _ in range(3)]
        E = 1.5 * p + 0.5 * rho * sum(c * c for c in v)
        return torch.stack([rho] + [rho * c for c in v] + [E], 1).to(dtype).contiguous()

    U = [states(len(p)) for p in pos]
    s = hydro.AmrSolver(n0, pos, U, 1.0 / 64, 5.0 / 3.0, bc, ghost=ghost)
    lib, stream = hydro.load(), torch.cuda.current_stream().cuda_stream
    code = 0 if dtype == torch.float64 else 1
    new0 = states(len(pos[0]))
    for l, a in ((0, 0.0), (1, 0.0), (1, 0.5)):
        fine, coarse = s._lvl(l), None if l == 0 else s._lvl(0)
        cp = None if coarse is None else ctypes.byref(coarse)
        old = None if l == 0 else U[0].data_ptr()
        new = None if l == 0 else new0.data_ptr()
        G, P = len(pos[l]), 16 + 2 * ghost
        pad = torch.zeros((G, 5, P, P, P), dtype=dtype, device="cuda")
        ff = torch.zeros((G, 9, 5, 16, 16), dtype=dtype, device="cuda")
        n_bad = torch.zeros(2, dtype=torch.int32, device="cuda")
        count = 0
        assert lib.hydro_amr_fill_ghosts(ctypes.byref(fine), cp, old, new, a, s._bcarr, ghost, code, pad.data_ptr(),
                                         stream) == 0
        ref = hydro.advance_ext(pad, 1e-3, s.dx0 / 2 ** l, 5.0 / 3.0, 1, n_bad=n_bad[:1], face_flux=ff)
        for finer in ((None, s._lvl(1)) if l == 0 else (None,)):
            out = torch.zeros_like(ref)
            scratch = torch.full_like(pad, float("nan"))   # what is read of it must have been written
            got = torch.zeros_like(ff)
            assert lib.hydro_amr_advance(ctypes.byref(fine), cp, old, new, a, s._bcarr, ghost, code, 1e-3,
                                         s.dx0 / 2 ** l, 5.0 / 3.0, 1, 1.5, out.data_ptr(), scratch.data_ptr(),
                                         n_bad[1:].data_ptr(), got.data_ptr(),
                                         None if finer is None else ctypes.byref(finer), stream) == 0
            assert torch.equal(out, ref)
            # the planes that the flux registers read, and no others
            need = flux_planes(n0, pos, l, bc, finer is not None)
            assert need.any() == (l == 1 or finer is not None)
            need = torch.from_numpy(need).to("cuda")
            assert torch.equal(got[need], ff[need]) and not bool(got[~need].any())
            count += 1
        assert int(n_bad[1]) == count * int(n_bad[0])
