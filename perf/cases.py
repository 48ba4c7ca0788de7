"""Timed cases of the patch-group Euler solver: what a program that uses it has
it do, through its public entry points (paper_1712_07070_amd.hydro).

Kinds of cases
  padded   one step of padded groups: hydro.fill_ghosts, hydro.cfl_dt,
           hydro.advance (a caller that builds its own ghost zones, or small
           batches of groups handed over one call at a time)
  level    one step of a level read from level storage, with the CFL time-step
           of the new state reduced on the device: hydro.advance_level
  wcycle   one coarse step of independent levels in W-cycle order, one
           persistent launch per stage: hydro.MultiLevel.coarse_step
  ext      one step with another scheme word: hydro.fill_ghosts and
           hydro.advance_ext (with dual energy on ghost zones the caller
           filled, since fill_ghosts takes 5 fields)
  adjoint  the cotangent of a level's state through one step:
           hydro.advance_level_adjoint
  rollout  a differentiable rollout, forward and backward: hydro.Rollout
  amr      one coarse step of a coupled nested hierarchy: hydro.AmrSolver.step

Initial states are drawn on the device from the seed: white noise, a shear
layer, a turbulence-like state, a smooth wave with a noisy target, a blast on
nested levels.

exact() evaluates the same steps in plain torch in FP64 (Schive et al. 2018,
Sec. 2.2): whole arrays of padded groups at a time, textbook forms, autograd
for the derivatives.
"""

import math

import torch

from paper_1712_07070_amd import hydro

N = 16               # cells per group edge
THETA = 1.5          # generalized minmod
XI = 0.01            # dual-energy threshold
C_CFL = 0.5
DTYPES = {"f64": torch.float64, "f32": torch.float32}
LIMITERS = ("gminmod", "vanleer", "vanalbada", "hybrid")
SOLVERS = ("hllc", "roe", "hlle")

# Floating-point operations (add, multiply, divide, square root, one each) per
# cell update of a 16^3 group with its boundary faces: the default step from
# the repository's operation count, the others counted on this file's exact().
FLOPS_STEP = 907.7
FLOPS_EXT = {"plm": 950.0, "ppm": 1450.0, "ctu": 750.0, "char": 200.0, "roe": 300.0}   # the last three: on top
FLOPS_ADJOINT = 3.0 * FLOPS_STEP   # the step again and its reverse


def listed():
    return [
        # A handful of groups per call, as a host code hands them over: latency
        # and launches (the smoke check's size).
        {"name": "padded_f64_8_groups", "kind": "padded", "dtype": "f64", "ngx": 2, "ngy": 2, "ngz": 2, "bc": "periodic",
         "data": "noise", "ghost": 3},
        # A small level: fewer groups than compute units.
        {"name": "level_f64_64cube", "kind": "level", "dtype": "f64", "ngx": 4, "ngy": 4, "ngz": 4, "bc": "periodic",
         "data": "noise", "davis": False, "cfl": True},
        # An ordinary uniform-grid run in double precision (the benchmark's workload).
        {"name": "level_f64_256cube", "kind": "level", "dtype": "f64", "ngx": 16, "ngy": 16, "ngz": 16, "bc": "periodic",
         "data": "shear", "davis": False, "cfl": True},
        # The largest level: turbulence in single precision.
        {"name": "level_f32_384cube", "kind": "level", "dtype": "f32", "ngx": 24, "ngy": 24, "ngz": 24, "bc": "periodic",
         "data": "turbulence", "davis": False, "cfl": True},
        # The W-cycle of levels with odd group counts, launched stage by stage.
        {"name": "wcycle_f64_125_343_1000", "kind": "wcycle", "dtype": "f64", "levels": 3, "n0": 5, "n1": 7, "n2": 10},
        # Sharper reconstruction at ordinary size: characteristic PLM, van Leer.
        {"name": "ext_f64_char_vanleer_256cube", "kind": "ext", "dtype": "f64", "ngx": 16, "ngy": 16, "ngz": 16,
         "bc": "periodic", "data": "shear", "ghost": 3, "ctu": False, "ppm": False, "char": True, "limiter": "vanleer",
         "solver": "hllc", "davis": False, "dual": False},
        # The scheme of the paper's galaxy runs: MHM, PPM, hybrid limiter, HLLC.
        {"name": "ext_f64_ppm_hybrid_256cube", "kind": "ext", "dtype": "f64", "ngx": 16, "ngy": 16, "ngz": 16,
         "bc": "periodic", "data": "shear", "ghost": 3, "ctu": False, "ppm": True, "char": False, "limiter": "hybrid",
         "solver": "hllc", "davis": False, "dual": False},
        # The most expensive integrator: CTU with Roe's solver.
        {"name": "ext_f64_ctu_roe_256cube", "kind": "ext", "dtype": "f64", "ngx": 16, "ngy": 16, "ngz": 16,
         "bc": "periodic", "data": "shear", "ghost": 3, "ctu": True, "ppm": False, "char": False, "limiter": "gminmod",
         "solver": "roe", "davis": False, "dual": False},
        # Single precision, dual energy, an odd number of groups, outflow.
        {"name": "ext_f32_ppm_dual_210_groups", "kind": "ext", "dtype": "f32", "ngx": 6, "ngy": 5, "ngz": 7,
         "bc": "outflow", "data": "turbulence", "ghost": 3, "ctu": False, "ppm": True, "char": True,
         "limiter": "vanalbada", "solver": "hlle", "davis": False, "dual": True},
        # One reverse step of a large single-precision level.
        {"name": "adjoint_f32_192cube", "kind": "adjoint", "dtype": "f32", "ngx": 12, "ngy": 12, "ngz": 12,
         "bc": "periodic", "data": "turbulence"},
        # Fitting an initial state to a target density through 8 steps.
        {"name": "rollout_f64_128cube", "kind": "rollout", "dtype": "f64", "ngx": 8, "ngy": 8, "ngz": 8,
         "bc": "periodic", "data": "wave", "steps": 8, "every": 4},
        # A coupled three-level hierarchy (512 / 1536 / 3072 groups) around a blast.
        {"name": "amr_f64_512_1536_3072", "kind": "amr", "dtype": "f64", "levels": 3, "n0x": 8, "n0y": 8, "n0z": 8,
         "m1y": 2, "m1z": 4, "m2x": 4, "m2y": 8, "m2z": 12},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _lattice(rng, most):
    """Three edge lengths, each odd as often as even, with at most `most` groups."""
    target = math.exp(rng.uniform(0.0, math.log(most)))
    edge = target ** (1.0 / 3.0)
    n = [max(1, int(round(edge * math.exp(rng.uniform(-0.5, 0.5))))) for _ in range(3)]
    while n[0] * n[1] * n[2] > most:
        n[n.index(max(n))] -= 1
    return {"ngx": n[0], "ngy": n[1], "ngz": n[2]}


def draw(rng):
    kind = rng.choice(["padded", "level", "level", "wcycle", "ext", "ext", "ext", "adjoint", "rollout", "amr"])
    c = {"kind": kind, "dtype": rng.choice(["f64", "f32"])}
    if kind == "wcycle":
        c["levels"] = rng.choice([2, 3])
        c["n0"], c["n1"], c["n2"] = _log_int(rng, 2, 8), _log_int(rng, 3, 10), _log_int(rng, 4, 12)
        return c
    if kind == "amr":
        c["levels"] = rng.choice([2, 3])
        lo = 5 if c["levels"] == 3 else 3
        c["n0x"], c["n0y"], c["n0z"] = rng.randint(lo, 6), rng.randint(lo, 6), rng.randint(lo, 6)
        c.update(m1y=2, m1z=2, m2x=4, m2y=8, m2z=8)
        return c
    most = {"padded": 1024, "level": 4096, "ext": 2048, "adjoint": 1728, "rollout": 343}[kind]
    c.update(_lattice(rng, most))
    c["bc"] = rng.choice(["periodic", "outflow", "mixed"])
    c["data"] = rng.choice(["noise", "shear", "turbulence"])
    if kind == "padded":
        c["ghost"] = rng.choice([2, 3])
    elif kind == "level":
        c["davis"], c["cfl"] = rng.random() < 0.25, rng.random() < 0.75
    elif kind == "ext":
        c["ctu"], c["ppm"] = rng.random() < 0.3, rng.random() < 0.5
        c["char"], c["davis"], c["dual"] = rng.random() < 0.4, rng.random() < 0.2, rng.random() < 0.2
        c["limiter"], c["solver"] = rng.choice(LIMITERS), rng.choice(SOLVERS)
        c["ghost"] = 3 if c["ppm"] else rng.choice([2, 3])
    elif kind == "rollout":
        c["data"], c["steps"], c["every"] = "wave", rng.randint(2, 8), rng.choice([1, 4])
    return c


# ------------------------------------------------------------------ inputs --

def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _gen(seed):
    return torch.Generator(device=_device()).manual_seed(int(seed))


def _gamma(case):
    return 1.4 if case.get("data") == "shear" else 5.0 / 3.0


def _bc(case):
    return {"periodic": (0,) * 6, "outflow": (1,) * 6, "mixed": (0, 0, 1, 1, 0, 0)}[case.get("bc", "periodic")]


def _ng(case):
    return case["ngx"], case["ngy"], case["ngz"]


def _dx(ng):
    return 1.0 / (N * max(ng))


def _conserved(rho, v, p, gamma):
    return torch.stack([rho, rho * v[0], rho * v[1], rho * v[2],
                        p / (gamma - 1.0) + 0.5 * rho * (v[0] * v[0] + v[1] * v[1] + v[2] * v[2])])


def _to_groups(grid, ng):
    """[f, Nz, Ny, Nx] -> level storage [G, f, 16, 16, 16]."""
    f = grid.shape[0]
    b = grid.reshape(f, ng[2], N, ng[1], N, ng[0], N).permute(1, 3, 5, 0, 2, 4, 6)
    return b.reshape(-1, f, N, N, N).contiguous()


def _random_field(g, shape, slope):
    """Periodic Gaussian random field with |f(k)|^2 ~ k^slope, zero mean, unit variance."""
    fk = torch.fft.rfftn(torch.randn(shape, generator=g, device=_device(), dtype=torch.float64))
    k = [torch.fft.fftfreq(n, device=_device(), dtype=torch.float64) * n for n in shape[:2]]
    kx = torch.fft.rfftfreq(shape[2], device=_device(), dtype=torch.float64) * shape[2]
    kk = (k[0][:, None, None] ** 2 + k[1][None, :, None] ** 2 + kx[None, None, :] ** 2).sqrt()
    kk[0, 0, 0] = 1.0
    amp = kk ** (0.5 * slope)
    amp[0, 0, 0] = 0.0
    f = torch.fft.irfftn(fk * amp, s=shape)
    f = f - f.mean()
    return f / f.std()


def _grid_state(kind, ng, seed):
    """Initial (rho, v, p) of a brick of ng groups as level storage, FP64."""
    g, dev = _gen(seed), _device()
    shape = tuple(N * n for n in reversed(ng))
    dx = _dx(ng)

    def uniform(lo, hi):
        return lo + (hi - lo) * torch.rand(shape, generator=g, device=dev, dtype=torch.float64)

    def normal(sigma):
        return sigma * torch.randn(shape, generator=g, device=dev, dtype=torch.float64)

    z, y, x = torch.meshgrid(*[(torch.arange(n, device=dev, dtype=torch.float64) + 0.5) * dx for n in shape],
                             indexing="ij")
    ly = shape[1] * dx
    if kind == "noise":
        rho, v, p = uniform(0.5, 2.0), [normal(0.3) for _ in range(3)], uniform(0.5, 2.0)
    elif kind == "shear":
        inner = (y - 0.5 * ly).abs() < 0.25 * ly
        rho = torch.where(inner, 1.0, 2.0).to(torch.float64)
        v = [torch.where(inner, -0.5, 0.5).to(torch.float64),
             0.01 * torch.sin(4.0 * math.pi * x) + normal(1e-3), torch.zeros_like(x)]
        p = torch.full_like(x, 2.5)
    elif kind == "turbulence":
        # rms Mach 3 and unit variance of ln(rho) on 384 cells; weaker on a
        # coarser grid, which does not resolve as strong gradients
        k = min(1.0, math.sqrt(min(shape) / 384.0))
        rho = torch.exp(k * _random_field(g, shape, -4.0) - 0.5)
        v = [_random_field(g, shape, -4.0) for _ in range(3)]
        rms = (v[0] ** 2 + v[1] ** 2 + v[2] ** 2).mean().sqrt()
        v = [c * (3.0 * k / rms) for c in v]
        p = rho / (5.0 / 3.0)
    else:  # a smooth wave in every field, phases from the seed
        ph = (2.0 * math.pi * torch.rand(5, generator=g, device=dev, dtype=torch.float64)).tolist()
        t = 2.0 * math.pi
        lz, lx = shape[0] * dx, shape[2] * dx
        x, y, z = x / lx, y / ly, z / lz
        rho = 1.0 + 0.01 * torch.sin(t * (x + y + z) + ph[0])
        v = [0.1 + 0.01 * torch.sin(t * (x + 2 * y + z) + ph[1]), 0.05 + 0.01 * torch.cos(t * (2 * x - y + z) + ph[2]),
             0.01 * torch.sin(t * (x + y - 2 * z) + ph[3])]
        p = 1.0 + 0.01 * torch.cos(t * (x + y - z) + ph[4])
    gamma = 1.4 if kind == "shear" else 5.0 / 3.0
    return _to_groups(_conserved(rho, v, p, gamma), ng)


def _cfl(U, dx, gamma):
    """Per-patch time-steps [G, 8] of level storage (Sec. 2.6, Eq. 2)."""
    U = U.double()
    v = U[:, 1:4] / U[:, 0:1]
    p = (gamma - 1.0) * (U[:, 4] - 0.5 * (U[:, 1:4] * v).sum(1))
    s = v.abs().sum(1) + 3.0 * torch.sqrt(gamma * p / U[:, 0])
    s = s.reshape(-1, 2, 8, 2, 8, 2, 8).amax(dim=(2, 4, 6)).reshape(-1, 8)
    return C_CFL * dx / s


def _chunks(total, size):
    return [(a, min(a + size, total)) for a in range(0, total, size)]


def _level_dt(U, dx, gamma):
    return min(float(_cfl(U[a:b], dx, gamma).min()) for a, b in _chunks(U.shape[0], 2048))


def _boxes(case):
    """Half-open boxes of refined patches (patch indices of the coarser level), x, y, z."""
    nx, ny, nz = case["n0x"], case["n0y"], case["n0z"]
    out = [((0, 2 * nx), (case["m1y"], 2 * ny - case["m1y"]), (case["m1z"], 2 * nz - case["m1z"]))]
    if case["levels"] == 3:
        out.append(((case["m2x"], 4 * nx - case["m2x"]), (case["m2y"], 4 * ny - case["m2y"]),
                    (case["m2z"], 4 * nz - case["m2z"])))
    return out


def _amr_state(case, seed):
    """Group positions (host lists) and states of a nested hierarchy: a blast
    at the centre of a smoothly varying flow, coarse cells under finer groups
    the mean of their children."""
    n0 = (case["n0x"], case["n0y"], case["n0z"])
    dx0, gamma, dev = _dx(n0), 5.0 / 3.0, _device()
    g = _gen(seed)
    ph = (2.0 * math.pi * torch.rand(5, generator=g, device=dev, dtype=torch.float64)).tolist()
    pos = [[(x, y, z) for z in range(n0[2]) for y in range(n0[1]) for x in range(n0[0])]]
    for bx, by, bz in _boxes(case):
        pos.append([(x, y, z) for z in range(*bz) for y in range(*by) for x in range(*bx)])
    size = [N * n * dx0 for n in n0]
    states = []
    for l, p in enumerate(pos):
        dx = dx0 / 2 ** l
        q = torch.tensor(p, device=dev, dtype=torch.float64)
        i = torch.arange(N, device=dev, dtype=torch.float64) + 0.5
        shape = (len(p), N, N, N)
        x = ((N * q[:, 0, None, None, None] + i[None, None, None, :]) * dx / size[0]).expand(shape)
        y = ((N * q[:, 1, None, None, None] + i[None, None, :, None]) * dx / size[1]).expand(shape)
        z = ((N * q[:, 2, None, None, None] + i[None, :, None, None]) * dx / size[2]).expand(shape)
        t = 2.0 * math.pi
        r2 = ((x - 0.5) * size[0]) ** 2 + ((y - 0.5) * size[1]) ** 2 + ((z - 0.5) * size[2]) ** 2
        rho = 1.0 + 0.2 * torch.sin(t * (x + y + z) + ph[0])
        v = [0.1 * torch.sin(t * (x + 2 * y + z) + ph[1]), 0.1 * torch.cos(t * (2 * x - y + z) + ph[2]),
             0.1 * torch.sin(t * (x + y - 2 * z) + ph[3])]
        pr = 1.0 + 0.1 * torch.cos(t * (x + y - z) + ph[4]) + 20.0 * torch.exp(-r2 / (2.0 * (2.0 * dx0) ** 2))
        U = _conserved(rho, v, pr, gamma).transpose(0, 1).contiguous().to(DTYPES[case["dtype"]])
        states.append(U)
    for l in range(len(pos) - 1, 0, -1):
        _restrict(states[l], states[l - 1], pos[l], pos[l - 1])
    return n0, dx0, gamma, pos, states


def _children_mean(U):
    return U.reshape(-1, 5, 8, 2, 8, 2, 8, 2).mean(dim=(3, 5, 7))


def _restrict(fine, coarse, pf, pc):
    """Coarse cells covered by fine groups become the mean of their children."""
    index = {p: i for i, p in enumerate(pc)}
    parent = torch.tensor([index[(x >> 1, y >> 1, z >> 1)] for x, y, z in pf], device=fine.device)
    half = torch.tensor([((z & 1) * 2 + (y & 1)) * 2 + (x & 1) for x, y, z in pf], device=fine.device)
    view = coarse.reshape(-1, 5, 2, 8, 2, 8, 2, 8).permute(0, 2, 4, 6, 1, 3, 5, 7)
    view[parent, half >> 2, (half >> 1) & 1, half & 1] = _children_mean(fine)


def _amr_dt(states, dx0, gamma):
    return 0.6 * min(_level_dt(U, dx0 / 2 ** l, gamma) * 2 ** l for l, U in enumerate(states))


def _wcycle_levels(case):
    """(lattice, dx) of each level."""
    out = []
    for l in range(case["levels"]):
        n = case["n%d" % l]
        out.append(((n, n, n), 1.0 / (N * case["n0"]) / 2 ** l))
    return out


def _wcycle_states(case, seed):
    dt = DTYPES[case["dtype"]]
    return [_grid_state("wave", ng, seed * 8 + l).to(dt) for l, (ng, _) in enumerate(_wcycle_levels(case))]


def _wcycle_dt(case, states):
    return 0.6 * min(_level_dt(U, dx, 5.0 / 3.0) * 2 ** l
                     for l, (U, (_, dx)) in enumerate(zip(states, _wcycle_levels(case))))


def _with_entropy(U, gamma):
    p = (gamma - 1.0) * (U[:, 4] - 0.5 * (U[:, 1:4] ** 2).sum(1) / U[:, 0])
    return torch.cat([U, (p / U[:, 0] ** (gamma - 1.0))[:, None]], dim=1)


def _word(case):
    w = hydro.SCHEME_CTU if case.get("ctu") else hydro.SCHEME_MHM
    w |= (0, hydro.LIMITER_VANLEER, hydro.LIMITER_VANALBADA, hydro.LIMITER_HYBRID)[LIMITERS.index(case.get("limiter", "gminmod"))]
    w |= (0, hydro.RIEMANN_ROE, hydro.RIEMANN_HLLE)[SOLVERS.index(case.get("solver", "hllc"))]
    w |= hydro.CHARACTERISTIC if case.get("char") else 0
    w |= hydro.PPM if case.get("ppm") else 0
    w |= hydro.DUAL_ENERGY if case.get("dual") else 0
    return w | (hydro.WAVESPEED_DAVIS if case.get("davis") else 0)


def _input(case, seed):
    """A level's state of the case's type, and what goes with it."""
    ng, bc = _ng(case), _bc(case)
    U = _grid_state(case["data"], ng, seed).to(DTYPES[case["dtype"]])
    return U, ng, bc, _dx(ng), _gamma(case)


def _cotangent(case, U, seed):
    g = _gen(seed + 1000003)
    return torch.randn(U.shape, generator=g, device=U.device, dtype=torch.float64).to(U.dtype)


def prepare(case, seed):
    kind = case["kind"]
    s = {"kind": kind}
    if kind == "amr":
        n0, dx0, gamma, pos, states = _amr_state(case, seed)
        s["dt0"] = _amr_dt(states, dx0, gamma)
        s["solver"] = hydro.AmrSolver(n0, pos, states, dx0, gamma)
        return s
    if kind == "wcycle":
        states = _wcycle_states(case, seed)
        s["ml"] = hydro.MultiLevel([(ng, dx, (0,) * 6) for ng, dx in _wcycle_levels(case)], 5.0 / 3.0,
                                   _wcycle_dt(case, states), dtype=states[0].dtype)
        for l, U in enumerate(states):
            s["ml"].load_state(l, U)
        return s
    U, ng, bc, dx, gamma = _input(case, seed)
    dt = _level_dt(U, dx, gamma)
    s.update(U=U, ng=ng, bc=bc, dx=dx, gamma=gamma, dt=dt, word=_word(case))
    dev, G = U.device, U.shape[0]
    s["n_bad"] = torch.zeros(1, dtype=torch.int32, device=dev)
    if kind in ("level", "padded"):
        s["dts"] = torch.full((3,), float("inf"), dtype=torch.float64, device=dev)
        s["dts"][0] = dt
        s["out"] = torch.empty_like(U)
        s["cfl"] = case.get("cfl", True)
    if kind in ("padded", "ext"):
        s["ghost"] = case["ghost"]
        P = N + 2 * case["ghost"]
        s["pad"] = torch.empty((G, 5, P, P, P), dtype=U.dtype, device=dev)
        s["dt_patch"] = torch.empty((G, 8), dtype=torch.float64, device=dev)
    if kind == "ext":
        s["dual"] = case["dual"]
        s["work"] = hydro.ext_workspace(G, case["ghost"], U.dtype, s["word"], dev)
        if case["dual"]:
            U6 = _with_entropy(U, gamma)
            s["pad"] = torch.cat([hydro.fill_ghosts(U, ng, case["ghost"], bc),
                                  hydro.fill_ghosts(U6[:, 1:].contiguous(), ng, case["ghost"], bc)[:, 4:]], dim=1)
        s["out"] = torch.empty((G, 6 if case["dual"] else 5, N, N, N), dtype=U.dtype, device=dev)
    if kind == "adjoint":
        s["g"] = _cotangent(case, U, seed)
        s["out"] = torch.empty_like(U)
        s["work"] = hydro.adjoint_workspace(G, U.dtype, True, dev)
    if kind == "rollout":
        s.update(steps=case["steps"], every=case["every"], dt=0.2 * dx)
        s["target"] = _target(case, U, seed)
        s["U"] = U.requires_grad_(True)
    return s


def _target(case, U, seed):
    """The density to fit: the initial one with noise of one percent."""
    return U[:, 0] + 0.01 * _cotangent(case, U[:, 0], seed)


def run(s):
    kind = s["kind"]
    if kind == "amr":
        s["solver"].step(s["dt0"])
        return {"U": s["solver"].U, "n_bad": s["solver"].n_bad}
    if kind == "wcycle":
        s["ml"].coarse_step()
        return {"U": [s["ml"].state(l) for l in range(s["ml"].L)], "n_bad": s["ml"].n_bad}
    if kind == "padded":
        hydro.fill_ghosts(s["U"], s["ng"], s["ghost"], s["bc"], out=s["pad"])
        hydro.cfl_dt(s["pad"], s["dx"], s["gamma"], C_CFL, out=s["dt_patch"], dt_min=s["dts"][1:2])
        hydro.advance(s["pad"], 1.0, s["dx"], s["gamma"], THETA, s["word"], out=s["out"], n_bad=s["n_bad"],
                      dt_dev=s["dts"][1:2])
        return {"U": s["out"], "dt_patch": s["dt_patch"], "n_bad": s["n_bad"]}
    if kind == "level":
        if s["cfl"]:
            hydro.advance_level(s["U"], s["ng"], s["bc"], 1.0, s["dx"], s["gamma"], THETA, s["word"], out=s["out"],
                                n_bad=s["n_bad"], dt_dev=s["dts"][0:1], c_cfl=C_CFL, dt_next=s["dts"][1:2],
                                dt_reset=s["dts"][2:3])
            return {"U": s["out"], "dt": s["dts"][1:2], "n_bad": s["n_bad"]}
        hydro.advance_level(s["U"], s["ng"], s["bc"], s["dt"], s["dx"], s["gamma"], THETA, s["word"], out=s["out"],
                            n_bad=s["n_bad"])
        return {"U": s["out"], "n_bad": s["n_bad"]}
    if kind == "ext":
        if not s["dual"]:
            hydro.fill_ghosts(s["U"], s["ng"], s["ghost"], s["bc"], out=s["pad"])
        hydro.advance_ext(s["pad"], s["dt"], s["dx"], s["gamma"], s["word"], THETA, out=s["out"], n_bad=s["n_bad"],
                          work=s["work"], xi=XI)
        return {"U": s["out"], "n_bad": s["n_bad"]}
    if kind == "adjoint":
        return hydro.advance_level_adjoint(s["U"], s["g"], s["ng"], s["bc"], s["dt"], s["dx"], s["gamma"], THETA,
                                           s["word"], out=s["out"], work=s["work"])
    UN = hydro.Rollout.apply(s["U"], s["ng"], s["bc"], s["steps"], s["dt"], s["dx"], s["gamma"], s["every"], THETA,
                             s["word"])
    loss = ((UN[:, 0] - s["target"]) ** 2).sum()
    grad, = torch.autograd.grad(loss, s["U"])
    return {"U": UN.detach(), "grad": grad}


def work(case):
    kind, size = case["kind"], 8 if case["dtype"] == "f64" else 4
    state = 5 * N ** 3 * size                     # bytes of a group's state
    if kind == "amr":
        G = [case["n0x"] * case["n0y"] * case["n0z"]]
        G += [(bx[1] - bx[0]) * (by[1] - by[0]) * (bz[1] - bz[0]) for bx, by, bz in _boxes(case)]
        return {"bytes": 2.0 * state * sum(G), "flops": FLOPS_STEP * N ** 3 * sum(g * 2 ** l for l, g in enumerate(G))}
    if kind == "wcycle":
        G = [ng[0] ** 3 for ng, _ in _wcycle_levels(case)]
        return {"bytes": 2.0 * state * sum(G), "flops": FLOPS_STEP * N ** 3 * sum(g * 2 ** l for l, g in enumerate(G))}
    G = case["ngx"] * case["ngy"] * case["ngz"]
    cells = float(G * N ** 3)
    if kind in ("padded", "level"):
        return {"bytes": 2.0 * state * G, "flops": FLOPS_STEP * cells}
    if kind == "ext":
        f = FLOPS_EXT["ppm"] if case["ppm"] else FLOPS_EXT["plm"]
        f += sum(FLOPS_EXT[k] for k, on in (("ctu", case["ctu"]), ("char", case["char"]),
                                            ("roe", case["solver"] == "roe")) if on)
        if case["dual"]:   # reads the ghost zones its stencil reaches
            P = N + (6 if case["ppm"] else 4)
            return {"bytes": 6.0 * size * G * (P ** 3 + N ** 3), "flops": 1.2 * f * cells}
        return {"bytes": 2.0 * state * G, "flops": f * cells}
    if kind == "adjoint":
        return {"bytes": 3.0 * state * G, "flops": FLOPS_ADJOINT * cells}
    return {"bytes": 3.2 * state * G, "flops": case["steps"] * (FLOPS_STEP + FLOPS_ADJOINT) * cells}


# ------------------------------------------- the steps in plain torch, FP64 --
# Arrays are [groups, fields, z, y, x]; axis d of space is dimension 4 - d.

def _cut(A, d, lo, hi):
    return A.narrow(4 - d, lo, hi - lo)


def _box(A, margins):
    """A without `margins[d]` cells on both sides of each axis."""
    for d, m in enumerate(margins):
        if m:
            A = _cut(A, d, m, A.shape[4 - d] - m)
    return A


def _primitive(U, gamma):
    v = U[:, 1:4] / U[:, 0:1]
    p = (gamma - 1.0) * (U[:, 4:5] - 0.5 * (U[:, 1:4] * v).sum(1, keepdim=True))
    return torch.cat([U[:, 0:1], v, p] + ([U[:, 5:6] / U[:, 0:1]] if U.shape[1] == 6 else []), 1)


def _limited(dm, dp, dc, limiter):
    same = dm * dp > 0
    one = torch.ones_like(dm)
    if limiter == "vanalbada":
        return torch.where(same, dm * dp * (dm + dp) / torch.where(same, dm * dm + dp * dp, one), 0.0)
    harmonic = 2.0 * dm * dp / torch.where(same, dm + dp, one)
    if limiter == "vanleer":
        return torch.where(same, harmonic, 0.0)
    m = torch.minimum(torch.minimum(THETA * dm.abs(), dc.abs()), THETA * dp.abs())
    if limiter == "hybrid":
        m = torch.minimum(m, harmonic.abs())
    return torch.where(same, m * torch.sign(dc), 0.0)


def _slopes(Wm, Wc, Wp, d, gamma, case):
    """Limited slopes of the cells Wc along axis d."""
    dm, dp = Wc - Wm, Wp - Wc
    lim = case.get("limiter", "gminmod")
    if not case.get("char"):
        return _limited(dm, dp, 0.5 * (Wp - Wm), lim)
    n, t1, t2 = 1 + d, 1 + (d + 1) % 3, 1 + (d + 2) % 3
    rho = Wc[:, 0]
    c = torch.sqrt(gamma * Wc[:, 4] / rho)

    def project(q):
        a = [0.5 * (q[:, 4] / c ** 2 - rho / c * q[:, n]), q[:, 0] - q[:, 4] / c ** 2, q[:, t1], q[:, t2],
             0.5 * (q[:, 4] / c ** 2 + rho / c * q[:, n])]
        return torch.stack(a + ([q[:, 5]] if q.shape[1] == 6 else []), 1)

    am, ap = project(dm), project(dp)
    a = _limited(am, ap, 0.5 * (am + ap), lim)
    s = [None] * Wc.shape[1]
    s[0] = a[:, 0] + a[:, 1] + a[:, 4]
    s[n], s[t1], s[t2] = c / rho * (a[:, 4] - a[:, 0]), a[:, 2], a[:, 3]
    s[4] = c * c * (a[:, 0] + a[:, 4])
    if len(s) == 6:
        s[5] = a[:, 5]
    return torch.stack(s, 1)


def _face_values(W, d, R, gamma, case):
    """Values on the low and the high face along axis d of the cells that lie
    R + 1... inside the block W (R cells of margin on every axis)."""
    others = [R if e != d else 0 for e in range(3)]
    V = _box(W, others)
    n = V.shape[4 - d] - 2 * R

    def at(o):
        return _cut(V, d, R + o, R + o + n)

    if not case.get("ppm"):
        s = _slopes(at(-1), at(0), at(1), d, gamma, case)
        return at(0) - 0.5 * s, at(0) + 0.5 * s
    sl = _slopes(_cut(V, d, 0, n + 2), _cut(V, d, 1, n + 3), _cut(V, d, 2, n + 4), d, gamma, case)
    sm, s0, sp = (_cut(sl, d, j, j + n) for j in range(3))
    q = at(0)
    qL = 0.5 * (at(-1) + q) - (s0 - sm) / 6.0
    qR = 0.5 * (q + at(1)) - (sp - s0) / 6.0
    flat = (qR - q) * (q - qL) <= 0
    dq, q6 = qR - qL, 6.0 * (q - 0.5 * (qL + qR))
    low, high = dq * q6 > dq * dq, -(dq * dq) > dq * q6
    lo = torch.where(flat, q, torch.where(low, 3.0 * q - 2.0 * qR, qL))
    hi = torch.where(flat, q, torch.where(high & ~low, 3.0 * q - 2.0 * qL, qR))
    return lo, hi


def _cons_flux(W, d, gamma):
    """Conserved state and physical flux along d of a primitive state."""
    rho, v, p, un = W[:, 0:1], W[:, 1:4], W[:, 4:5], W[:, 1 + d:2 + d]
    E = p / (gamma - 1.0) + 0.5 * rho * (v * v).sum(1, keepdim=True)
    U = torch.cat([rho, rho * v, E] + ([rho * W[:, 5:6]] if W.shape[1] == 6 else []), 1)
    return U, _flux(U, un, p, d)


def _flux(U, un, p, d):
    F = list((U * un).split(1, 1))
    F[1 + d] = F[1 + d] + p
    F[4] = F[4] + p * un
    return torch.cat(F, 1)


def _riemann(L, R, d, gamma, case):
    """Flux through faces normal to d between the conserved states L and R."""
    WL, WR = _primitive(L, gamma), _primitive(R, gamma)
    rL, rR, pL, pR = L[:, 0:1], R[:, 0:1], WL[:, 4:5], WR[:, 4:5]
    n = 1 + d
    uL, uR = WL[:, n:n + 1], WR[:, n:n + 1]
    cL, cR = torch.sqrt(gamma * pL / rL), torch.sqrt(gamma * pR / rR)
    FL, FR = _flux(L, uL, pL, d), _flux(R, uR, pR, d)
    wL, wR = torch.sqrt(rL), torch.sqrt(rR)
    va = (wL * WL[:, 1:4] + wR * WR[:, 1:4]) / (wL + wR)
    ua = va[:, d:d + 1]
    Ha = (wL * (L[:, 4:5] + pL) / rL + wR * (R[:, 4:5] + pR) / rR) / (wL + wR)
    q2 = (va * va).sum(1, keepdim=True)
    a2 = (gamma - 1.0) * (Ha - 0.5 * q2)
    if case.get("davis"):
        SL, SR = torch.minimum(uL - cL, uR - cR), torch.maximum(uL + cL, uR + cR)
    else:
        SL, SR = torch.minimum(uL - cL, ua - a2.sqrt()), torch.maximum(uR + cR, ua + a2.sqrt())
    solver = case.get("solver", "hllc")
    if solver == "hlle":
        F = torch.where(SL >= 0, FL, torch.where(SR <= 0, FR, (SR * FL - SL * FR + SL * SR * (R - L)) / (SR - SL)))
    else:
        Ss = (pR - pL + rL * uL * (SL - uL) - rR * uR * (SR - uR)) / (rL * (SL - uL) - rR * (SR - uR))

        def star(U, W, u, p, S, F):
            k = U[:, 0:1] * (S - u) / (S - Ss)
            v = list(W[:, 1:4].split(1, 1))
            v[d] = Ss
            e = U[:, 4:5] / U[:, 0:1] + (Ss - u) * (Ss + p / (U[:, 0:1] * (S - u)))
            Us = torch.cat([k] + [k * c for c in v] + [k * e] + ([U[:, 5:6]] if U.shape[1] == 6 else []), 1)
            return F + S * (Us - U)

        F = torch.where(SL >= 0, FL, torch.where(Ss >= 0, star(L, WL, uL, pL, SL, FL),
                                                 torch.where(SR > 0, star(R, WR, uR, pR, SR, FR), FR)))
    if solver == "roe":
        a = a2.clamp_min(0).sqrt()
        D = R - L
        d0, dn = D[:, 0:1], D[:, n:n + 1]
        t = [1 + (d + 1) % 3, 1 + (d + 2) % 3]
        sh = [D[:, i:i + 1] - va[:, i - 1:i] * d0 for i in t]
        al2 = (gamma - 1.0) / a2 * (d0 * (Ha - ua * ua) + ua * dn
                                    - (D[:, 4:5] - sh[0] * va[:, t[0] - 1:t[0]] - sh[1] * va[:, t[1] - 1:t[1]]))
        al1 = (d0 * (ua + a) - dn - a * al2) / (2.0 * a)
        al5 = d0 - al1 - al2

        def wave(un, e):
            K = [torch.ones_like(ua)] + list(va.split(1, 1)) + [e]
            K[n] = un
            return torch.cat(K, 1)

        K1, K2, K5 = wave(ua - a, Ha - ua * a), wave(ua, 0.5 * q2), wave(ua + a, Ha + ua * a)
        M = list((al2 * K2).split(1, 1))
        for i, s in zip(t, sh):
            M[i] = M[i] + s
            M[4] = M[4] + s * va[:, i - 1:i]
        M = torch.cat(M, 1)
        S1 = L[:, :5] + al1 * K1
        S2 = S1 + M
        ok = a2 > 0
        for S in (S1, S2):
            ok = ok & (S[:, 0:1] > 0) & (_primitive(S, gamma)[:, 4:5] > 0)
        Fr = 0.5 * (FL + FR)[:, :5] - 0.5 * ((ua - a).abs() * al1 * K1 + ua.abs() * M + (ua + a).abs() * al5 * K5)
        F = torch.cat([torch.where(ok, Fr, F[:, :5]), F[:, 5:]], 1)
    if F.shape[1] == 6:
        m = F[:, 0:1]
        F = torch.cat([F[:, :5], m * torch.where(m >= 0, WL[:, 5:6], WR[:, 5:6])], 1)
    return F


def _exact_step(U, gh, dt, dx, gamma, case):
    """One step of padded groups [n, f, P, P, P] in FP64: the new interiors
    and the three axes' interior fluxes."""
    R = 2 if case.get("ppm") else 1
    m = gh - 1 - R
    U = _box(U, (m, m, m))
    W = _primitive(U, gamma)
    lam = dt / dx
    sides, dF = [], []
    for d in range(3):
        lo, hi = _face_values(W, d, R, gamma, case)
        (Ul, Fl), (Uh, Fh) = _cons_flux(lo, d, gamma), _cons_flux(hi, d, gamma)
        sides.append((Ul, Uh))
        dF.append(Fl - Fh)
    if not case.get("ctu"):
        s = dF[0] + dF[1] + dF[2]
        dF = [s, s, s]
    sides = [(a + 0.5 * lam * f, b + 0.5 * lam * f) for (a, b), f in zip(sides, dF)]   # cells -1 .. 16

    def solve(d, lo, hi):
        n = lo.shape[4 - d]
        return _riemann(_cut(hi, d, 0, n - 1), _cut(lo, d, 1, n), d, gamma, case)

    if case.get("ctu"):
        first = [solve(d, *sides[d]) for d in range(3)]
        diff = [_cut(f, d, 1, 17) - _cut(f, d, 0, 16) for d, f in enumerate(first)]    # cells 0 .. 15 along d
        new = []
        for d in range(3):
            corr = 0.0
            for e in range(3):
                if e != d:
                    corr = corr + _box(diff[e], [1 if k not in (d, e) else 0 for k in range(3)])
            cells = [0 if k == d else 1 for k in range(3)]
            new.append(tuple(_box(S, cells) - 0.5 * lam * corr for S in sides[d]))
        sides = new
    else:
        sides = [tuple(_box(S, [0 if k == d else 1 for k in range(3)]) for S in sides[d]) for d in range(3)]
    flux = [solve(d, *sides[d]) for d in range(3)]
    out = _box(U, (1 + R,) * 3)
    div = 0.0
    for d, f in enumerate(flux):
        div = div + (_cut(f, d, 1, 17) - _cut(f, d, 0, 16))
    out = out - lam * div
    if out.shape[1] == 6:
        ekin = 0.5 * (out[:, 1:4] ** 2).sum(1) / out[:, 0]
        eth, rg = out[:, 4] - ekin, out[:, 0] ** (gamma - 1.0)
        low = eth < XI * ekin
        E = torch.where(low, out[:, 5] * rg / (gamma - 1.0) + ekin, out[:, 4])
        s = torch.where(low, out[:, 5], (gamma - 1.0) * eth / rg)
        out = torch.cat([out[:, :4], E[:, None], s[:, None]], 1)
    return out, flux


def _axis_map(n, lo, hi, i):
    """Source cells of the cell coordinates i on an axis of n cells."""
    below = (i % n) if lo == 0 else i.clamp_min(0)
    above = (i % n) if hi == 0 else i.clamp_max(n - 1)
    return torch.where(i < 0, below, torch.where(i >= n, above, i))


def _pad_index(ng, bc, gh, a, b):
    """Offsets [b - a, P, P, P] into one field of level storage (its groups
    5 * 4096 elements apart) of the padded groups a .. b - 1."""
    g = torch.arange(a, b, device=_device())
    i = torch.arange(N + 2 * gh, device=_device()) - gh
    at = [g % ng[0], (g // ng[0]) % ng[1], g // (ng[0] * ng[1])]
    x, y, z = (_axis_map(N * ng[d], bc[2 * d], bc[2 * d + 1], N * q[:, None] + i) for d, q in enumerate(at))
    x, y, z = x[:, None, None, :], y[:, None, :, None], z[:, :, None, None]
    group = ((z // N) * ng[1] + y // N) * ng[0] + x // N
    return group * (5 * N ** 3) + ((z % N) * N + y % N) * N + x % N


def _padded(U, ng, bc, gh, a, b):
    """Padded groups a .. b - 1 of level storage U (5 fields)."""
    at = _pad_index(ng, bc, gh, a, b)
    flat = U.reshape(-1)
    return torch.stack([flat[at + q * N ** 3] for q in range(5)], 1), at


def _exact_level(U, ng, bc, gh, dt, dx, gamma, case, size=256):
    out = []
    for a, b in _chunks(U.shape[0], size):
        pad, _ = _padded(U, ng, bc, gh, a, b)
        out.append(_exact_step(pad, gh, dt, dx, gamma, case)[0])
    return torch.cat(out)


def _exact_adjoint(U, g, ng, bc, dt, dx, gamma):
    grad = torch.zeros_like(U).reshape(-1)
    for a, b in _chunks(U.shape[0], 64):
        pad, at = _padded(U, ng, bc, 2, a, b)
        pad.requires_grad_(True)
        with torch.enable_grad():
            out, _ = _exact_step(pad, 2, dt, dx, gamma, {})
        gp, = torch.autograd.grad(out, pad, g[a:b])
        for q in range(5):
            grad.index_add_(0, (at + q * N ** 3).reshape(-1), gp[:, q].reshape(-1))
    return grad.reshape(U.shape)


class _Hierarchy:
    """The coupled W-cycle on dense index maps (Secs. 2.1, 2.2, 3.2), periodic."""

    def __init__(self, n0, dx0, gamma, pos, states):
        dev = states[0].device
        self.n0, self.dx0, self.gamma = n0, dx0, gamma
        self.host = pos
        self.pos = [torch.tensor(p, device=dev) for p in pos]
        self.U = [u.double().clone() for u in states]
        self.map = []
        for l, p in enumerate(self.pos):
            n = [v << l for v in n0]
            m = torch.full((n[2], n[1], n[0]), -1, dtype=torch.int64, device=dev)
            m[p[:, 2], p[:, 1], p[:, 0]] = torch.arange(len(p), device=dev)
            self.map.append(m)

    def cells(self, l, x, y, z):
        """Group (-1 where absent) and offset in it of cells of level l, wrapped."""
        n = [N * (v << l) for v in self.n0]
        x, y, z = x % n[0], y % n[1], z % n[2]
        return self.map[l][z // N, y // N, x // N], ((z % N) * N + y % N) * N + x % N

    def values(self, U, group, off):
        return torch.stack([U.reshape(-1)[(group * 5 + q) * N ** 3 + off] for q in range(5)], 1)

    def fill(self, l, old, a, lo, hi, gh):
        """Padded groups lo .. hi - 1 of level l; `old`: the coarse level before its step."""
        P = N + 2 * gh
        i = torch.arange(P, device=self.U[0].device) - gh
        p = self.pos[l][lo:hi] * N
        shape = (hi - lo, P, P, P)
        x = (p[:, 0, None, None, None] + i[None, None, None, :]).expand(shape)
        y = (p[:, 1, None, None, None] + i[None, None, :, None]).expand(shape)
        z = (p[:, 2, None, None, None] + i[None, :, None, None]).expand(shape)
        group, off = self.cells(l, x, y, z)
        out = self.values(self.U[l], group.clamp_min(0), off)
        miss = group < 0
        if bool(miss.any()):
            x, y, z = x[miss], y[miss], z[miss]
            coarse = (1.0 - a) * old + a * self.U[l - 1] if a else old
            c = [x.div(2, rounding_mode="floor"), y.div(2, rounding_mode="floor"), z.div(2, rounding_mode="floor")]

            def at(d, o):
                q = [c[e] + (o if e == d else 0) for e in range(3)]
                return self.values(coarse, *self.cells(l - 1, *q))

            mid = at(0, 0)
            v = mid
            for d, f in enumerate((x, y, z)):
                dm, dp = mid - at(d, -1), at(d, 1) - mid
                s = torch.where(dm * dp > 0, torch.where(dm.abs() < dp.abs(), dm, dp), 0.0)
                v = v + s * torch.where(f % 2 == 1, 0.25, -0.25)[:, None]
            out = out.transpose(0, 1)
            out[:, miss] = v.transpose(0, 1)
            out = out.transpose(0, 1).contiguous()
        return out

    def advance(self, l, dt, old, a, reg):
        dx = self.dx0 / 2 ** l
        before = self.U[l].clone()
        new, planes = [], [[], [], []]
        for lo, hi in _chunks(len(self.host[l]), 256):
            out, flux = _exact_step(self.fill(l, old, a, lo, hi, 2), 2, dt, dx, self.gamma, {})
            new.append(out)
            for d in range(3):   # faces on the patch boundaries, normal coordinate 0, 8, 16 first
                planes[d].append(flux[d].movedim(4 - d, 1)[:, ::8].contiguous())
        self.U[l] = torch.cat(new)
        planes = [torch.cat(p) for p in planes]   # [G, 3, 5, b, a]: the other two axes, the higher one first
        if reg is not None:
            for d in range(3):
                for hi in range(2):
                    f = planes[d][:, 2 * hi].reshape(-1, 5, 8, 2, 8, 2)
                    reg[2 * d + hi] += 0.5 * 0.25 * f.sum(dim=(3, 5))
        if l + 1 < len(self.U):
            nf = len(self.host[l + 1])
            child = [torch.zeros((nf, 5, 8, 8), dtype=torch.float64, device=before.device) for _ in range(6)]
            self.advance(l + 1, 0.5 * dt, before, 0.0, child)
            self.advance(l + 1, 0.5 * dt, before, 0.5, child)
            _restrict(self.U[l + 1], self.U[l], self.host[l + 1], self.host[l])
            self.fix_up(l, dt / dx, planes, child)

    def fix_up(self, l, lam, planes, reg):
        """Uncovered coarse cells across each open side of a fine group: the
        coarse flux of the shared face is replaced by the register."""
        p = self.pos[l + 1]
        n = [v << (l + 1) for v in self.n0]
        i = torch.arange(8, device=p.device)
        flat = self.U[l].reshape(-1)
        for d in range(3):
            for hi in range(2):
                q = p.clone()
                q[:, d] = (q[:, d] + (1 if hi else -1)) % n[d]
                open_ = self.map[l + 1][q[:, 2], q[:, 1], q[:, 0]] < 0
                if not bool(open_.any()):
                    continue
                q = q[open_] * 8                     # the coarse patch across the side
                e, f = [k for k in range(3) if k != d]   # a along e, b along f (f > e)
                c = [None] * 3
                c[d] = (q[:, d, None, None] + (0 if hi else 7)).expand(-1, 8, 8)
                c[e] = (q[:, e, None, None] + i[None, None, :]).expand(-1, 8, 8)
                c[f] = (q[:, f, None, None] + i[None, :, None]).expand(-1, 8, 8)
                group, off = self.cells(l, *c)
                k = ((c[d] % N) + (0 if hi else 1)) // 8
                fc = planes[d][group, k, :, c[f] % N, c[e] % N]            # [m, 8, 8, 5]
                r = reg[2 * d + hi][open_].permute(0, 2, 3, 1)
                corr = (lam if hi else -lam) * (r - fc)
                for v in range(5):
                    flat.index_add_(0, ((group * 5 + v) * N ** 3 + off).reshape(-1), corr[..., v].reshape(-1))


def exact(case, seed):
    with torch.no_grad():
        return _exact(case, seed)


def _exact(case, seed):
    kind = case["kind"]
    if kind == "amr":
        n0, dx0, gamma, pos, states = _amr_state(case, seed)
        h = _Hierarchy(n0, dx0, gamma, pos, states)
        h.advance(0, _amr_dt(states, dx0, gamma), None, 0.0, None)
        return {"U": h.U, "n_bad": None}
    if kind == "wcycle":
        states = _wcycle_states(case, seed)
        dt0 = _wcycle_dt(case, states)
        out = []
        for l, (U, (ng, dx)) in enumerate(zip(states, _wcycle_levels(case))):
            U = U.double()
            for _ in range(2 ** l):
                U = _exact_level(U, ng, (0,) * 6, 2, dt0 / 2 ** l, dx, 5.0 / 3.0, {})
            out.append(U)
        return {"U": out, "n_bad": None}
    U, ng, bc, dx, gamma = _input(case, seed)
    dt = _level_dt(U, dx, gamma)
    given = U
    U = U.double()
    if kind in ("padded", "level"):
        out = _exact_level(U, ng, bc, 2, dt, dx, gamma, case)
        got = {"U": out, "n_bad": None}
        if kind == "padded":
            got["dt_patch"] = _cfl(U, dx, gamma)
        elif case["cfl"]:
            got["dt"] = torch.tensor([_level_dt(out, dx, gamma)], dtype=torch.float64)
        return got
    if kind == "ext":
        if not case["dual"]:
            return {"U": _exact_level(U, ng, bc, 3, dt, dx, gamma, case), "n_bad": None}
        U6 = _with_entropy(given, gamma).double()
        out = []
        for a, b in _chunks(U.shape[0], 128):
            pad, _ = _padded(U, ng, bc, 3, a, b)
            ent, _ = _padded(U6[:, 1:].contiguous(), ng, bc, 3, a, b)
            out.append(_exact_step(torch.cat([pad, ent[:, 4:]], 1), 3, dt, dx, gamma, case)[0])
        return {"U": torch.cat(out), "n_bad": None}
    if kind == "adjoint":
        return _exact_adjoint(U, _cotangent(case, given, seed).double(), ng, bc, dt, dx, gamma)
    dt = 0.2 * dx
    states = [U]
    for _ in range(case["steps"]):
        states.append(_exact_level(states[-1], ng, bc, 2, dt, dx, gamma, {}))
    g = torch.zeros_like(U)
    g[:, 0] = 2.0 * (states[-1][:, 0] - _target(case, given, seed).double())
    for n in range(case["steps"] - 1, -1, -1):
        g = _exact_adjoint(states[n], g, ng, bc, dt, dx, gamma)
    return {"U": states[-1], "grad": g}
