"""Timed cases of the DEM library: what a program that simulates spheres has it do.

A pass is one turn of such a program's loop: it advances the simulation by an
output (or coupling) interval and takes the results.  The cases run from the
20 spheres of the paper's example input file to the 4.3 million of the
cylindrical silo, with the search schedules, force laws, integrators, walls,
precisions and readouts that the library offers.

Inputs are beds of touching spheres made from the seed alone: a periodic tile
of a disordered packing (about 1.8 touching and 4.6 candidate pairs per equal
sphere, as a rotating drum's bed has them) fills the lower part of the
geometry, with the motion of the bulk and random velocities and spins on top.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2106_09576_amd import Dem
from paper_2106_09576_amd.dem import load_library

INF = float("inf")
GLASS = dict(density=2500.0, youngs=1.0e6, poisson=0.3, restitution=0.9, friction=0.3,
             rolling_friction=0.1)
DRUM = dict(GLASS, restitution=0.8, friction=0.5, rolling_friction=0.2)
HOPPER = dict(GLASS, youngs=1.0e7, friction=0.4)
APPENDIX = dict(density=2000.0, youngs=1.0e6, poisson=0.3, restitution=0.3, friction=0.1,
                rolling_friction=0.05)


# ------------------------------------------------------------------- cases

def _case(name, kind, n, steps, **kw):
    c = dict(name=name, kind=kind, n=n, steps=steps, precision="fp64", K=20, out="host",
             model="nonlinear", rolling="constant", integrator="verlet")
    c.update(kw)
    if name is None:
        del c["name"]
    return c


def listed():
    return [
        # the paper's example input file: 20 spheres dropped on a floor that
        # translates; nothing but launches and their latency
        _case("floor_20", "floor", 20, 200),
        # the 1,000-sphere box with six walls, read out every 100 steps
        _case("box_1000", "box", 1000, 100),
        # a small odd-sized bed with four materials and unequal spheres under
        # the other laws, its forces and contact list read every 20 steps (a
        # program that analyses contacts)
        _case("mixed_3001", "mixed", 3001, 20, model="linear", rolling="viscous",
              integrator="euler", out="contacts"),
        # a parameter study: 64 drums of 500 to 8,000 spheres in one context,
        # every instance's state collected after 100 steps
        _case("drums_64", "drums", 64, 100, K=0),
        # a mid-sized drum with the default schedule and the FP32 law, the
        # library's own usage example
        _case("drum_100k", "drum", 100_000, 500, precision="fp32"),
        # the same drum saved and resumed: checkpoint, a new context from it,
        # histories restored, 20 more steps
        _case("resume_100k", "drum", 100_000, 20, out="resume"),
        # the wedge silo's discharge, spheres of 2 to 3 mm
        _case("wedge_200k", "wedge", 200_000, 400, K=0),
        # a drum whose cylinder is a triangle mesh
        _case("mesh_200k", "mesh", 200_000, 200, K=0),
        # the million-sphere drum between two outputs, FP64 law
        _case("drum_1m", "drum", 1_000_000, 1000, K=0),
        # the same drum under the FP32 law inside a coupled program on the
        # GPU that takes the state every 20 steps
        _case("drum_1m_coupled", "drum", 1_000_000, 20, precision="fp32", out="device"),
        # the collapsing dam break: fast flow, frequent searches
        _case("dam_1280k", "dam", 1_280_000, 400, K=0),
        # the cylindrical silo with its hopper, log-normal sizes, coupled
        _case("hopper_4300k", "hopper", 4_300_000, 20, K=0, precision="fp32", out="device"),
    ]


def draw(rng):
    """A case of the same ranges: any scene, sizes log-uniform over the
    scene's range, mostly odd, any schedule, law and readout."""
    kind = rng.choice(["box", "mixed", "drums", "drum", "drum", "wedge", "mesh", "dam"])
    lo, hi = dict(box=(50, 4000), mixed=(200, 20_000), drums=(4, 64), drum=(3000, 1_000_000),
                  wedge=(3000, 200_000), mesh=(5000, 200_000), dam=(10_000, 1_000_000))[kind]
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    big = n > 150_000
    out = rng.choice(["host", "device"] + ([] if big else ["contacts"]))
    if kind in ("drum", "box") and not big and rng.random() < 0.15:
        out = "resume"
    kw = dict(precision=rng.choice(["fp64", "fp32"]), out=out)
    kw["K"] = 20 if out == "resume" else rng.choice([0, 0, 10 if kind == "dam" else 20])
    if kind in ("mixed", "drum"):
        kw["model"] = rng.choice(["nonlinear", "nonlinear", "linear"])
        kw["rolling"] = rng.choice(["none", "constant", "constant", "viscous"])
    if kind == "mixed":
        kw["integrator"] = rng.choice(["verlet", "euler"])
    steps = 20 if out in ("device", "resume") else rng.choice([20, 100, 250])
    return _case(None, kind, n, steps, **kw)


# --------------------------------------------------------------------- beds

def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _tile(rng, diameters, phi, m=10, iterations=30):
    """A periodic cube of m^3 spheres at packing fraction phi: a jittered
    lattice whose overlaps are pushed apart, which leaves a disordered packing
    of spheres that touch or just do not."""
    r = 0.5 * diameters(m ** 3)
    n = r.size
    side = (np.sum(4.0 / 3.0 * math.pi * r ** 3) / phi) ** (1.0 / 3.0)
    g = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3)
    x = (g + 0.5 + rng.uniform(-0.25, 0.25, g.shape)) * (side / m)
    iu, ju = np.triu_indices(n, 1)
    for k in range(iterations):
        if k % 15 == 0:
            d2 = np.zeros(iu.size)
            for a in range(3):
                d = x[iu, a] - x[ju, a]
                d -= side * np.round(d / side)
                d2 += d * d
            near = d2 < (1.35 * (r[iu] + r[ju])) ** 2
            i, j = iu[near], ju[near]
            s = r[i] + r[j]
        d = x[i] - x[j]
        d -= side * np.round(d / side)
        dist = np.sqrt((d ** 2).sum(1))
        q = d * (0.4 * np.maximum(1.002 * s - dist, 0.0) / dist)[:, None]
        for a in range(3):
            x[:, a] += np.bincount(i, q[:, a], n) - np.bincount(j, q[:, a], n)
    return x % side, r, side


def _bed(seed, n, diameters, lo, hi, inside, height, phi=0.54):
    """The n spheres of a packing over the box [lo, hi] that lie inside (a
    test on centres and radii) and lowest (by `height` of the centres), in
    random order: positions and radii."""
    rng = np.random.default_rng([seed, n])
    xt, rt, side = _tile(rng, lambda k: diameters(rng, k), phi)
    dev = _device()
    gen = torch.Generator(device=dev).manual_seed(int(rng.integers(1 << 62)))
    xt, rt = torch.tensor(xt, device=dev), torch.tensor(rt, device=dev)
    reps = [max(1, math.ceil((b - a) / side)) for a, b in zip(lo, hi)]
    corner = torch.stack(torch.meshgrid(*[torch.arange(k, device=dev) for k in reps],
                                        indexing="ij"), -1).reshape(-1, 1, 3)
    off = torch.tensor(lo, dtype=torch.float64, device=dev)
    x = ((corner.to(torch.float64) * side + off) + xt).reshape(-1, 3)
    r = rt.expand(corner.shape[0], -1).reshape(-1)
    keep = inside(x, r)
    x, r = x[keep], r[keep]
    if x.shape[0] < n:
        raise ValueError(f"only {x.shape[0]} sites for {n} spheres")
    low = torch.sort(height(x), stable=True).indices[:n]
    low = low[torch.randperm(n, generator=gen, device=dev)]
    x, r = x[low], r[low]
    # the copies of the tile differ a little
    x = x + 2e-4 * float(rt.mean()) * torch.randn(x.shape, generator=gen, device=dev,
                                                  dtype=torch.float64)
    return x, r, gen


def _spheres(x, r, gen, bulk, spin=(0.0, 0.0, 0.0), dv=0.02, dw=5.0, types=None):
    """Particle arrays: bulk velocity (a tensor or three numbers) and spin
    plus random parts."""
    def random(scale, base):
        base = torch.as_tensor(base, dtype=torch.float64, device=x.device)
        return base + scale * torch.randn(x.shape, generator=gen, device=x.device,
                                          dtype=torch.float64)
    vel, omega = random(dv, bulk), random(dw, spin)
    n = x.shape[0]
    return dict(pos=x.cpu().numpy(), radius=r.cpu().numpy(), vel=vel.cpu().numpy(),
                omega=omega.cpu().numpy(),
                types=np.zeros(n, dtype=np.int32) if types is None else types)


def _plane(point, normal, **kw):
    w = dict(kind="plane", point=tuple(point), normal=tuple(normal), material=0, extent=None,
             axis_point=None, omega=None, t_on=-INF, t_off=INF, velocity=None)
    w.update(kw)
    return w


def _round(kind, point, axis, radius, s_min, s_max, omega=0.0, slope=0.0):
    """A cylinder or cone wall around its particles."""
    w = dict(kind=kind, axis_point=tuple(point), axis_dir=tuple(axis), s_min=s_min, s_max=s_max,
             inside=True, material=0, omega=omega, t_on=-INF, t_off=INF, velocity=None)
    w.update(dict(radius=radius) if kind == "cylinder" else dict(radius0=radius, slope=slope))
    return w


def _box_walls(lo, hi):
    walls = []
    for k in range(3):
        e = [0.0, 0.0, 0.0]
        e[k] = 1.0
        walls += [_plane(lo, e), _plane(hi, [-v for v in e])]
    return walls


def _equal(d):
    return lambda rng, k: np.full(k, d)


def _scene(case, dt, lo, hi, walls, particles, materials, gravity=(0.0, 0.0, -9.81),
           cell_factor=1.3):
    return dict(config=dict(dt=dt, gravity=gravity, domain_lo=tuple(lo), domain_hi=tuple(hi),
                            neighbor_threshold=1.3, cell_factor=cell_factor,
                            rebuild_interval=case["K"], integrator=case["integrator"],
                            rolling_model=case["rolling"], contact_model=case["model"],
                            characteristic_velocity=0.5 if case["model"] == "linear" else 0.0),
                materials=materials, walls=walls, particles=particles)


def _drum(case, seed, n=None, omega=1.0, friction=None, meshed=False):
    """A drum spinning about the x axis, 35 % full, length twice its radius."""
    n = case["n"] if n is None else n
    d = 3.0e-3
    R = (n * math.pi * d ** 3 / 6.0 / 0.6 / 0.35 / (2.0 * math.pi)) ** (1.0 / 3.0)
    # the bed is looser than 0.6, and a small drum loses more of it at its walls
    R, L = R * (1.0 + 3.0 * d / R), 2.0 * R * (1.0 + 3.0 * d / R)

    segments, rings = max(24, int(2 * math.pi * R / (2.4 * d))), max(4, int(L / (3.06 * d)))
    inner = R * math.cos(math.pi / segments) if meshed else R

    def inside(x, r):
        c = 0.995 * r
        rho = torch.sqrt(x[:, 1] ** 2 + x[:, 2] ** 2)
        return (rho <= inner - c) & (x[:, 0].abs() <= L / 2 - c)

    x, r, gen = _bed(seed, n, _equal(d), (-L / 2, -R, -R), (L / 2, R, 0.6 * R), inside,
                     lambda x: x[:, 2] - 0.3 * x[:, 1])
    turn = torch.stack([torch.zeros_like(x[:, 0]), -omega * x[:, 2], omega * x[:, 1]], 1)
    p = _spheres(x, r, gen, turn, (omega, 0.0, 0.0))
    if meshed:
        side = _drum_mesh(R, L, omega, segments, rings)
    else:
        side = _round("cylinder", (0.0, 0.0, 0.0), (1.0, 0.0, 0.0), R, -L / 2, L / 2, omega)
    walls = [side] + [_plane((s * L / 2, 0.0, 0.0), (-s, 0.0, 0.0), axis_point=(0.0, 0.0, 0.0),
                             omega=(omega, 0.0, 0.0)) for s in (-1.0, 1.0)]
    m = dict(DRUM) if friction is None else dict(DRUM, friction=friction)
    e = 2 * d
    return _scene(case, 5.0e-6, (-L / 2 - e, -R - e, -R - e), (L / 2 + e, R + e, R + e), walls,
                  p, [m])


def _drum_mesh(R, L, omega, segments, rings):
    ring, seg = np.meshgrid(np.arange(rings + 1), np.arange(segments), indexing="ij")
    a = 2.0 * math.pi * seg.ravel() / segments
    vertices = np.stack([-L / 2 + L * ring.ravel() / rings, R * np.cos(a), R * np.sin(a)], 1)
    ring, seg = (v.ravel() for v in np.meshgrid(np.arange(rings), np.arange(segments),
                                                indexing="ij"))
    a0, a1 = ring * segments + seg, ring * segments + (seg + 1) % segments
    triangles = np.concatenate([np.stack([a0, a1 + segments, a1], 1),
                                np.stack([a0, a0 + segments, a1 + segments], 1)])
    return dict(kind="mesh", vertices=vertices, triangles=triangles.astype(np.int32), material=0,
                axis_point=(0.0, 0.0, 0.0), omega=(omega, 0.0, 0.0), t_on=-INF, t_off=INF,
                velocity=None)


def _drums(case, seed):
    sizes = np.exp(np.random.default_rng(case["n"]).uniform(math.log(500), math.log(8000),
                                                            case["n"])).round().astype(int)
    rng = np.random.default_rng([seed, 64])
    return [_drum(case, seed * 1000 + k, int(m), float(rng.uniform(0.5, 3.0)),
                  float(rng.uniform(0.1, 0.5))) for k, m in enumerate(sizes)]


def _floor(case, seed):
    """Spheres of 5 mm dropped into a cube whose floor translates; about half
    of them have just landed."""
    rng = np.random.default_rng([seed, 20])
    n, d, half = case["n"], 5.0e-3, 0.07
    site = rng.permutation(9 * 9 * 2)[:n]
    x = np.stack([site % 9, site // 9 % 9, site // 81], 1) * 0.011 - (0.044, 0.044, 0.0675)
    x = x + rng.uniform(-1.0, 1.0, x.shape) * (5.0e-4, 5.0e-4, 5.0e-5)
    walls = _box_walls((-half,) * 3, (half,) * 3)
    walls[4] = dict(walls[4], velocity=(0.15, 0.0, 0.0))
    p = dict(pos=x, radius=np.full(n, d / 2), vel=np.zeros((n, 3)), omega=np.zeros((n, 3)),
             types=np.zeros(n, dtype=np.int32))
    return _scene(case, 1.0e-5, (-half - 2 * d,) * 3, (half + 2 * d,) * 3, walls, p,
                  [dict(APPENDIX)])


def _box(case, seed):
    """Equal spheres on the floor of a cube with six walls."""
    n, d = case["n"], 3.0e-3
    L = 0.05 * max(1.0, (n / 1000.0) ** (1.0 / 3.0))

    def inside(x, r):
        return ((x >= 0.995 * r[:, None]) & (x <= L - 0.995 * r[:, None])).all(1)

    x, r, gen = _bed(seed, n, _equal(d), (0.0,) * 3, (L, L, L), inside, lambda x: x[:, 2])
    return _scene(case, 1.0e-5, (-d,) * 3, (L + d,) * 3, _box_walls((0.0,) * 3, (L,) * 3),
                  _spheres(x, r, gen, (0.0, 0.0, 0.0)), [dict(GLASS)], cell_factor=1.2)


def _mixed(case, seed):
    """Unequal spheres of four materials in a box that the outer ones touch."""
    n, d = case["n"], 3.0e-3
    L = d * (n * math.pi / 6.0 * 0.7 / 0.5) ** (1.0 / 3.0) + d

    def inside(x, r):
        return ((x >= 0.98 * r[:, None]) & (x <= L - 0.98 * r[:, None])).all(1)

    x, r, gen = _bed(seed, n, lambda rng, k: rng.uniform(0.7 * d, d, k), (0.0,) * 3,
                     (L, L, 1.6 * L), lambda x, r: inside(x * x.new_tensor([1, 1, 1 / 1.6]), r),
                     lambda x: x[:, 2], phi=0.56)
    types = np.random.default_rng([seed, 3]).integers(0, 4, n).astype(np.int32)
    mats = [dict(GLASS, restitution=e, friction=f, youngs=y, poisson=p, density=q)
            for e, f, y, p, q in ((0.9, 0.3, 1e6, 0.3, 2500.0), (0.5, 0.1, 5e6, 0.25, 3000.0),
                                  (0.7, 0.5, 2e6, 0.35, 2000.0), (0.3, 0.05, 1e7, 0.2, 7850.0))]
    hi = (L, L, 1.6 * L)
    return _scene(case, 1.0e-5, (-d,) * 3, tuple(v + d for v in hi),
                  _box_walls((0.0,) * 3, hi), _spheres(x, r, gen, (0.0, 0.0, 0.0), dv=0.05,
                                                       dw=20.0, types=types), mats)


def _wedge(case, seed):
    """A silo whose floor is two planes at 30 degrees around an open slot."""
    n, d = case["n"], 3.0e-3
    f = min(1.0, (n / 200_000.0) ** (1.0 / 3.0))
    width, depth = 0.2 * f, 0.04 * f
    height = 0.9 * f
    ho, a = 0.5 * max(0.012 * f, 2.0 * d), math.radians(30.0)
    sa, ca = math.sin(a), math.cos(a)
    run = width / 2 - ho
    rise, hl, hv = run * math.tan(a), 0.5 * run / ca, depth / 2 + d
    nl, nr = (sa, 0.0, ca), (-sa, 0.0, ca)
    pl, pr = (-ho - run / 2, 0.0, rise / 2), (ho + run / 2, 0.0, rise / 2)
    walls = [_plane(pl, nl, extent=(-ca, 0.0, sa, hl, hv)),
             _plane(pr, nr, extent=(ca, 0.0, sa, hl, hv)),
             _plane((-width / 2, 0.0, 0.0), (1.0, 0.0, 0.0)),
             _plane((width / 2, 0.0, 0.0), (-1.0, 0.0, 0.0)),
             _plane((0.0, -depth / 2, 0.0), (0.0, 1.0, 0.0)),
             _plane((0.0, depth / 2, 0.0), (0.0, -1.0, 0.0))]

    def inside(x, r):
        c = 0.995 * r
        dl = (x[:, 0] - pl[0]) * sa + (x[:, 2] - pl[2]) * ca
        dr = -(x[:, 0] - pr[0]) * sa + (x[:, 2] - pr[2]) * ca
        return ((dl >= c) & (dr >= c) & (x[:, 2] >= c) & (x[:, 0].abs() <= width / 2 - c) &
                (x[:, 1].abs() <= depth / 2 - c))

    x, r, gen = _bed(seed, n, lambda rng, k: rng.uniform(2.0e-3, d, k),
                     (-width / 2, -depth / 2, 0.0), (width / 2, depth / 2, height), inside,
                     lambda x: x[:, 2], phi=0.58)
    e = 2 * d
    return _scene(case, 5.0e-6, (-width / 2 - e, -depth / 2 - e, -e),
                  (width / 2 + e, depth / 2 + e, height + e), walls,
                  _spheres(x, r, gen, (0.0, 0.0, -0.05)), [dict(GLASS)])


def _hopper(case, seed):
    """A cylinder on a cone of 60 degrees, open at its outlet of 40 mm."""
    n, dmin, dmax = case["n"], 2.0e-3, 3.5e-3
    R, r0 = 0.25, 0.02
    slope = 1.0 / math.tan(math.radians(60.0))
    q = math.sqrt(1.0 + slope * slope)
    top = (R - r0) / slope
    high = top + 1.1 * n * math.pi / 6.0 * 2.52e-3 ** 3 / 0.58 / (math.pi * R * R) + 0.02

    def inside(x, r):
        c = 0.995 * r
        rho, z = torch.sqrt(x[:, 0] ** 2 + x[:, 1] ** 2), x[:, 2]
        return (rho <= R - c) & ((z >= top) | (rho <= r0 + slope * z - c * q)) & (z >= c)

    mu = math.log(2.5e-3) - 0.005
    x, r, gen = _bed(seed, n, lambda rng, k: np.append(
        np.clip(np.exp(rng.normal(mu, 0.1, k - 1)), dmin, dmax), dmax),
        (-R, -R, 0.0), (R, R, high), inside, lambda x: x[:, 2], phi=0.58)
    walls = [_round("cone", (0.0,) * 3, (0.0, 0.0, 1.0), r0, 0.0, top, slope=slope),
             _round("cylinder", (0.0,) * 3, (0.0, 0.0, 1.0), R, top, high + 0.1)]
    e = 2 * dmax
    return _scene(case, 2.0e-6, (-R - e, -R - e, -e), (R + e, R + e, high + 0.1), walls,
                  _spheres(x, r, gen, (0.0, 0.0, -0.05)), [dict(HOPPER)])


def _dam(case, seed):
    """The heap of the dam break just after the dam's removal, spreading
    along x (gravity -y)."""
    n, d = case["n"], 1.0e-3
    f = min(1.0, (n / 160_000.0) ** (1.0 / 3.0))
    length, height, depth = 0.4 * f, 0.2 * f, max(0.01 * n / 160_000.0, 0.01 * f)
    hi = (length, height, depth)

    def inside(x, r):
        top = x.new_tensor(hi)
        return ((x >= 0.995 * r[:, None]) & (x <= top - 0.995 * r[:, None])).all(1)

    x, r, gen = _bed(seed, n, _equal(d), (0.0,) * 3, hi, inside,
                     lambda x: x[:, 1] + 0.35 * x[:, 0])
    fall = 0.6 * f * x / x.new_tensor([length, height, depth])
    bulk = torch.stack([fall[:, 0], -fall[:, 1], torch.zeros_like(fall[:, 0])], 1)
    e = 2 * d
    walls = _box_walls((0.0,) * 3, hi)
    del walls[3]  # open above
    return _scene(case, 1.0e-5, (-e,) * 3, tuple(v + e for v in hi), walls,
                  _spheres(x, r, gen, bulk, dv=0.05), [dict(APPENDIX)],
                  gravity=(0.0, -9.81, 0.0))


def _scenes(case, seed):
    if case["kind"] == "drums":
        return _drums(case, seed)
    if case["kind"] == "mesh":
        return [_drum(case, seed, meshed=True)]
    return [dict(floor=_floor, box=_box, mixed=_mixed, drum=_drum, wedge=_wedge, hopper=_hopper,
                 dam=_dam)[case["kind"]](case, seed)]


# ------------------------------------------------------------------- passes

def prepare(case, seed):
    """A running program's hands: its context with the particles set."""
    scenes = _scenes(case, seed)
    sim = Dem.from_scenes(scenes, precision=case["precision"])
    state = dict(case=case, scenes=scenes, sim=sim)
    if case["out"] == "device":
        n = [s["particles"]["radius"].size for s in scenes]
        state["buffers"] = [{k: torch.empty(m, 3, dtype=torch.float64, device="cuda")
                             for k in ("pos", "vel", "omega")} for m in n]
    return state


def _host(sim, count):
    """Every instance's state, one after the other."""
    got = [sim.get_state(k) for k in range(count)]
    return {k: got[0][k] if count == 1 else np.concatenate([g[k] for g in got])
            for k in ("pos", "vel", "omega", "active")}


def _to_device(state):
    """The state into a program's own device tensors (C interface)."""
    lib, sim = load_library(), state["sim"]
    for k, b in enumerate(state["buffers"]):
        rc = lib.dem_get_state_device(sim._h, k, b["pos"].data_ptr(), b["vel"].data_ptr(),
                                      b["omega"].data_ptr(), None)
        if rc:
            raise RuntimeError(lib.dem_last_error(None).decode())
    if len(state["buffers"]) == 1:
        return state["buffers"][0]
    return {k: torch.cat([b[k] for b in state["buffers"]]) for k in ("pos", "vel", "omega")}


def _resume(state):
    """Save the simulation and go on in a new context from what was saved."""
    sim, scene, case = state["sim"], state["scenes"][0], state["case"]
    saved = sim.checkpoint()
    particles = dict(scene["particles"], **{k: saved[k] for k in ("pos", "vel", "omega")})
    again = Dem.from_scene(dict(scene, particles=particles), precision=case["precision"])
    again.restore(saved)
    again.step(case["steps"])
    out = _host(again, 1)
    out["force"], out["torque"] = again.get_forces()
    again.close()
    return out


def _filled(a, rows):
    """The rows of a in an array of the program's own capacity."""
    b = np.zeros((rows,) + a.shape[1:], dtype=a.dtype)
    b[:a.shape[0]] = a
    return b


def run(state):
    sim, case = state["sim"], state["case"]
    sim.step(case["steps"])
    if case["out"] == "device":
        return _to_device(state)
    if case["out"] == "resume":
        return _resume(state)
    out = _host(sim, len(state["scenes"]))
    if case["out"] == "contacts":
        out["force"], out["torque"] = sim.get_forces()
        for key, a in zip(("pairs", "delta_t", "touching"), sim.get_contacts()):
            out[key] = _filled(a, 16 * sim.counts[0])
    return out


def work(case):
    """What a pass cannot do without: every step reads and writes each
    sphere's state (72 + 72 bytes and 8 of radius and material) and reads and
    writes each candidate pair (56 bytes: identity, tangential overlap), with
    about 350 operations for each of the touching ones (both sides); a search
    reads and writes the state and the lists once more; the readout writes
    the results."""
    n = case["n"] * (2700 if case["kind"] == "drums" else 1)
    pairs, touch = {"floor": (0.2, 0.1), "mixed": (6.0, 2.0), "wedge": (8.0, 2.3),
                    "hopper": (9.5, 2.3)}.get(case["kind"], (4.6, 1.8))
    steps = case["steps"] * (2 if case["out"] == "resume" else 1)
    every = case["K"] if case["K"] else {"dam": 20}.get(case["kind"], 50)
    b = steps * n * (152 + 56 * pairs) + (steps / every) * n * (300 + 60 * pairs) + 72 * n
    if case["out"] in ("contacts", "resume"):
        b += n * (48 + 41 * pairs)  # forces, torques and the contact list
    return dict(bytes=b, flops=steps * n * touch * 700.0)


# ---------------------------------------------------- the same in plain torch

def _near_pairs(x, reach):
    """Pairs (i, j) of rows of x closer than reach, each once."""
    lo = x.min(0).values
    c = torch.floor((x - lo) / reach).to(torch.int64) + 1
    m = c.max(0).values + 2
    key = (c[:, 2] * m[1] + c[:, 1]) * m[0] + c[:, 0]
    order = torch.argsort(key)
    key_s, n = key[order], x.shape[0]
    out = []
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                d = int((dz * m[1] + dy) * m[0] + dx)
                if d < 0:
                    continue
                first = torch.searchsorted(key_s, key_s + d)
                count = torch.searchsorted(key_s, key_s + d, right=True) - first
                i = torch.repeat_interleave(torch.arange(n, device=x.device), count)
                k = torch.arange(i.numel(), device=x.device) - (count.cumsum(0) - count)[i]
                j = first[i] + k
                keep = j > i if d == 0 else torch.ones_like(i, dtype=torch.bool)
                i, j = order[i[keep]], order[j[keep]]
                near = ((x[i] - x[j]) ** 2).sum(1) < reach * reach
                out.append((i[near], j[near]))
    return torch.cat([a for a, _ in out]), torch.cat([b for _, b in out])


def _coefficients(case, a, b, mean):
    """kn, kt, en, et, mu, mur of two materials' contacts (b: the wall's when
    not mean)."""
    ye = 1.0 / ((1 - a["poisson"] ** 2) / a["youngs"] + (1 - b["poisson"] ** 2) / b["youngs"])
    ge = 1.0 / (2 * (2 - a["poisson"]) * (1 + a["poisson"]) / a["youngs"] +
                2 * (2 - b["poisson"]) * (1 + b["poisson"]) / b["youngs"])
    e, mu, mur = (0.5 * (a[k] + b[k]) if mean else b[k]
                  for k in ("restitution", "friction", "rolling_friction"))
    le = math.log(e)
    if case["model"] == "linear":
        k = 16.0 / 15.0 * ye * (15.0 * 0.5 ** 2 / (16.0 * ye)) ** 0.2
        c = 2.0 / math.sqrt(1.0 + (math.pi / le) ** 2)
        return [k, k, c, c, mu, mur]
    beta = -2.0 * math.sqrt(5.0 / 6.0) * le / math.sqrt(le * le + math.pi ** 2)
    return [4.0 / 3.0 * ye, 8.0 * ge, beta * math.sqrt(2 * ye), beta * math.sqrt(8 * ge), mu, mur]


def _law(case, c, dt, dn, n, v, wrel, vroll, me, re, ri, delta):
    """Force and torque on the first body of touching contacts and their new
    tangential overlaps."""
    def col(k):
        return c[:, k:k + 1]
    dn, me, re, ri = (t[:, None] for t in (dn, me, re, ri))
    vn = (v * n).sum(1, keepdim=True) * n
    vt = v - vn
    delta = delta + vt * dt
    if case["model"] == "linear":
        kn = kt = col(0) * (re * re * me) ** 0.2
        en = et = col(2) * torch.sqrt(me * kn)
    else:
        q = torch.sqrt(re * dn)
        kn, kt = col(0) * q, col(1) * q
        en, et = col(2) * torch.sqrt(me * q), col(3) * torch.sqrt(me * q)
    fn = -(kn * dn) * n - en * vn
    ft = -kt * delta - et * vt
    size = fn.norm(dim=1, keepdim=True)
    ftn = ft.norm(dim=1, keepdim=True)
    slip = (ftn >= col(4) * size) & (ftn > 0)
    fh = torch.where(slip, col(4) * size * ft / torch.where(ftn > 0, ftn, 1.0), ft)
    delta = torch.where(slip, -(fh + et * vt) / kt, delta)
    m = ri * torch.linalg.cross(n, fh)
    if case["rolling"] != "none":
        wn = wrel.norm(dim=1, keepdim=True)
        mag = col(5) * re * size
        if case["rolling"] == "viscous":
            mag = mag * vroll.norm(dim=1, keepdim=True)
        m = m - torch.where(wn > 0, mag * wrel / torch.where(wn > 0, wn, 1.0), 0.0)
    return fn + fh, m, delta


def _wall_contact(w, x, r, t):
    """Touching centres of a wall: mask, normals towards the wall, overlaps,
    contact points."""
    def vec(v):
        return x.new_tensor(v)
    shift = vec(w["velocity"]) * t if w.get("velocity") is not None else vec((0.0,) * 3)
    if w["kind"] == "plane":
        nrm = vec(w["normal"])
        nrm = nrm / nrm.norm()
        rel = x - vec(w["point"]) - shift
        dist = rel @ nrm
        on = (dist < r) & (dist > -r)
        if w["extent"] is not None:
            u = vec(w["extent"][:3])
            u = u - (u @ nrm) * nrm
            u = u / u.norm()
            on &= ((rel @ u).abs() <= w["extent"][3]) & \
                  ((rel @ torch.linalg.cross(nrm, u)).abs() <= w["extent"][4])
        return on, (-nrm).expand_as(x), r - dist, x - dist[:, None] * nrm
    ax = vec(w["axis_dir"])
    rel = x - vec(w["axis_point"]) - shift
    s = rel @ ax
    radial = rel - s[:, None] * ax
    rho = radial.norm(dim=1)
    slope = w.get("slope", 0.0)
    q = math.sqrt(1.0 + slope * slope)
    er = radial / torch.where(rho > 0, rho, 1.0)[:, None]
    dist = (w.get("radius0", w.get("radius")) + slope * s - rho) / q
    n = (er - slope * ax) / q
    on = (s >= w["s_min"]) & (s <= w["s_max"]) & (rho > 0) & (dist < r) & (dist > -r)
    return on, n, r - dist, x + dist[:, None] * n


def _simulate(case, scene, steps):
    """The scene's state after `steps` steps: pos, vel, omega, force, torque."""
    cfg, p, dev = scene["config"], scene["particles"], _device()
    x, v, w, r = (torch.tensor(p[k], device=dev) for k in ("pos", "vel", "omega", "radius"))
    kind = torch.tensor(p["types"].astype(np.int64), device=dev)
    mats = scene["materials"]
    mass = x.new_tensor([m["density"] for m in mats])[kind] * (4.0 / 3.0 * math.pi) * r ** 3
    inertia = 0.4 * mass * r * r
    dt, g = cfg["dt"], x.new_tensor(cfg["gravity"])
    pp, pw = (x.new_tensor([[_coefficients(case, a, b, mean) for b in mats] for a in mats])
              for mean in (True, False))
    # pairs that can come to touch while nothing is faster than 3 m/s
    i, j = _near_pairs(x, 2.0 * float(r.max()) + 6.0 * dt * (steps + 1))
    gap = (x[i] - x[j]).norm(dim=1) - r[i] - r[j]
    i, j = i[gap < 6.0 * dt * (steps + 1)], j[gap < 6.0 * dt * (steps + 1)]
    c = pp[kind[i], kind[j]]
    delta = torch.zeros(i.numel(), 3, dtype=x.dtype, device=dev)
    wdelta = [torch.zeros_like(x) for _ in scene["walls"]]
    force, torque = torch.zeros_like(x), torch.zeros_like(x)

    def evaluate(t):
        force, torque = torch.zeros_like(x), torch.zeros_like(x)
        d = x[j] - x[i]
        dist = d.norm(dim=1)
        k = torch.nonzero(dist < r[i] + r[j])[:, 0]
        a, b, n = i[k], j[k], d[k] / dist[k, None]
        vroll = torch.linalg.cross(r[a, None] * w[a] + r[b, None] * w[b], n)
        f, m, new = _law(case, c[k], dt, r[a] + r[b] - dist[k], n, v[a] - v[b] + vroll,
                         w[a] - w[b], vroll, mass[a] * mass[b] / (mass[a] + mass[b]),
                         r[a] * r[b] / (r[a] + r[b]), r[a], delta[k])
        delta.zero_()
        delta[k] = new
        # the tangential part turns both bodies the same way, by their own
        # radii; the rolling part is opposite
        nf = torch.linalg.cross(n, f)
        roll = m - r[a, None] * nf
        force.index_add_(0, a, f).index_add_(0, b, -f)
        torque.index_add_(0, a, m).index_add_(0, b, r[b, None] * nf - roll)
        for wl, wd in zip(scene["walls"], wdelta):
            if not wl["t_on"] <= t < wl["t_off"]:
                wd.zero_()
                continue
            on, n, dn, point = _wall_contact(wl, x, r, t)
            k = torch.nonzero(on)[:, 0]
            n = n[k]
            om = wl["omega"]
            if om is None:
                om = (0.0,) * 3
            om = x.new_tensor(om if wl["kind"] == "plane" else [om * u for u in wl["axis_dir"]])
            vel = x.new_tensor(wl["velocity"] if wl.get("velocity") is not None else (0.0,) * 3)
            at = wl["axis_point"] if wl["axis_point"] is not None else wl["point"]
            arm = point[k] - x.new_tensor(at) - vel * t
            wrel = w[k] - om
            vroll = torch.linalg.cross(r[k, None] * wrel, n)
            slip = v[k] - vel - torch.linalg.cross(om.expand_as(arm), arm) + \
                torch.linalg.cross(r[k, None] * w[k], n)
            f, m, new = _law(case, pw[kind[k], wl["material"]], dt, dn[k], n, slip, wrel, vroll,
                             mass[k], r[k], r[k], wd[k])
            wd.zero_()
            wd[k] = new
            force.index_add_(0, k, f)
            torque.index_add_(0, k, m)
        return force, torque

    for step in range(1, steps + 1):
        if case["integrator"] == "euler":
            force, torque = evaluate((step - 1) * dt)
            x = x + v * dt
            v = v + (force / mass[:, None] + g) * dt
            w = w + torque / inertia[:, None] * dt
            continue
        v = v + (force / mass[:, None] + g) * (0.5 * dt)
        w = w + torque / inertia[:, None] * (0.5 * dt)
        x = x + v * dt
        force, torque = evaluate(step * dt)
        v = v + (force / mass[:, None] + g) * (0.5 * dt)
        w = w + torque / inertia[:, None] * (0.5 * dt)
    return dict(pos=x, vel=v, omega=w, force=force, torque=torque)


def exact(case, seed):
    """The results of a first pass in 64 bits.  None where there are none to
    tell: after about 50 steps a dense bed's rounding has grown past its
    results' own digits (the rolling torque follows the sign of small spins),
    and triangle meshes are left to the library."""
    steps = case["steps"] * (2 if case["out"] == "resume" else 1)
    if case["kind"] == "mesh" or (steps > 50 and case["kind"] != "floor"):
        return None
    got = [_simulate(case, s, steps) for s in _scenes(case, seed)]
    keys = ("pos", "vel", "omega") + \
        (() if case["out"] in ("host", "device") else ("force", "torque"))
    return {k: torch.cat([g[k] for g in got]) for k in keys}
