"""The force kernel's ways of sharing a launch among lanes and caches, chosen by
the number of particles of the context: contributions are added in row order in
each, so a simulation gives the same bits whichever way its context takes."""
import numpy as np
import pytest

import workloads as W
from oracle import oracle_from_scene

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def Dem():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2106_09576_amd import Dem as D
    return D


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 63, 64, 65, 257])
def test_few_particles_against_the_oracle(Dem, n):
    # four lanes per particle, 16 particles to a wavefront: whole and partial
    # wavefronts and blocks, rows longer and shorter than four entries
    # (one or two spheres would touch more walls than a particle has slots for)
    sc = W.dense_snapshot(n=n, seed=n, polydisperse=0.2, n_types=2, overlap=0.04, walls=n > 2)
    g, o = Dem.from_scene(sc), oracle_from_scene(sc)
    g.step(3)
    o.step(3)
    Fg, Tg = g.get_forces()
    Fo, To, S = o.forces()
    R = sc["particles"]["radius"]
    # the tolerance of the other FP64 parity tests: only the order of sums differs
    assert np.all(np.linalg.norm(Fg - Fo, axis=1) <= 1e-11 * (np.linalg.norm(Fo, axis=1) + S))
    assert np.all(np.linalg.norm(Tg - To, axis=1) <= 1e-11 * (np.linalg.norm(To, axis=1) + S * R))
    g.close()


# totals on either side of each line of the rule
@pytest.mark.parametrize("total", [50_000, 50_001, 120_000, 120_001, 600_000, 600_001,
                                   1_200_000, 1_200_001])
@pytest.mark.parametrize("n_types,precision,integrator", [(1, "fp64", "verlet"),
                                                          (3, "fp32", "euler")])
def test_same_bits_in_contexts_of_any_size(Dem, total, n_types, precision, integrator):
    sc = W.dense_snapshot(n=1003, seed=5, polydisperse=0.15, n_types=n_types, overlap=0.03, K=10,
                          integrator=integrator)
    # the rest of the context: resting spheres that touch nothing
    m = total - 1003
    side = int(np.ceil(m ** (1 / 3)))
    x = np.stack(np.unravel_index(np.arange(m), (side,) * 3), 1) * 0.01 + 0.01
    rest = dict(sc, walls=[], particles=W._particles(x, 1.5e-3),
                config=dict(sc["config"], domain_lo=(0.0,) * 3, domain_hi=(0.01 * side + 0.02,) * 3))
    alone = Dem.from_scene(sc, precision=precision)
    among = Dem.from_scenes([rest, sc], precision=precision)
    for sim in (alone, among):
        sim.step(25)
    a, b = alone.get_state(0), among.get_state(1)
    for k in ("pos", "vel", "omega", "active"):
        assert np.array_equal(a[k], b[k]), k
    for p, q in zip(alone.get_forces(0), among.get_forces(1)):
        assert np.array_equal(p, q)
    assert np.array_equal(alone.get_wall_contacts(0)[1], among.get_wall_contacts(1)[1])
    alone.close()
    among.close()
