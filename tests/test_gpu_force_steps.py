"""Several steps in one launch, which small contexts take between two searches,
against one launch per step, which any context takes while it is timed: the same
state, forces, contact lists and schedule of searches, bit for bit."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def Dem():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2106_09576_amd import Dem as D
    return D


def _same(a, b, k):
    p, q = a.get_state(k), b.get_state(k)
    for key in ("pos", "vel", "omega", "active"):
        assert np.array_equal(p[key], q[key]), key
    for u, v in zip(a.get_forces(k), b.get_forces(k)):
        assert np.array_equal(u, v)
    for u, v in zip(a.get_contacts(k), b.get_contacts(k)):
        assert np.array_equal(u, v)
    for u, v in zip(a.get_wall_contacts(k), b.get_wall_contacts(k)):
        assert np.array_equal(u, v)


def _run(Dem, scenes, steps, **kw):
    several, single = Dem.from_scenes(scenes, **kw), Dem.from_scenes(scenes, **kw)
    single.set_timing(True)
    for m in steps:
        for sim in (several, single):
            sim.step(m)
        for k in range(len(scenes)):
            _same(several, single, k)
    several.close()
    single.close()


# whole and partial wavefronts of 16 particles, one and several of them, both
# sides of the largest context, and calls that end anywhere between two searches
@pytest.mark.parametrize("n", [1, 16, 17, 100, 127, 128, 129])
@pytest.mark.parametrize("precision,model,rolling,integrator,n_types,K", [
    ("fp64", "nonlinear", "constant", "verlet", 1, 5),
    ("fp64", "linear", "viscous", "euler", 3, 7),
    ("fp32", "nonlinear", "viscous", "verlet", 3, 0),
    ("fp32", "linear", "constant", "euler", 1, 0)])
def test_same_bits_as_one_launch_per_step(Dem, n, precision, model, rolling, integrator, n_types, K):
    sc = W.dense_snapshot(n=n, seed=n, polydisperse=0.2, n_types=n_types, overlap=0.03,
                          walls=n > 2, rolling=rolling, integrator=integrator, model=model, K=K,
                          V=0.5 if model == "linear" else 0.0)
    if n > 2:  # a sliding floor: the time of a step matters
        sc["walls"][4]["velocity"] = (0.05, 0.0, 0.0)
    _run(Dem, [sc], (1, 2, 4, 23, 60), precision=precision)


def test_small_batch_and_leaving_particles(Dem):
    # 128 particles in instances of their own kinds; some fly out of the domain
    scenes = [W.dense_snapshot(n=n, seed=n, n_types=1, K=6, polydisperse=0.1, vmax=v,
                               walls=n > 2 and v < 1.0)
              for n, v in ((1, 0.05), (40, 3.0), (30, 0.05), (57, 0.05))]
    for sc in scenes:
        sc["config"] = dict(sc["config"], dt=scenes[0]["config"]["dt"])
    _run(Dem, scenes, (3, 30, 301), precision="fp64")


def test_more_steps_than_a_launch_takes(Dem):
    sc = W.dense_snapshot(n=60, seed=3, K=700, vmax=0.001, wmax=0.1, dt=1e-8)
    _run(Dem, [sc], (255, 1, 256, 1500), precision="fp64")
