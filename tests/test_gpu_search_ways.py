"""The ways of the contact search (by blocks of cells, by the occupied ones of
them, one thread per particle): lists, flags and carried overlaps against the
oracle for each, and the same bits whichever way a context's other instances
make it take.  Domains of 2^24 search blocks and more are accepted."""
import numpy as np
import pytest

import workloads as W
from oracle import oracle_from_scene

pytestmark = pytest.mark.gpu

D = 3.0e-3


@pytest.fixture(scope="module")
def Dem():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2106_09576_amd import Dem as D
    return D


def in_domain(sc, blocks):
    """The scene with its domain made longer, to about this many search blocks
    of 4 x 4 x 4 cells."""
    c = sc["config"]
    h = 4 * 1.3 * D
    lo, hi = np.array(c["domain_lo"]), np.array(c["domain_hi"])
    hi[2] = lo[2] + h * np.ceil(blocks / np.prod(np.ceil((hi - lo)[:2] / h)))
    return dict(sc, config=dict(c, domain_hi=tuple(hi)))


def clusters(m, spacing=8.0):
    """m^3 clusters of 27 overlapping spheres, far apart."""
    rng = np.random.default_rng(m)
    c = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 1, 3) * spacing * D
    s = np.stack(np.meshgrid(*[np.arange(3)] * 3, indexing="ij"), -1).reshape(1, -1, 3) * 0.97 * D
    x = (c + s).reshape(-1, 3) + rng.uniform(-0.01 * D, 0.01 * D, (27 * m ** 3, 3)) + D
    v, w = rng.uniform(-0.02, 0.02, x.shape), rng.uniform(-10.0, 10.0, x.shape)
    cfg = W._cfg(1e-5, (0.0, 0.0, 0.0), tuple(x.max(axis=0) + D), K=4, gravity=(0.0, 0.0, 0.0))
    return dict(name="clusters", config=cfg, materials=[dict(W.BOX_MATERIAL)], walls=[],
                particles=W._particles(x, D / 2, v, w))


def dense(n, blocks):
    sc = W.dense_snapshot(n=n, seed=n, overlap=0.02, K=4, walls=False)
    sc["config"]["gravity"] = (0.0, 0.0, 0.0)
    return in_domain(sc, blocks)


# (scene, a scene beside it in a batch that changes the way)
CASES = {
    # occupied blocks of 130 particles; beside clusters: few to a block
    "listed_by_blocks": (lambda: dense(6000, 2500), lambda: clusters(20)),
    # occupied blocks of a few particles; beside a bed: many
    "listed_each": (lambda: in_domain(clusters(6), 2500), lambda: dense(120000, 900)),
    # more blocks than half the particles; beside a bed: fewer, and full ones
    "each": (lambda: dense(700, 3000), lambda: dense(60000, 500)),
}


@pytest.mark.parametrize("case", list(CASES))
def test_ways(Dem, case):
    sc, other = CASES[case][0](), CASES[case][1]()
    a, b, o = Dem.from_scene(sc), Dem.from_scenes([other, sc]), oracle_from_scene(sc)
    for n in (0, 11):
        a.step(n)
        b.step(n)
        o.step(n)
        pairs, delta, touching = a.get_contacts()
        op, od, ot = o.contacts()
        assert np.array_equal(pairs, op) and np.array_equal(touching, ot) and touching.any()
        assert np.max(np.abs(delta - od)) <= 1e-11 * max(np.max(np.abs(od)), 1e-300)
        for x, y in zip((pairs, delta, touching), b.get_contacts(1)):
            assert np.array_equal(x, y)
        for k, v in a.get_state().items():
            assert np.array_equal(v, b.get_state(1)[k]), k
    a.close()
    b.close()


def test_a_domain_of_2_to_the_24_blocks(Dem):
    # spheres so unequal that the blocks are 2 x 2 x 2 cells: 514^3 cells are more
    # than 2^24 of them
    rng = np.random.default_rng(1)
    R = np.array([0.5 * D] + [0.1 * D] * 400)
    h = 1.3 * D * (1 + 1e-9)
    x = np.concatenate([[[0.0, 0.0, 0.0]], rng.uniform(-3 * D, 3 * D, (400, 3))])
    far = np.linalg.norm(x, axis=1) > 0.61 * D
    far[0] = True
    R, x = R[far], x[far] + 100 * D
    cfg = W._cfg(1e-6, (0.0, 0.0, 0.0), (513.5 * h,) * 3, gravity=(0.0, 0.0, 0.0))
    sc = dict(name="wide", config=cfg, materials=[dict(W.BOX_MATERIAL)], walls=[],
              particles=W._particles(x, R))
    small = dict(sc, config=dict(cfg, domain_hi=(110 * D,) * 3))
    a, b = Dem.from_scene(sc, max_neighbors=128), Dem.from_scene(small, max_neighbors=128)
    assert a.get_stats()["n_cells"] == 514 ** 3 > 8 * 2 ** 24
    a.step(3)
    b.step(3)
    for p, q in zip(a.get_contacts(), b.get_contacts()):
        assert len(p) > 0 and np.array_equal(p, q)
    a.close()
    b.close()
