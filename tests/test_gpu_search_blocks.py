"""The contact search by blocks of cells: candidate lists, touching flags and
carried overlaps against the oracle where a block's region fits in LDS and
where it does not, where a particle has more candidates than its list or its
row holds in LDS, and on grids with very few cells along an axis."""
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


def check(Dem, sc, steps=12):
    g, o = Dem.from_scene(sc), oracle_from_scene(sc)
    for n in (0, steps):
        g.step(n)
        o.step(n)
        gp, gd, gt = g.get_contacts()
        op, od, ot = o.contacts()
        assert np.array_equal(gp, op) and np.array_equal(gt, ot)
        assert len(gp) > 0
        # the overlaps of a few steps: rounding only (the scale of the largest)
        assert np.max(np.abs(gd - od)) <= 1e-11 * max(np.max(np.abs(od)), 1e-300)
    g.resort()  # carries every overlap into a new list
    gp, gd, gt = g.get_contacts()
    assert np.array_equal(gp, op)
    assert np.max(np.abs(gd - od)[gt]) <= 1e-11 * np.max(np.abs(od))
    g.close()


# cells of 1.3 to 6 diameters: 4 x 4 x 4 cells to a block, then smaller blocks,
# then regions that no longer fit
@pytest.mark.parametrize("cell_factor", [1.3, 1.6, 2.0, 2.6, 4.0, 6.0])
@pytest.mark.parametrize("n", [1, 2, 700, 4099])
def test_cell_sizes(Dem, cell_factor, n):
    sc = W.dense_snapshot(n=max(n, 8), seed=n, polydisperse=0.3, overlap=0.03, K=4)
    if n < 8:
        sc["particles"] = {k: v[:n] for k, v in sc["particles"].items()}
    sc["config"]["cell_factor"] = cell_factor
    if n >= 8:
        check(Dem, sc)
    else:
        g = Dem.from_scene(sc)
        g.step(5)
        assert g.get_stats()["n_active"] == n
        g.close()


# a few large spheres among many small ones: their rows are far longer than the
# mean row, beyond the list's and the row's part in LDS
@pytest.mark.parametrize("ratio", [2.0, 3.0])
def test_long_rows(Dem, ratio):
    sc = W.dense_snapshot(n=3000, seed=3, overlap=0.02, K=4, walls=False)
    p = sc["particles"]
    d = 2 * p["radius"][0]
    x = p["pos"]
    c = x.mean(axis=0) + np.array([[0.0, 0.0, 0.0], [2.5 * ratio * d, 0.0, 0.0]])
    far = np.min(np.linalg.norm(x[:, None] - c[None], axis=2), axis=1) > (0.5 * ratio + 0.49) * d
    n = int(far.sum()) + len(c)
    particles = W._particles(np.concatenate([x[far], c]),
                             np.concatenate([p["radius"][far], np.full(len(c), ratio * d / 2)]),
                             np.concatenate([p["vel"][far], np.zeros((len(c), 3))]),
                             np.concatenate([p["omega"][far], np.zeros((len(c), 3))]))
    assert particles["pos"].shape[0] == n
    check(Dem, dict(sc, particles=particles))


# one, two, three and five cells along an axis, also of a batch
@pytest.mark.parametrize("cells", [(1, 9, 9), (9, 2, 9), (9, 9, 3), (1, 1, 40), (5, 2, 1)])
def test_thin_grids(Dem, cells):
    d = 3.0e-3
    rng = np.random.default_rng(4)
    h = 1.3 * d * (1 + 1e-9)
    size = np.array(cells) * h * 0.999
    ax = [np.arange(0.5 * d, s - 0.4 * d, 0.97 * d) for s in size]
    x = np.stack(np.meshgrid(*ax, indexing="ij"), -1).reshape(-1, 3)
    x += rng.uniform(-0.02 * d, 0.02 * d, x.shape)
    cfg = W._cfg(1e-5, (0.0, 0.0, 0.0), tuple(size), K=4, gravity=(0.0, 0.0, 0.0))
    sc = dict(name="thin", config=cfg, materials=[dict(W.BOX_MATERIAL)], walls=[],
              particles=W._particles(x, d / 2, rng.uniform(-0.02, 0.02, x.shape)))
    check(Dem, sc)
    # the same instance between two others of other grids
    other = W.dense_snapshot(n=300, seed=1, K=4)
    other["config"] = dict(cfg, domain_lo=other["config"]["domain_lo"],
                           domain_hi=other["config"]["domain_hi"])
    a, b = Dem.from_scene(sc), Dem.from_scenes([other, sc, other])
    a.step(9)
    b.step(9)
    for p, q in zip(a.get_contacts(0), b.get_contacts(1)):
        assert np.array_equal(p, q)
    for k, v in a.get_state(0).items():
        assert np.array_equal(v, b.get_state(1)[k]), k
    a.close()
    b.close()


# contexts that one workgroup sorts and the sizes just beyond (4,096 particles,
# 16,383 cells, 64 KB of LDS): the same order, so the same bits
@pytest.mark.parametrize("n,extra_cells", [(1, 0), (63, 0), (1023, 0), (1025, 0), (4096, 0),
                                           (4097, 0), (500, 4000), (500, 14000), (500, 40000)])
def test_small_sorts(Dem, n, extra_cells):
    sc = W.dense_snapshot(n=n, seed=n + 1, polydisperse=0.1, K=3, walls=n > 8)
    # a longer box of empty cells, and a particle that has left it
    c = sc["config"]
    h = 1.3 * 2 * float(sc["particles"]["radius"].max())
    lo, hi = np.array(c["domain_lo"]), np.array(c["domain_hi"])
    layer = max(1, int(np.prod(np.ceil((hi - lo)[:2] / h))))
    hi[2] += extra_cells / layer * h
    sc = dict(sc, config=dict(c, domain_hi=tuple(hi)))
    p = sc["particles"]
    out = W._particles(np.concatenate([p["pos"], [hi + 1.0]]), np.append(p["radius"], 1e-3),
                       np.concatenate([p["vel"], np.zeros((1, 3))]),
                       np.concatenate([p["omega"], np.zeros((1, 3))]))
    sc = dict(sc, particles=out)
    g, o = Dem.from_scene(sc), oracle_from_scene(sc)
    g.step(7)
    o.step(7)
    gp, gd, gt = g.get_contacts()
    op, od, ot = o.contacts()
    assert np.array_equal(gp, op) and np.array_equal(gt, ot)
    st = g.get_state()
    assert not st["active"][n] and st["active"][:n].all()
    # a context too large for one workgroup holds the same instance: same bits
    rest = W.dense_snapshot(n=5000, seed=2, K=3, walls=False)
    b = Dem.from_scenes([rest, sc])
    b.step(7)
    for k, v in st.items():
        assert np.array_equal(v, b.get_state(1)[k]), k
    for x, y in zip(g.get_contacts(), b.get_contacts(1)):
        assert np.array_equal(x, y)
    g.close()
    b.close()
