"""Resume where the saved contacts are put into the context's idle memory and
where they do not fit there: the same run, bit for bit."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


# (beside 44 neighbours per particle the arguments fit; a chain of spheres between
# walls has 2, so that a context for 3 holds 72 bytes of histories per particle
# and the arguments are more)
@pytest.mark.parametrize("max_neighbors", [0, 3])
def test_restore_with_and_without_room(max_neighbors):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2106_09576_amd import Dem
    d, n = 3.0e-3, 1500
    rng = np.random.default_rng(8)
    x = np.column_stack([np.arange(n) * 0.995 * d, np.zeros(n), np.zeros(n)]) + 2 * d
    x += rng.uniform(-0.002 * d, 0.002 * d, x.shape)
    lo, hi = 2 * d - 0.49 * d, 2 * d + 0.49 * d
    walls = [W.plane((0, lo, 0), (0, 1, 0)), W.plane((0, hi, 0), (0, -1, 0)),
             W.plane((0, 0, lo), (0, 0, 1)), W.plane((0, 0, hi), (0, 0, -1))]
    cfg = W._cfg(1e-6, (0.0, 0.0, 0.0), (x[:, 0].max() + 2 * d, 4 * d, 4 * d), K=10)
    sc = dict(name="chain", config=cfg, materials=[dict(W.BOX_MATERIAL)], walls=walls,
              particles=W._particles(x, d / 2, rng.uniform(-0.01, 0.01, x.shape),
                                     rng.uniform(-5.0, 5.0, x.shape)))
    a = Dem.from_scene(sc, max_neighbors=max_neighbors)
    a.step(20)
    ck = a.checkpoint()
    cap = a.get_stats()["max_neighbors"] * ((n + 63) // 64 * 64)
    size = 8 + 56 * len(ck["pairs"]) + 48 * len(ck["wall_pairs"]) + 48 * n
    assert (size <= 24 * cap) == (max_neighbors == 0)
    p = dict(sc["particles"], pos=ck["pos"], vel=ck["vel"], omega=ck["omega"])
    b = Dem.from_scene(dict(sc, particles=p), max_neighbors=max_neighbors)
    with pytest.raises(Exception):  # refused, and nothing is changed
        b.restore(dict(ck, pairs=np.array([[0, n - 1]]), delta_t=np.zeros((1, 3))))
    b.restore(ck)
    for steps in (0, 13, 40):
        a.step(steps)
        b.step(steps)
        for u, v in zip(a.get_contacts() + a.get_wall_contacts() + a.get_forces(),
                        b.get_contacts() + b.get_wall_contacts() + b.get_forces()):
            assert np.array_equal(u, v)
        for k, v in a.get_state().items():
            assert np.array_equal(v, b.get_state()[k]), k
    a.close()
    b.close()
