"""Device memory of a context whose cell grid was tuned: what a context built
with that grid holds."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cell_factor", [1.3, 2.5])
def test_tuned_context_holds_one_grid(cell_factor):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2106_09576_amd import Dem
    sc = W.dense_snapshot(n=2000, seed=4, K=5, vmax=0.01, walls=False)
    c = sc["config"]
    hi = np.array(c["domain_hi"]) * (1.0, 1.0, 200.0)  # tables of some megabytes
    sc = dict(sc, config=dict(c, domain_hi=tuple(hi), gravity=(0.0, 0.0, 0.0),
                              cell_factor=cell_factor))
    sim = Dem.from_scene(sc)
    for _ in range(2):
        t = sim.autotune(trial_steps=10)
        fresh = Dem.from_scene(dict(sc, config=dict(sc["config"], cell_factor=t["cell_factor"])))
        a, b = sim.get_stats(), fresh.get_stats()
        fresh.close()
        assert a["n_cells"] == b["n_cells"] > 50000
        assert a["device_bytes"] == b["device_bytes"]
    sim.close()
