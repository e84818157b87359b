"""GPU tests of Adam steps whose moments are kept in units of what a gradient adds to them."""
import numpy as np
import pytest

from test_gpu_parity import REL_F32, bb, forced_steps, layer_slices, relerr, small_problem  # noqa: F401

pytestmark = pytest.mark.gpu


# the betas' edges: no memory at all, a second moment that never moves (a step size of zero), nearly one; eps zero and large
@pytest.mark.parametrize("b1,b2,eps", [(0.0, 0.0, 1e-8), (0.9, 0.5, 0.0), (0.5, 1.0, 1e-8), (0.99, 0.99999, 1e-3)])
@pytest.mark.parametrize("d,c,hidden", [(20, 2, [70]), (20, 2, [150]), (64, 10, [100]), (80, 5, [150]), (30, 3, [40, 20]), (20, 2, [100, 40]),
                                        (20, 2, [50, 30, 60])])
def test_single_steps_from_oracle_state(bb, oracle, d, c, hidden, b1, b2, eps):  # noqa: F811
    cfg = small_problem(d + hidden[0], 300, d, c)
    hp = {"hidden": hidden, "solver": "adam", "batch_size": 50, "alpha": 0.1, "lr": 0.003, "beta1": b1, "beta2": b2, "eps": eps,
          "epochs": 3, "seed": 77}
    for t, g, th, rg, rth in forced_steps(bb, oracle, cfg, hp, 1, 0, [1, 6], 9):
        assert np.isfinite(th).all()
        for name, sl in layer_slices(d, hidden, c):
            assert relerr(g[sl], rg[sl]) < REL_F32, (t, name, "grad")
            assert relerr(th[sl], rth[sl]) < REL_F32, (t, name, "theta")
