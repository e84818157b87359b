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


# Targets of 3e19: the square of a gradient is a float, and so is the second moment, but not the sum of thirty squares.
@pytest.mark.parametrize("b1,b2", [(0.9, 0.999), (0.0, 0.99), (0.9, 1.0 - 2.0 ** -24)])
@pytest.mark.parametrize("d,hidden", [(13, [50]), (20, [150]), (45, [60]), (80, [150]), (100, [40]), (20, [100, 40]), (20, [50, 30, 60])])
def test_gradients_as_large_as_their_squares_allow(bb, oracle, d, hidden, b1, b2):  # noqa: F811
    cfg = small_problem(d + hidden[0], 300, d, 0)
    cfg["y"] *= np.float32(3e19)
    hp = {"hidden": hidden, "solver": "adam", "batch_size": 50, "alpha": 0.1, "lr": 1e-4, "beta1": b1, "beta2": b2, "epochs": 8, "seed": 7}
    for t, g, th, rg, rth in forced_steps(bb, oracle, cfg, hp, 1, 0, [1, 36], 38):
        assert 3e18 < np.abs(rg).max() < 1.8e19
        for name, sl in layer_slices(d, hidden, 0):
            assert relerr(g[sl], rg[sl]) < REL_F32, (t, name, "grad")
        # (no parameter is off by a twentieth of a step's length; one that stands still is by about a whole one)
        assert np.abs(th - rth).max() < 0.05 * hp["lr"]
