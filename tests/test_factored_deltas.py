"""GPU tests of hidden deltas that leave the output weight to the end of the step: models with one output column."""
import numpy as np
import pytest
import torch

from test_gpu_parity import bb, layer_slices, small_problem  # noqa: F401

pytestmark = pytest.mark.gpu


# inputs, hidden, batch, classes: two and four tiles of inputs (split products) and three (fp32), one to three unit tiles a
# wave with the last one missing in some, an odd number of row tiles, one row past a chunk; two classes, one logit, regression
@pytest.mark.parametrize("d,h,bs,c", [(17, 70, 16, 1), (32, 129, 65, 1), (30, 192, 48, 0), (25, 160, 130, 2), (20, 224, 17, 1),
                                      (63, 128, 33, 1), (50, 20, 64, 0), (33, 40, 80, 1), (48, 200, 31, 2)])
def test_gradients_are_as_close_to_exact_as_fp32_sums(bb, oracle, d, h, bs, c):  # noqa: F811
    """The first step's gradients, with a third of the rows zero (a unit is then on or off by its bias alone), against pure
    fp64: no further off than the oracle's own with fp32 running sums, give or take the rounding of the result and the
    roundings in between that both make (the bound of the tests of split products)."""
    cfg = small_problem(d + h, 300, d, c)
    cfg["X"][::3] = 0
    hp = {"hidden": [h], "solver": "sgd", "batch_size": bs, "alpha": 0.1, "lr": 1e-3, "momentum": 0.0, "epochs": 1, "seed": 5}
    X, y, ft = bb.to_device(cfg)
    tr = bb.bbo_mlp_cv_eval(X, y, c, ft, 5, [hp], 0, trace=(0, 1, 0, 1))[-1]
    torch.cuda.synchronize()
    exact, sums = (oracle.train_one(cfg["X"], cfg["y"], c, cfg["fold_idx"], hp, 1, prec=p, step_begin=0, step_end=1)["grad"][0]
                   for p in (1, 2))
    for name, sl in layer_slices(d, [h], max(c, 1)):
        if sl.stop - sl.start < 16:
            continue  # the output bias: the norm-wise error of one or two numbers is the rounding of one
        want = exact[sl].astype(np.float64)
        off = lambda g: np.linalg.norm(g.astype(np.float64) - want) / np.linalg.norm(want)
        here, fp32 = off(tr["grad"][0, sl].cpu().numpy()), off(sums[sl])
        print("%s d %d h %d bs %d c %d: %.2e, fp32 sums %.2e" % (name, d, h, bs, c, here, fp32))
        assert here < 1.5 * fp32 + 2.0 ** -24, name
