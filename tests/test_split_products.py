"""GPU tests of products in three bfloat16 parts: how far a step's gradient is from the exact one, against what fp32 sums give."""
import numpy as np
import pytest
import torch

from test_gpu_parity import bb, layer_slices, small_problem  # noqa: F401

pytestmark = pytest.mark.gpu


# inputs, hidden, batch, scale of the inputs: two and four tiles of inputs, an odd number of row tiles, rows past a chunk
@pytest.mark.parametrize("d,h,bs,c", [(17, 100, 64, 2), (30, 200, 80, 2), (32, 130, 49, 2), (30, 210, 17, 2), (50, 64, 33, 2),
                                      (63, 128, 200, 2), (64, 100, 80, 10), (40, 200, 96, 7), (64, 256, 65, 16), (64, 256, 97, 16), (75, 100, 33, 5)])
@pytest.mark.parametrize("scale", [1.0, 2.0 ** -30, 2.0 ** 10])
def test_gradients_are_as_close_to_exact_as_fp32_sums(bb, oracle, d, h, bs, c, scale):  # noqa: F811
    """The first step's gradients against pure fp64: no further off than the oracle's own with fp32 running sums, which
    round after every term, give or take a rounding of the result (2^-24) and the roundings in between that both make
    (outputs, deltas).  Weights only: a norm-wise error of two output biases is the rounding of one number, which says
    nothing about a sum's."""
    cfg = small_problem(d + h, 300, d, c)
    cfg["X"] = (cfg["X"] * np.float32(scale)).astype(np.float32)
    hp = {"hidden": [h], "solver": "sgd", "batch_size": bs, "alpha": 0.0, "lr": 1e-3, "momentum": 0.0, "epochs": 1, "seed": 5}
    X, y, ft = bb.to_device(cfg)
    tr = bb.bbo_mlp_cv_eval(X, y, c, ft, 5, [hp], 0, trace=(0, 1, 0, 1))[-1]
    torch.cuda.synchronize()
    exact, sums = (oracle.train_one(cfg["X"], cfg["y"], c, cfg["fold_idx"], hp, 1, prec=p, step_begin=0, step_end=1)["grad"][0]
                   for p in (1, 2))
    for name, sl in layer_slices(d, [h], c):
        if name[0] != "W":
            continue
        want = exact[sl].astype(np.float64)
        off = lambda g: np.linalg.norm(g.astype(np.float64) - want) / np.linalg.norm(want)
        here, fp32 = off(tr["grad"][0, sl].cpu().numpy()), off(sums[sl])
        print("%s d %d h %d bs %d scale %g: %.2e, fp32 sums %.2e" % (name, d, h, bs, scale, here, fp32))
        assert here < 1.5 * fp32 + 2.0 ** -24, name
