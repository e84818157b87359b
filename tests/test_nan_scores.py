"""A NaN in the data reaches the score of every model that meets it, whichever kernel the model runs on, and no other model's."""
import pytest
import torch

from test_gpu_parity import bb, small_problem  # noqa: F401

pytestmark = pytest.mark.gpu

# inputs, classes, hidden, batch, dtype: fp32 and split products of each register-resident kernel, both sides of the line between
# them, the full-batch kernel, two and three hidden layers, no hidden layer, any shape, bfloat16
SHAPES = [(10, 2, [20], 24, 0), (30, 2, [20], 24, 0), (30, 2, [100], 24, 0), (30, 1, [130], 64, 0), (40, 3, [50], 40, 0),
          (60, 2, [64], 64, 0), (60, 3, [64], 64, 0), (4, 3, [20], 0, 0), (30, 2, [40], 0, 0), (20, 0, [17], 0, 0),
          (64, 10, [40], 32, 0), (64, 10, [100], 32, 0), (64, 10, [200], 64, 0), (64, 10, [200], 96, 0), (100, 5, [64], 32, 0),
          (30, 2, [40, 24], 24, 0), (30, 3, [100, 90], 24, 0), (20, 2, [70, 128, 30], 40, 0), (30, 2, [], 24, 0), (64, 10, [], 24, 0),
          (30, 2, [300], 24, 0), (70, 2, [40, 24], 0, 0), (64, 10, [128, 128], 64, 1), (64, 10, [256], 300, 1), (30, 2, [40, 24], 24, 1)]


@pytest.mark.parametrize("d,c,hidden,batch,dtype", SHAPES)
@pytest.mark.parametrize("row", [0, 77])
def test_a_nan_in_a_row(bb, d, c, hidden, batch, dtype, row):  # noqa: F811
    cfg = small_problem(5 + d, 230, d, c, bf16=bool(dtype))
    X, y, ft = bb.to_device(cfg)
    f = int(ft[row])
    # the second model trains on no row: only the fold that holds the row meets its NaN
    hps = [{"hidden": hidden, "batch_size": batch, "epochs": e, "lr": 0.01, "seed": 3} for e in (2, 0)]
    X[row, d // 2] = float("nan")
    scores, status, pf = bb.bbo_mlp_cv_eval(X, y, c, ft, 5, hps, dtype, want_per_fold=True)
    torch.cuda.synchronize()
    assert status.tolist() == [1, 1] and bool(torch.isnan(scores[:, 0]).all())
    assert bool(torch.isnan(pf[0, :, 0]).all())
    assert [bool(x) for x in torch.isnan(pf[1, :, 0])] == [k == f for k in range(5)]
    ft[row] = -1
    scores, status = bb.bbo_mlp_cv_eval(X, y, c, ft, 5, hps, dtype)
    X[row] = 0.0
    without, _ = bb.bbo_mlp_cv_eval(X, y, c, ft, 5, hps, dtype)
    torch.cuda.synchronize()
    assert status.tolist() == [0, 0] and torch.equal(scores, without)


@pytest.mark.parametrize("d,c,hidden,batch,dtype", SHAPES)
def test_an_eps_of_zero_moves_no_parameter_without_a_gradient(bb, d, c, hidden, batch, dtype):  # noqa: F811
    """A column of zeros and no penalty: its weights never have a gradient, and Adam's 0 / 0 is no step."""
    cfg = small_problem(7 + d, 230, d, c, bf16=bool(dtype))
    cfg["X"][:, 1] = 0
    X, y, ft = bb.to_device(cfg)
    hp = {"hidden": hidden, "batch_size": batch, "epochs": 3, "lr": 1e-3, "alpha": 0.0, "eps": 0.0, "seed": 3}
    scores, status, _, tr = bb.bbo_mlp_cv_eval(X, y, c, ft, 5, [hp], dtype, want_per_fold=True, trace=(0, 1, 0, 3))
    _, untraced = bb.bbo_mlp_cv_eval(X, y, c, ft, 5, [hp] * 3, dtype)
    first = bb.bbo_mlp_init_params(d, c, hp, 1)
    torch.cuda.synchronize()
    assert status.tolist() == [0] and untraced.tolist() == [0] * 3 and bool(torch.isfinite(scores).all())
    out = hidden[0] if hidden else max(c, 1)
    after = tr["theta_after"]
    assert bool(torch.isfinite(after).all())
    assert torch.equal(after[:, out:2 * out], first[out:2 * out].expand(3, out))
    assert not torch.equal(after[0, :out], first[:out])
