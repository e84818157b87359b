"""GPU tests of the kernel for models that take all their rows in every step, at the edges of its shapes (tiles of 16 rows,
of 16 units, input columns with the bias, four and eight waves), against the CPU oracle."""
import pytest
import torch

from test_gpu_parity import ABS_SCORE, REL_F32, bb, forced_steps, layer_slices, relerr, small_problem  # noqa: F401

pytestmark = pytest.mark.gpu


# n, inputs, classes, hidden; batch 0, n or more: all rows.  The last ones belong to the kernel that walks chunks.
SHAPES = [(12, 1, 2, 1), (20, 4, 3, 16), (21, 5, 0, 17), (80, 15, 1, 48), (81, 15, 2, 33), (99, 7, 4, 48), (100, 3, 1, 49),
          (160, 16, 3, 16), (161, 31, 2, 32), (255, 2, 3, 48), (256, 2, 3, 64), (400, 30, 4, 20), (1200, 4, 2, 20),
          (99, 7, 2, 64), (161, 32, 2, 32), (161, 31, 2, 33)]


@pytest.mark.parametrize("n,d,c,h", SHAPES)
@pytest.mark.parametrize("solver", ["adam", "sgd"])
def test_steps_and_score(bb, oracle, n, d, c, h, solver):  # noqa: F811
    hp = {"hidden": [h], "solver": solver, "nesterov": True, "batch_size": 0 if solver == "adam" else n, "alpha": 0.3,
          "lr": 0.003, "momentum": 0.9, "epochs": 5, "seed": 7 + n}
    cfg = small_problem(n + d, n, d, c)
    f, T = 1, 5
    X, y, ft = bb.to_device(cfg)
    _, _, pf, tr = bb.bbo_mlp_cv_eval(X, y, c, ft, 5, [hp], 0, want_per_fold=True, trace=(0, f, 0, T))
    torch.cuda.synchronize()
    ref = oracle.train_one(cfg["X"], cfg["y"], c, cfg["fold_idx"], hp, f, step_begin=0, step_end=T)
    for t in range(T):
        assert abs(tr["loss"][t].item() - ref["loss"][t]) < 1e-4 * max(1.0, abs(ref["loss"][t]))
        for name, sl in layer_slices(d, [h], c if c >= 2 else 1):
            assert relerr(tr["grad"][t, sl].cpu(), ref["grad"][t, sl]) < REL_F32, (t, name, "grad")
            assert relerr(tr["theta_after"][t, sl].cpu(), ref["theta_after"][t, sl]) < REL_F32, (t, name, "theta")
    assert abs(pf[0, f, 0].item() - ref["scores"][0]) < ABS_SCORE
    for t, g, th, rg, rth in forced_steps(bb, oracle, cfg, hp, f, 0, [T - 1], T):
        for name, sl in layer_slices(d, [h], c if c >= 2 else 1):
            assert relerr(g[sl], rg[sl]) < REL_F32 and relerr(th[sl], rth[sl]) < REL_F32, (t, name)


@pytest.mark.parametrize("n,c", [(60, 3), (150, 2), (300, 1)])
@pytest.mark.parametrize("stop", [{}, {"n_iter_no_change": 2, "tol": 1e-4},
                                  {"n_iter_no_change": 2, "tol": 1e-4, "validation_fraction": 0.2}])
def test_one_launch_for_several_widths_gives_each_model_the_bits_of_its_own_call(bb, n, c, stop):  # noqa: F811
    cfg = small_problem(3, n, 6, c)
    X, y, ft = bb.to_device(cfg)
    hps = [dict({"hidden": [h], "batch_size": 0, "epochs": 12, "lr": 0.01, "seed": i}, **stop)
           for i, h in enumerate([8, 16, 17, 32, 40, 48, 5])]
    s, st = bb.bbo_mlp_cv_eval(X, y, c, ft, 5, hps, 0)
    many, _ = bb.bbo_mlp_cv_eval(X, y, c, ft, 5, hps * 20, 0)  # enough of them for a launch each
    for i, hp in enumerate(hps):
        s1, st1 = bb.bbo_mlp_cv_eval(X, y, c, ft, 5, [hp], 0)
        torch.cuda.synchronize()
        assert torch.equal(s[i], s1[0]) and torch.equal(many[i + 7], s1[0]) and torch.equal(st[i:i + 1], st1), hp


def test_a_row_of_nans_stays_out_of_the_training_of_models_that_do_not_train_on_it(bb):  # noqa: F811
    """Rows of the held fold lie beside the others in LDS, in no product of theirs; rows of no fold nowhere."""
    cfg = small_problem(5, 150, 4, 3)
    X, y, ft = bb.to_device(cfg)
    row = int((ft == 2).nonzero()[0])
    hp = [{"hidden": [20], "batch_size": 0, "epochs": 6, "lr": 0.01, "seed": 1}]
    theta = []
    for _ in range(2):  # fold 2's own model, without and with NaNs in a row that it is scored on
        tr = bb.bbo_mlp_cv_eval(X, y, 3, ft, 5, hp, 0, trace=(0, 2, 0, 6))[-1]
        theta.append(tr["theta_after"].clone())
        X[row] = float("nan")
    torch.cuda.synchronize()
    assert torch.equal(theta[0], theta[1]) and bool(torch.isfinite(theta[0]).all())
    ft[row] = -1
    with_nans, _ = bb.bbo_mlp_cv_eval(X, y, 3, ft, 5, hp, 0)
    X[row] = 0.0
    without, _ = bb.bbo_mlp_cv_eval(X, y, 3, ft, 5, hp, 0)
    torch.cuda.synchronize()
    assert torch.equal(with_nans, without)
