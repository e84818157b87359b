"""GPU tests of the fp32 kernel for several hidden layers at the edges of its cut (four or eight waves, input tiles, where
the moments live, ragged chunks and row tiles, levels of different width), against the CPU oracle."""
import pytest
import torch

from test_gpu_parity import ABS_SCORE, REL_F32, bb, forced_steps, layer_slices, relerr, small_problem  # noqa: F401

pytestmark = pytest.mark.gpu

# n, inputs, classes, hidden, batch: one shape on each side of every line; the last two go to the kernel for any shape
SHAPES = [
    (150, 4, 3, [16, 16], 0), (150, 16, 2, [17, 33], 16), (203, 17, 1, [64, 64], 17), (203, 30, 2, [64, 1], 48),
    (203, 32, 0, [1, 64], 65), (203, 33, 4, [65, 16], 64), (203, 48, 16, [128, 128], 100), (203, 64, 10, [16, 128], 1),
    (203, 49, 5, [50, 40], 33), (150, 8, 2, [16, 16, 16], 0), (203, 16, 1, [33, 64, 20], 50), (203, 30, 2, [64, 64, 64], 31),
    (203, 31, 0, [128, 128, 128], 130), (203, 47, 3, [20, 128, 50], 63), (203, 64, 16, [128, 16, 65], 80),
    (900, 60, 2, [128, 128, 128], 200), (5000, 9, 2, [24, 40], 900), (66000, 3, 2, [20, 20], 9000),
    (203, 65, 2, [40, 40], 64), (203, 30, 2, [129, 16], 64)]


@pytest.mark.parametrize("n,d,c,hidden,bs", SHAPES)
@pytest.mark.parametrize("solver", ["adam", "sgd"])
def test_steps_and_score_at_the_edges_of_a_cut(bb, oracle, n, d, c, hidden, bs, solver):  # noqa: F811
    hp = {"hidden": hidden, "solver": solver, "nesterov": True, "batch_size": bs, "alpha": 0.3, "lr": 0.003,
          "momentum": 0.9, "epochs": 2, "seed": 99 + n}
    edge = (n, d, c, hidden, bs) in SHAPES[-2:]
    assert bb.bbo_mlp_kernel_class(n, d, c, hp, 0) == (bb.KERNEL_GENERIC if edge else bb.KERNEL_DEEP)
    cfg = small_problem(n + d, n, d, c)
    c_out, f = c if c >= 2 else 1, 1
    n_tr = int((cfg["fold_idx"] != f).sum())
    T = min(6, 2 * -(-n_tr // (bs if 0 < bs <= n_tr else n_tr)))
    X, y, ft = bb.to_device(cfg)
    _, _, pf, tr = bb.bbo_mlp_cv_eval(X, y, c, ft, 5, [hp], 0, want_per_fold=True, trace=(0, f, 0, T))
    torch.cuda.synchronize()
    ref = oracle.train_one(cfg["X"], cfg["y"], c, cfg["fold_idx"], hp, f, step_begin=0, step_end=T)
    assert torch.allclose(tr["loss"].cpu().double(), torch.as_tensor(ref["loss"]).double(), rtol=1e-4)
    for t in range(T):
        for name, sl in layer_slices(d, hidden, c_out):
            assert relerr(tr["grad"][t, sl].cpu(), ref["grad"][t, sl]) < REL_F32, (t, name, "grad")
            assert relerr(tr["theta_after"][t, sl].cpu(), ref["theta_after"][t, sl]) < REL_F32, (t, name, "theta")
    assert abs(pf[0, f, 0].item() - ref["scores"][0]) < ABS_SCORE
    if T > 1:  # a run taken up from the oracle's parameters and moments
        for t, g, th, rg, rth in forced_steps(bb, oracle, cfg, hp, f, 0, [T - 1], T):
            for name, sl in layer_slices(d, hidden, c_out):
                assert relerr(g[sl], rg[sl]) < REL_F32 and relerr(th[sl], rth[sl]) < REL_F32, (t, name)


@pytest.mark.parametrize("hidden", [[20, 50], [100, 30], [64, 16, 33], [70, 128, 90]])
def test_early_stopping_hands_back_the_best_epoch(bb, hidden):  # noqa: F811
    """A run that stops some epochs after its best one on the held rows scores bit for bit as the run of that length."""
    cfg = small_problem(11, 400, 20, 2)
    X, y, ft = bb.to_device(cfg)
    E = 40
    hp = {"hidden": hidden, "batch_size": 50, "lr": 0.05, "alpha": 0.001, "epochs": E, "seed": 61,
          "validation_fraction": 0.15, "tol": 0.0, "n_iter_no_change": 3}
    _, _, pf = bb.bbo_mlp_cv_eval(X, y, 2, ft, 5, [dict(hp, epochs=e) for e in range(1, E + 1)], 0, want_per_fold=True)
    torch.cuda.synchronize()
    full = pf[E - 1, :, 0]
    first = [int((pf[:, f, 0] == full[f]).nonzero()[0]) + 1 for f in range(5)]
    assert all(e < E for e in first) and bool(torch.isfinite(full).all()), first


def test_a_zero_epsilon_leaves_the_pads_alone(bb, oracle):  # noqa: F811
    """Adam with eps = 0 divides 0 by 0 in pad elements: they must not reach the parameters."""
    cfg = small_problem(5, 203, 30, 3)
    X, y, ft = bb.to_device(cfg)
    for hidden in ([20, 50], [70, 33, 90]):
        hp = {"hidden": hidden, "batch_size": 64, "lr": 1e-3, "alpha": 0.1, "eps": 0.0, "epochs": 2, "seed": 4}
        _, _, pf = bb.bbo_mlp_cv_eval(X, y, 3, ft, 5, [hp], 0, want_per_fold=True)
        torch.cuda.synchronize()
        ref = oracle.train_one(cfg["X"], cfg["y"], 3, cfg["fold_idx"], hp, 0)
        assert abs(pf[0, 0, 0].item() - ref["scores"][0]) < 1e-2 * max(1.0, abs(ref["scores"][0])), hidden


@pytest.mark.parametrize("n,d,c,K,shapes,dtype", [
    (361, 20, 5, 3, [[125, 20]] * 40, 0), (78, 122, 2, 5, [[72]] * 40, 0),
    (64, 29, 0, 6, [[41, 75, 2]] * 16 + [[30]] * 16, 0), (80, 112, 10, 8, [[62], [30], [2], [2], [33, 14, 88], [10]], 1)])
def test_the_static_workspace_holds_these_calls_on_fewer_workgroups(bb, n, d, c, K, shapes, dtype):  # noqa: F811
    """Calls whose full plan is larger than the static array: fewer workgroups, or shared slots; the same bits."""
    cfg = small_problem(3, n, d, c, bf16=bool(dtype))
    cfg["fold_idx"] = (cfg["fold_idx"] * 0 + torch.arange(n).numpy() % K).astype("int32")
    X, y, ft = bb.to_device(cfg)
    hps = [{"hidden": h, "batch_size": 16, "epochs": 2, "seed": i} for i, h in enumerate(shapes)]
    s0, st0 = bb.bbo_mlp_cv_eval(X, y, c, ft, K, hps, dtype)
    s1 = torch.empty(len(hps), 2, device=X.device)
    st1 = torch.empty(len(hps), dtype=torch.int32, device=X.device)
    bb.bbo_mlp_cv_eval_static(X, y, c, ft, K, hps, dtype, scores=s1, status=st1)
    torch.cuda.synchronize()
    assert torch.equal(s0, s1) and torch.equal(st0, st1)
