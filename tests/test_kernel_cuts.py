"""GPU tests of the cuts the fp32 kernels make of a model (unit tiles per wave, waves, input tiles, where the moments
live, which row tables fit), at the edges of each cut, against the CPU oracle."""
import pytest
import torch

from test_gpu_parity import ABS_SCORE, REL_F32, bb, forced_steps, layer_slices, relerr, small_problem  # noqa: F401

pytestmark = pytest.mark.gpu

# n, inputs, classes, hidden, batch: one shape on each side of every line
ONE_SMALL_LAYER = [
    (150, 16, 2, [32], 0), (150, 17, 1, [33], 64), (203, 32, 3, [64], 65), (203, 15, 2, [193], 63), (203, 32, 1, [224], 1),
    (203, 33, 4, [128], 48), (203, 48, 2, [129], 80), (300, 49, 1, [64], 128), (300, 63, 3, [65], 17), (300, 63, 2, [130], 64),
    (4096, 8, 2, [16], 500), (4097, 8, 1, [16], 500), (40000, 3, 2, [24], 4000), (66000, 3, 2, [24], 9000)]
WIDE_HEAD = [
    (150, 16, 5, [64], 0), (150, 5, 16, [65], 33), (203, 48, 7, [129], 64), (203, 64, 10, [128], 63), (203, 64, 2, [129], 65),
    (203, 65, 12, [128], 17), (203, 80, 10, [256], 100), (203, 96, 1, [200], 80), (203, 97, 3, [64], 50), (203, 112, 0, [128], 64),
    (203, 127, 16, [16], 1), (203, 127, 10, [128], 90), (5000, 64, 10, [40], 1000), (66000, 6, 5, [24], 9000)]
# (the last two of each: the data set no longer fits into LDS, too many inputs)
LINEAR = [(n, d, c, [], bs) for c in (0, 1, 2) for n, d, bs in (
    (150, 7, 0), (151, 8, 17), (203, 15, 64), (203, 16, 1), (300, 31, 65), (300, 32, 130), (520, 47, 33), (520, 55, 200),
    (520, 60, 63), (400, 63, 128), (1500, 7, 700), (4000, 30, 900), (203, 64, 50))]


@pytest.mark.parametrize("n,d,c,hidden,bs", ONE_SMALL_LAYER + WIDE_HEAD + LINEAR)
@pytest.mark.parametrize("solver", ["adam", "sgd"])
def test_steps_and_score_at_the_edges_of_a_cut(bb, oracle, n, d, c, hidden, bs, solver):  # noqa: F811
    hp = {"hidden": hidden, "solver": solver, "nesterov": True, "batch_size": bs, "alpha": 0.3, "lr": 0.003,
          "momentum": 0.9, "epochs": 2, "seed": 99 + n}
    cls = bb.bbo_mlp_kernel_class(n, d, c, hp, 0)
    assert cls == (bb.KERNEL_LINEAR if not hidden else
                   bb.KERNEL_SMALL if (n, d, c, hidden, bs) in ONE_SMALL_LAYER else bb.KERNEL_MID)
    cfg = small_problem(n + d, n, d, c)
    c_out, f = c if c >= 2 else 1, 1
    n_tr = int((cfg["fold_idx"] != f).sum())
    T = min(6, 2 * -(-n_tr // (bs if 0 < bs <= n_tr else n_tr)))
    X, y, ft = bb.to_device(cfg)
    _, _, pf, tr = bb.bbo_mlp_cv_eval(X, y, c, ft, 5, [hp], 0, want_per_fold=True, trace=(0, f, 0, T))
    torch.cuda.synchronize()
    ref = oracle.train_one(cfg["X"], cfg["y"], c, cfg["fold_idx"], hp, f, step_begin=0, step_end=T)
    for t in range(T):
        for name, sl in layer_slices(d, hidden, c_out):
            assert relerr(tr["grad"][t, sl].cpu(), ref["grad"][t, sl]) < REL_F32, (t, name, "grad")
            assert relerr(tr["theta_after"][t, sl].cpu(), ref["theta_after"][t, sl]) < REL_F32, (t, name, "theta")
    assert abs(pf[0, f, 0].item() - ref["scores"][0]) < ABS_SCORE
    if T > 1:  # a run taken up from the oracle's parameters and moments
        for t, g, th, rg, rth in forced_steps(bb, oracle, cfg, hp, f, 0, [T - 1], T):
            for name, sl in layer_slices(d, hidden, c_out):
                assert relerr(g[sl], rg[sl]) < REL_F32 and relerr(th[sl], rth[sl]) < REL_F32, (t, name)


def test_variants_side_by_side_score_as_alone(bb):  # noqa: F811
    """One call with many kernel variants (more than there are streams for them): the bits of each suggestion's own call."""
    cfg = small_problem(7, 400, 40, 7)
    X, y, ft = bb.to_device(cfg)
    hps = [{"hidden": h, "batch_size": 48, "epochs": 3, "lr": 0.003, "seed": i}
           for i, h in enumerate([[20], [64], [100], [130], [250], [], [300], [40, 30], [64, 64, 64], [16] * 4] * 3)]
    for _ in range(3):
        s, st = bb.bbo_mlp_cv_eval(X, y, 7, ft, 5, hps, 0)
        for i in range(10):
            s1, st1 = bb.bbo_mlp_cv_eval(X, y, 7, ft, 5, [hps[i]], 0)
            torch.cuda.synchronize()
            assert torch.equal(s[i], s1[0]) and torch.equal(st[i:i + 1], st1), hps[i]


@pytest.mark.parametrize("n,d,c,widest,narrower,dtype", [
    (300, 30, 2, [224], [[20 + 5 * i % 205] for i in range(256)], 0),
    (300, 30, 2, [224], [[192]] * 256, 0),
    (200, 64, 10, [256], [[20 + 7 * i % 230] for i in range(120)], 0),
    (200, 30, 2, [128, 128, 128], [[128, 128, 128], [64, 60, 64]] * 60, 0),
    (200, 24, 3, [300, 200], [[300, 200], [250, 150], [40, 24], []] * 40, 0),
    (300, 64, 10, [256, 256], [[256, 256], [256, 128], [64, 64], []] * 20, 1)])
def test_a_workspace_for_the_widest_models_gives_a_narrower_mix_the_same_bits(bb, n, d, c, widest, narrower, dtype):  # noqa: F811
    cfg = small_problem(9, n, d, c, bf16=bool(dtype))
    X, y, ft = bb.to_device(cfg)
    hps = [{"hidden": h, "batch_size": 50, "epochs": 1, "lr": 0.003, "seed": i} for i, h in enumerate(narrower)]
    want, want_st = bb.bbo_mlp_cv_eval(X, y, c, ft, 5, hps, dtype)
    size = bb.bbo_mlp_workspace_bytes(n, d, c, 5, [dict(h, hidden=widest) for h in hps], dtype)
    ws = bb.alloc_workspace(size + 4096, X.device)
    ws[size:] = 0xA5  # what lies behind the workspace stays as it is
    for _ in range(2):
        s, st = bb.bbo_mlp_cv_eval(X, y, c, ft, 5, hps, dtype, workspace=ws[:size])
        torch.cuda.synchronize()
        assert torch.equal(s, want) and torch.equal(st, want_st) and bool((ws[size:] == 0xA5).all())
