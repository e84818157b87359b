"""Several workgroups that train one bf16 model together: which calls get them, and that they change no bit of a score."""
import numpy as np
import pytest
import torch

from test_gpu_parity import bb, small_problem  # noqa: F401
from test_host_launches import child  # noqa: F401

CUS = 256


def expected(models, n, batch):
    """(workgroups, of which each model has)"""
    if batch == 0 and n > 256 or batch > 256 and n > 256:
        return min(models, CUS)
    each = max(1, min(8, CUS // 8 // -(-models // 8)))
    return models if each == 1 else -(-models // 8) * 8 * each


@pytest.mark.parametrize("models", [1, 3, 8, 9, 16, 40, 64, 65, 96, 127, 128, 129, 200, 256])
def test_workgroups_of_a_call(child, models):  # noqa: F811
    grids = child("""
        got = []
        for n, batch in ((1000, 64), (1000, 256), (1000, 257), (1000, 0), (256, 0), (256, 500)):
            shapes = [[200, 130 + i %% 9] for i in range(%d)]
            log()
            rc = L.bbo_mlp_cv_eval(P(4096), P(4096), C.c_int64(n), 128, 10, P(4096), 1, records(shapes, batch), len(shapes), 1,
                                   P(4096), P(4096), P(0), P(4096), C.c_size_t(1 << 40), P(900))
            got.append([rc] + [int(l[2]) for l in log() if l[0] == "launch"])
        print(json.dumps(got))
    """ % models)
    for (n, batch), got in zip(((1000, 64), (1000, 256), (1000, 257), (1000, 0), (256, 0), (256, 500)), grids):
        assert got[0] == 0 and expected(models, n, batch) in got[1:], (n, batch, got)


def test_no_room_for_the_control_blocks_no_team(child):  # noqa: F811
    """The least workspace that holds a call gives every model one workgroup, as many bytes more as its team meets at a team."""
    least, alone, grids = child("""
        shapes = [[200, 130]] * 20
        def grid(room):
            log()
            rc = L.bbo_mlp_cv_eval(P(4096), P(4096), C.c_int64(1000), 128, 10, P(4096), 2, records(shapes, 64), len(shapes), 1,
                                   P(4096), P(4096), P(0), P(4096), C.c_size_t(room), P(900))
            return [int(l[2]) for l in log() if l[0] == "launch"][1] if rc == 0 else 0
        lo, hi = 0, 1 << 40
        while hi - lo > 1:
            mid = (lo + hi) // 2
            lo, hi = (lo, mid) if grid(mid) else (mid, hi)
        print(json.dumps([hi, grid(hi), [grid(hi + 64 * 40 - 1), grid(hi + 64 * 40), grid(need(1000, 128, 10, 2, shapes, 1))]]))
    """)
    assert alone == 40 and grids == [40, 40 * 6, 40 * 6], (least, alone, grids)


# rows, inputs, classes, folds, models; a few small ones, whose weights a CU's vector cache holds from step to step
CASES = [(300, 16, 0, 3, 1), (300, 8, 1, 2, 2), (700, 128, 10, 5, 3), (400, 200, 2, 5, 13), (1000, 256, 16, 4, 30)]


@pytest.mark.gpu
@pytest.mark.parametrize("n,d,c,K,models", CASES)
def test_a_team_changes_no_bit(bb, n, d, c, K, models):  # noqa: F811
    """The same suggestions in a call that has a CU for each of its models at most."""
    X, y, ft = bb.to_device(dict(small_problem(11, n, d, c, bf16=True), n_folds=K, fold_idx=np.arange(n, dtype=np.int32) % K))
    hps = [{"hidden": [[17 + 31 * i % 240], [128 + 13 * i % 120, 40 + 29 * i % 210], [256, 256], [33, 256]][i % 4],
            "batch_size": [64, 33, 256, 100, 200][i % 5], "epochs": 3, "lr": 1e-3, "alpha": 0.1, "seed": 7 + i,
            "solver": "sgd" if i % 7 == 6 else "adam", "nesterov": True, "n_iter_no_change": i % 3 // 2, "tol": 1e-3}
           for i in range(models)]
    many = hps + [dict(hps[i % models], seed=1000 + i) for i in range(130)]
    apart = bb.bbo_mlp_cv_eval(X, y, c, ft, K, many, bb.BF16, want_per_fold=True)[2][:models]
    for _ in range(3):
        together = bb.bbo_mlp_cv_eval(X, y, c, ft, K, hps, bb.BF16, want_per_fold=True)[2]
        assert torch.equal(together, apart)
