"""What a workspace of a given size holds: calls that were taken before kernels came with more workgroups a CU or larger slots."""
import pytest
import torch

from test_gpu_parity import bb, small_problem  # noqa: F401
from test_host_launches import child  # noqa: F401

# rows, inputs, classes, folds, suggestions: two workgroups of these three layers share a CU ...
DEEP = [(150, 64, 3, 5, [[64, 64, 64]] * 400), (150, 64, 2, 5, [[48, 48, 48]] * 400),
        (659, 34, 10, 5, [[64 - i % 3, 64, 64 - i % 5] for i in range(388)]), (820, 47, 3, 5, [[34, 64, 1]] * 86)]
# ... and models of one layer keep more of their state in the slot past 64 rows a step
MID = [(200000, 64, 10, 5, [[200]] * 60), (530000, 40, 7, 5, [[256]] * 60)]


@pytest.mark.parametrize("n,d,c,K,shapes", DEEP + MID)
@pytest.mark.parametrize("batch", [0, 32, 200])
def test_the_static_workspace_holds_these_calls(child, n, d, c, K, shapes, batch):  # noqa: F811
    rc, grids = child("""
        n, d, c, K, shapes, batch = %r
        rc = L.bbo_mlp_cv_eval_static(P(4096), P(4096), C.c_int64(n), d, c, P(4096), K, records(shapes, batch), len(shapes), 0,
                                      P(4096), P(4096), P(0), P(900))
        print(json.dumps([rc, [int(l[2]) for l in log() if l[0] == "launch"]]))
    """ % ((n, d, c, K, shapes, batch),))
    assert rc == 0 and max(grids) >= 64


# two unit tiles a wave, two to five input tiles: split products past 64 or 95 rows a step, and a larger slot with three and four
@pytest.mark.parametrize("n,d,c,h", [(1797, 64, 10, 200), (40, 47, 10, 256), (453, 45, 10, 130), (273, 60, 7, 254), (300, 20, 5, 150),
                                     (300, 80, 5, 150)])
@pytest.mark.parametrize("count,folds", [(1, 1), (1, 3), (40, 5), (300, 5)])
def test_a_workspace_holds_the_same_models_at_any_batch_size(child, n, d, c, h, count, folds):  # noqa: F811
    sizes, grids = child("""
        n, d, c, h, count, K = %r
        shapes, batches = [[h - 30 * (i %% 2)] for i in range(count)], (0, 1, 32, 64, 65, 95, 96)
        sizes, grids = [], []
        for made in batches:
            out = C.c_size_t(0)
            assert L.bbo_mlp_workspace_bytes(C.c_int64(n), d, c, K, records(shapes, made), count, 0, C.byref(out)) == 0
            sizes.append(out.value)
            log()
            rcs = [L.bbo_mlp_cv_eval(P(4096), P(4096), C.c_int64(n), d, c, P(4096), K, records(shapes, b), count, 0, P(4096),
                                     P(4096), P(0), P(4096), out, P(900)) for b in batches]
            assert rcs == [0] * 7, (made, rcs)
            grids.append([int(l[2]) for l in log() if l[0] == "launch"])
        print(json.dumps([sizes, grids]))
    """ % ((n, d, c, h, count, folds),))
    assert all(g == grids[0] for g in grids) and len(set(sizes)) == 1, sizes  # and on as many workgroups


@pytest.mark.gpu
def test_fewer_workgroups_give_the_same_bits(bb):  # noqa: F811
    n, d, c, K, shapes = DEEP[0]
    cfg = small_problem(3, n, d, c)
    X, y, ft = bb.to_device(cfg)
    hps = [{"hidden": h, "batch_size": 40, "epochs": 1, "seed": i} for i, h in enumerate(shapes)]
    s0, st0 = bb.bbo_mlp_cv_eval(X, y, c, ft, K, hps, 0)
    s1 = torch.empty(len(hps), 2, device=X.device)
    st1 = torch.empty(len(hps), dtype=torch.int32, device=X.device)
    bb.bbo_mlp_cv_eval_static(X, y, c, ft, K, hps, 0, scores=s1, status=st1)
    torch.cuda.synchronize()
    assert torch.equal(s0, s1) and torch.equal(st0, st1)
