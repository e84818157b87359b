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
    each = max(1, min(8, CUS // 2 // 8 // -(-models // 8)))  # half of the CUs: the others are other callers'
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
            got.append([rc] + [int(l[2]) for l in log() if l[0] == "launch" and "k_train_tiled" in l[5]])
        print(json.dumps(got))
    """ % models)
    for (n, batch), got in zip(((1000, 64), (1000, 256), (1000, 257), (1000, 0), (256, 0), (256, 500)), grids):
        assert got == [0, expected(models, n, batch)], (n, batch, got)
        assert got[1] == models or got[1] <= CUS // 2


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
    assert alone == 40 and grids == [40, 40 * 3, 40 * 3], (least, alone, grids)


# rows, inputs, classes, folds, models; a few small ones, whose weights a CU's vector cache holds from step to step
CASES = [(300, 16, 0, 3, 1), (300, 8, 1, 2, 2), (700, 128, 10, 5, 3), (400, 200, 2, 5, 13), (1000, 256, 16, 4, 30),
         (400, 200, 2, 4, 15), (1000, 256, 16, 4, 8), (700, 136, 7, 3, 7)]


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


def teams_of(workspace, models):
    """(members, meetings of each) per model, from the control blocks that a call leaves in its workspace: 16 words a team, the
    list (four bits a member, 8 | its XCD, the leader's first; the highest bit says that it is closed) and from the ninth on how
    many meetings each member has come to."""
    w = workspace.cpu().numpy().view(np.uint32)
    w = w[:w.size // 16 * 16].reshape(-1, 16)
    closed = (w[:, 1] == 0x80000000) & (w[:, 0] & 8 > 0) & (w[:, 2] == 0)
    first = next(i for i in range(len(w)) if closed[i:i + models].all() and closed[i:i + models].size == models)
    out = []
    for block in w[first:first + models]:
        nibbles = [int(block[0]) >> 4 * k & 15 for k in range(8)]
        members = sum(x == nibbles[0] for x in nibbles)
        out.append((members, [int(x) for x in block[8:8 + members]]))
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("models", [1, 8, 30, 64])
def test_teams_form_and_meet_after_every_step(bb, models):  # noqa: F811
    """On a device without other work.  (Two meetings before the first step; one that is alone has none.)"""
    n, d, c = 400, 64, 3
    fold = np.where(np.arange(n) < 100, 0, 1).astype(np.int32)  # one fold of 300 training rows
    X, y, ft = bb.to_device(dict(small_problem(5, n, d, c, bf16=True), n_folds=1, fold_idx=fold))
    hps = [{"hidden": [100 + i % 50], "batch_size": 64, "epochs": 3, "seed": i} for i in range(models)]
    need = bb.bbo_mlp_workspace_bytes(n, d, c, 1, hps, bb.BF16)
    ws = torch.zeros(need, dtype=torch.uint8, device=X.device)
    bb.bbo_mlp_cv_eval(X, y, c, ft, 1, hps, bb.BF16, workspace=ws)
    torch.cuda.synchronize()
    teams = teams_of(ws, models)
    steps = 3 * -(-300 // 64)
    print("members", sorted({m for m, _ in teams}))
    assert all(m >= 2 for m, _ in teams)
    assert all(met == [2 + steps] * m for m, met in teams), teams


@pytest.mark.gpu
def test_calls_at_once_change_no_bit(bb):  # noqa: F811
    """Four calls on streams of their own, whose teams together ask for more workgroups than there are CUs: some come late."""
    n, d, c, K = 600, 64, 4, 4
    X, y, ft = bb.to_device(dict(small_problem(9, n, d, c, bf16=True), n_folds=K, fold_idx=np.arange(n, dtype=np.int32) % K))
    calls = [[{"hidden": [40 + 31 * i % 200] * (1 + i % 2), "batch_size": 64, "epochs": 4, "seed": 100 * j + i, "alpha": 0.1}
              for i in range(10)] for j in range(4)]
    alone = [bb.bbo_mlp_cv_eval(X, y, c, ft, K, hps, bb.BF16, want_per_fold=True)[2] for hps in calls]
    rooms = [torch.empty(bb.bbo_mlp_workspace_bytes(n, d, c, K, hps, bb.BF16), dtype=torch.uint8, device=X.device) for hps in calls]
    streams = [torch.cuda.Stream() for _ in calls]
    torch.cuda.synchronize()
    for _ in range(3):
        got = []
        for hps, room, s in zip(calls, rooms, streams):
            with torch.cuda.stream(s):
                got.append(bb.bbo_mlp_cv_eval(X, y, c, ft, K, hps, bb.BF16, want_per_fold=True, workspace=room)[2])
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(alone, got))
