"""GPU test: a call on the static workspace whose suggestions need several kernels, captured into a graph."""
import pytest
import torch

from test_gpu_parity import bb, small_problem  # noqa: F401

pytestmark = pytest.mark.gpu


def test_mixed_shapes_captured_and_replayed(bb):  # noqa: F811
    cfg = small_problem(7, 300, 30, 3)
    X, y, ft = bb.to_device(cfg)
    hps = [{"hidden": h, "batch_size": 48, "epochs": 2, "lr": 0.003, "seed": i}
           for i, h in enumerate([[20], [100], [], [40, 30], [70, 20]])]
    s = torch.empty(len(hps), 2, device=X.device)
    st = torch.empty(len(hps), dtype=torch.int32, device=X.device)
    bb.bbo_mlp_cv_eval_static(X, y, 3, ft, 5, hps, 0, scores=s, status=st)
    torch.cuda.synchronize()
    want, want_st = s.clone(), st.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        bb.bbo_mlp_cv_eval_static(X, y, 3, ft, 5, hps, 0, scores=s, status=st)
    for _ in range(4):
        s.fill_(-7.0)
        st.fill_(-7)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(s, want) and torch.equal(st, want_st)
        bb.bbo_mlp_cv_eval(X, y, 3, ft, 5, hps[:2], 0)  # the program's own eager work between the replays
        torch.cuda.synchronize()
