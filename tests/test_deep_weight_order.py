"""Hidden weights that waves of the kernel for several hidden layers share through global memory: a step's data gradient
reads all of them before its update stores the next ones."""
import os
import re
import shutil
import subprocess

import pytest
import torch

from test_gpu_parity import ABS_SCORE, REL_F32, bb, layer_slices, relerr, small_problem  # noqa: F401
from test_wide_stores import CSRC


def weight_stores(listing):
    """{(input tiles, hidden layers, waves): (the updates' stores of hidden weights, those behind a fetch of weights with no
    barrier between, how many stores stand in front of each barrier)}.  The backward pass fetches 16 bytes a lane through
    pointers.  With three hidden layers on eight waves the update stores 4 bytes a lane through its descriptor; with two,
    through pointers behind the moments' 16-byte stores."""
    out, name = {}, None
    for line in listing.split("\n"):
        m = re.match(r"_ZN\S*k_train_deepILi(\d)ELi(\d)ELi(\d)E\S*:", line)
        if m:
            name, stores, bad, ahead, fetched, update = tuple(int(x) for x in m.groups()), 0, 0, set(), False, False
        elif name and line.startswith(".Lfunc_end"):
            out[name] = (stores, bad, ahead)
            name = None
        elif name and line.split():
            op, streamed = line.split()[0], name[1:] == (3, 8)
            fetched = op == "global_load_dwordx4" or fetched and op != "s_barrier"
            update = op == "buffer_store_dwordx4" or update and not op.startswith("v_mfma")
            if op == "s_barrier":
                ahead.add(stores)
            if op == "buffer_store_dword" if streamed else update and op == "global_store_dword":
                stores += 1
                bad += fetched
    return out


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not on PATH")
def test_a_barrier_parts_the_backward_pass_from_the_weights_stores(tmp_path):
    """On eight waves: the waves of the first level fetch out tiles 4.. of the layer above behind the last barrier inside the
    backward pass, and without one more the waves that own these tiles may be past their update's arithmetic by then."""
    kinds = [(1, 2, 8), (1, 3, 8)]
    src, out = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text('#include "%s"\nnamespace {\n%s}\n' % (
        os.path.join(CSRC, "train_deep_f32.h"),
        "".join("template __global__ void k_train_deep<%d, %d, %d>(const TrainParams);\n" % k for k in kinds)))
    cmd = ["hipcc", "-O3", "--offload-arch=gfx950", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "--cuda-device-only", "-S", str(src), "-o", str(out)]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    found = weight_stores(out.read_text())
    assert sorted(found) == kinds
    stores, bad, _ = found[1, 2, 8]
    assert stores >= 8 * 4 and bad == 0, (stores, bad)
    # for each solver 8 blocks of 4 values of the upper layer, which need no barrier of their own, then layer 1's
    stores, _, ahead = found[1, 3, 8]
    assert stores == 128 and {32, 96} <= ahead, (stores, ahead)


# A first level of one tile below one of eight, and more than 32 rows in the last chunk of every step: the reader has the
# longest way to its fetch, the owners of the tiles the shortest to their stores.
@pytest.mark.gpu
@pytest.mark.parametrize("d,c,hidden", [(10, 2, [16, 128, 16]), (10, 3, [16, 128]), (60, 1, [5, 100, 128])])
@pytest.mark.parametrize("solver", ["adam", "sgd"])
def test_a_narrow_level_below_a_wide_one(bb, oracle, d, c, hidden, solver):  # noqa: F811
    hp = {"hidden": hidden, "solver": solver, "nesterov": True, "batch_size": 64, "alpha": 0.3, "lr": 0.003, "momentum": 0.9,
          "epochs": 2, "seed": 5}
    cfg = small_problem(31 + d, 203, d, c)
    X, y, ft = bb.to_device(cfg)
    ref = [oracle.train_one(cfg["X"], cfg["y"], c, cfg["fold_idx"], hp, f) for f in range(5)]
    _, _, alone = bb.bbo_mlp_cv_eval(X, y, c, ft, 5, [hp], 0, want_per_fold=True)  # (no step is traced)
    _, _, many = bb.bbo_mlp_cv_eval(X, y, c, ft, 5, [hp] * 300, 0, want_per_fold=True)
    torch.cuda.synchronize()
    assert torch.equal(many, alone.expand_as(many))
    for f in range(5):
        assert abs(alone[0, f, 0].item() - ref[f]["scores"][0]) < ABS_SCORE
    T = 4
    tr = bb.bbo_mlp_cv_eval(X, y, c, ft, 5, [hp], 0, trace=(0, 1, 0, T))[-1]
    torch.cuda.synchronize()
    steps = oracle.train_one(cfg["X"], cfg["y"], c, cfg["fold_idx"], hp, 1, step_begin=0, step_end=T)
    for t in range(T):
        for name, sl in layer_slices(d, hidden, c if c >= 2 else 1):
            assert relerr(tr["theta_after"][t, sl].cpu(), steps["theta_after"][t, sl]) < REL_F32, (t, name)
