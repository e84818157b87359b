"""Static checks of the built kernels (no GPU needed): which variants there are, and the loop nest of the
wavefront-per-model kernel's generated code.

Every wavefront of that kernel pops its next model from the work queue with all 64 lanes taking part.
A pop under `if (lane == 0)` compiled into a kernel that never ended: the loop body finishes with
another branch on the same condition, the compiler joined the two across the back edge, and lanes
1..63 went round the loop on their own, past the pop.  In the generated code that shows as one more
loop level around the per-model body.  This test compiles two variants of the kernel to assembly and
checks that the loop nest is as deep as the source's (queue, epoch, step, chunk, inner loop) and no
deeper."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2012_04201_amd", "csrc")


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not on PATH")
def test_linear_kernel_loop_nest_is_the_sources(tmp_path):
    src = tmp_path / "probe.hip"
    src.write_text('#include "%s"\nnamespace {\n'
                   "template __global__ void k_train_linear<2, 1>(const TrainParams);\n"
                   "template __global__ void k_train_linear<16, 1>(const TrainParams);\n}\n"
                   % os.path.join(CSRC, "train_linear_f32.h"))
    out = tmp_path / "probe.s"
    cmd = ["hipcc", "-O3", "--offload-arch=gfx950", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "--cuda-device-only", "-S", str(src), "-o", str(out)]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    lines = out.read_text().split("\n")
    starts = [i for i, l in enumerate(lines) if "k_train_linear" in l and l.startswith("_Z") and ":" in l]
    assert len(starts) == 2
    for s in starts:
        e = next(i for i in range(s, len(lines)) if lines[i].startswith(".Lfunc_end"))
        depth = [int(m.group(1)) for l in lines[s:e] for m in [re.search(r"Loop Header: Depth=(\d+)", l)] if m]
        assert depth, "no loops found: the listing's annotations changed"
        # queue loop 1, epoch 2, step 3, chunk 4, the chunk's inner loops 5
        assert max(depth) == 5, depth
        body = "\n".join(lines[s:e])
        assert "global_atomic_add" in body and "s_endpgm" in body


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not on PATH")
def test_a_team_drops_the_lines_of_its_cache_before_the_first_step(tmp_path):
    """Zeros and initial values are written by any member and read by a tile's owner with ordinary loads: its CU's vector cache is
    invalidated in between, once, by the workgroup-scope instruction (the agent's drops lines of the L2 too)."""
    out = tmp_path / "tiled.s"
    cmd = ["hipcc", "-O3", "--offload-arch=gfx950", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "--cuda-device-only", "-S", os.path.join(CSRC, "kernels_tiled.hip"), "-o", str(out)]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    text = out.read_text()
    found = {}
    for name in re.findall(r"^(_Z\w*k_train_tiled\w*):", text, re.M):
        body = text[text.index("\n" + name + ":"):]
        body = body[:body.index(".Lfunc_end")]
        found["team" in name] = re.findall(r"buffer_inv (.*)", body)
    assert found == {False: [], True: ["sc0"]}


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not on PATH")
@pytest.mark.parametrize("cut,most", [("3, 2, 8", 12), ("2, 3, 8", 4)])
def test_deep_kernels_on_eight_waves_keep_their_registers(tmp_path, cut, most):
    """<3, 2, 8>: the branch that parts the update's blocks is what keeps its registers; with another form of its condition the
    compiler spilled 25 vector registers instead of 8 (569 x 40, 100-70, 24 rows a step 3302 -> 3580 us a call).  <2, 3, 8>: what
    few steps do is marked as rare and spills there; 8 registers where it is not (569 x 30, 128-100-60 5229 -> 5880)."""
    src = tmp_path / "probe.hip"
    src.write_text('#include "%s"\nnamespace {\ntemplate __global__ void k_train_deep<%s>(const TrainParams);\n}\n'
                   % (os.path.join(CSRC, "train_deep_f32.h"), cut))
    cmd = ["hipcc", "-O3", "--offload-arch=gfx950", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "--cuda-device-only", "-c", "-Rpass-analysis=kernel-resource-usage", str(src), "-o", os.devnull]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    spilled = [int(x) for x in re.findall(r"VGPRs Spill: (\d+)", res.stderr)]
    assert len(spilled) == 1 and spilled[0] <= most, spilled


@pytest.mark.skipif(shutil.which("nm") is None, reason="nm not on PATH")
def test_the_library_holds_the_variants_that_the_cuts_can_ask_for():
    """The register-resident kernels are compiled for each way a model of their shapes is cut, and for no other."""
    lib = os.path.join(ROOT, "paper_2012_04201_amd", "libbbo_mlp.so")
    if not os.path.exists(lib):
        from paper_2012_04201_amd import build
        build.build_lib()
    names = subprocess.run(["nm", "-C", lib], capture_output=True, text=True, check=True).stdout
    built = lambda k: sorted(tuple(int(x) for x in m.split(",")) for m in
                             re.findall(r"__device_stub__k_train_%s<([0-9, ]+)>" % k, names))
    tiles = lambda x: -(-x // 16)
    small, mid = set(), set()
    for d in range(1, 128):
        for h in range(1, 257):
            kt, nut = tiles(d), tiles(h)
            for c in (1, 2, 4):
                if d <= 63 and h <= 224:
                    per_wave = 1 if kt == 4 else (2 if kt == 3 or c == 4 else 3)
                    waves = 2 if kt == 1 and nut <= 2 else 4
                    waves = 8 if nut > waves * per_wave else waves
                    small.add((kt, -(-nut // waves), c, waves))
            waves = 4 if nut <= 4 else 8  # (with 5 to 16 outputs every shape is one of the wider kernel's)
            if kt * -(-nut // waves) <= 12:
                mid.add((kt, -(-nut // waves), waves))
    assert built("small") == sorted(small)
    assert built("mid") == sorted(mid)
    assert built("deep") == sorted((kt, layers, waves) for kt in range(1, 5) for layers in (2, 3) for waves in (4, 8))
