"""Models without a hidden layer on data sets that do not fit a CU's LDS: the first columns stay in global memory."""
import os
import shutil
import subprocess

import pytest

import test_gpu_parity as parity
from test_gpu_parity import bb  # noqa: F401

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2012_04201_amd", "csrc")

PLAN = r"""
#include <cstdio>
#include "%s"
int main() {
  int far_most = 0, at_735_52 = 0, none = 0;
  for (int d = 1; d <= 63; d++)
    for (int n = 1; n <= 4096; n++)
      for (int c = 1; c <= 2; c++) {
        const LinLds l = ll_plan(n, d, c);
        if (!l.waves) { none += n < 2300; continue; }
        const int S = ll_stride(l.dd, l.far);
        bool ok = l.waves >= 4 && l.shared + (uint64_t)l.waves * l.wave_bytes <= LL_LDS_LIMIT;
        ok &= l.shared >= (uint32_t)n * (S + 1) * 4 && l.dd >= d + 1 && (S / 4) %% 2 == 1 && S %% 4 == 0;
        ok &= l.far == 0 || (l.far %% 2 == 1 && 4 * l.far <= d && S == l.dd - 4 * l.far);
        if (!ok) { printf("bad %%d %%d %%d\n", n, d, c); return 1; }
        if (l.far > far_most) far_most = l.far;
        if (n == 735 && d == 52) at_735_52 = l.far;
      }
  printf("%%d %%d %%d\n", far_most, at_735_52, none);
}
"""


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not on PATH")
def test_every_plan_fits_the_lds(tmp_path):
    src = tmp_path / "plan.hip"
    src.write_text(PLAN % os.path.join(CSRC, "train_linear_lds_f32.h"))
    exe = str(tmp_path / "plan")
    res = subprocess.run(["hipcc", "-O1", "--offload-arch=gfx950", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                          "-packed-fp32-ops", str(src), "-o", exe], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    res = subprocess.run([exe], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout
    far_most, at_735_52, none = map(int, res.stdout.split())
    # (none: no plan below 2300 rows)
    assert far_most == 15 and at_735_52 == 3 and none == 0


# one group of far columns (826 x 39 has none) and the most, ragged and odd row lengths (rows that do not begin
# at 16 bytes), one class, two and none, full batch, and more rows than early stopping's cut leaves for a step
@pytest.mark.gpu
@pytest.mark.parametrize("n,d,c,solver,bs", [
    (735, 52, 2, "adam", 100), (827, 39, 2, "sgd", 64), (1200, 63, 1, "adam", 129), (1000, 47, 0, "sgd", 250),
    (4096, 60, 2, "adam", 500), (4096, 5, 1, "adam", 700), (2200, 56, 2, "adam", 0), (3000, 15, 0, "adam", 333)])
def test_steps_and_scores(bb, oracle, n, d, c, solver, bs):  # noqa: F811
    parity.test_linear_models_steps_and_scores(bb, oracle, n, d, c, solver, bs)
