"""Builds libbbo_mlp.so (HIP, gfx950) in-tree with hipcc, the kernel families side by side, and the packer of suggestions."""
import os
import subprocess
import sysconfig
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libbbo_mlp.so")
SOURCES = ["kernels_tiled.hip", "kernels_deep3.hip", "kernels_deep2.hip", "kernels_mid.hip", "kernels_full.hip", "kernels_small2.hip",
           "kernels_small1.hip", "kernels_small3.hip", "kernels_small4.hip", "kernels_linear_lds.hip", "kernels_linear.hip", "bbo_mlp.hip"]
FLAGS = ["-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall", "-Wno-unused-function"]


def _run(cmd):
    res = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(cmd[0] + " failed:\n" + err)
    return err


def build_lib(verbose=False):
    jobs = int(os.environ.get("MAX_JOBS", 0)) or min(8, os.cpu_count() or 1)
    with tempfile.TemporaryDirectory() as tmp, ThreadPoolExecutor(jobs) as pool:
        objs = [os.path.join(tmp, s + ".o") for s in SOURCES]
        errs = list(pool.map(lambda so: _run(["hipcc"] + FLAGS + ["-c", os.path.join(CSRC, so[0]), "-o", so[1]]),
                             zip(SOURCES, objs)))
        errs.append(_run(["hipcc", "--offload-arch=gfx950", "-shared"] + objs + ["-o", LIB]))
    err = "\n".join(e for e in errs if e.strip())
    if verbose and err:
        print(err)
    _run(["gcc", "-O2", "-shared", "-fPIC", "-Wall", "-I" + sysconfig.get_paths()["include"],
          os.path.join(CSRC, "pack_hparams.c"), "-o", os.path.join(HERE, "_pack.so")])
    return LIB


if __name__ == "__main__":
    print(build_lib(verbose=True))
