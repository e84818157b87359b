"""Static check of the kernels' generated code (no GPU needed): 16-byte stores through a buffer descriptor.

Where such a store's offset comes from a scalar register too, the hardware still reads its data when the next instruction
issues, and the compiler leaves no wait state (it does where the scalar offset is a constant): an instruction
right behind it that overwrites the data made the last lanes of each row of 16 store the new value.  The sources either give the
constant 0 or keep the stores together, which the generated code has to show."""
import glob
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2012_04201_amd", "csrc")

def arguments(text, start):
    """The arguments of the call whose opening bracket is at text[start]."""
    depth, args, last = 0, [], start + 1
    for i in range(start, len(text)):
        depth += {"(": 1, ")": -1}.get(text[i], 0)
        if depth == 0 or (depth == 1 and text[i] == ","):
            args.append(text[last:i].strip())
            last = i + 1
        if depth == 0:
            return args

def registers(operands):
    found = set()
    for kind, lo, hi in re.findall(r"\b([va])\[(\d+):(\d+)\]", operands):
        found |= {(kind, n) for n in range(int(lo), int(hi) + 1)}
    return found | {(kind, int(n)) for kind, n in re.findall(r"\b([va])(\d+)\b", operands)}


def overwritten(listing):
    """(wide buffer stores, those whose data the next instruction overwrites)"""
    code = [l.strip() for l in listing.split("\n")]
    code = [l for l in code if l and not l.startswith((";", ".")) and not l.endswith(":")]
    stores, bad = 0, []
    for here, behind in zip(code, code[1:]):
        m = re.match(r"buffer_store_dwordx[34] ([va]\[\d+:\d+\]), \S+ \S+ (\S+)", here)
        if m:
            stores += 1
            if re.match(r"s\d|m0", m.group(2)) and behind.startswith("v_") and \
                    registers(m.group(1)) & registers(behind.split(None, 1)[1].split(",")[0]):
                bad.append((here, behind))
    return stores, bad


def test_the_check_sees_an_overwritten_store():
    store = "buffer_store_dwordx4 v[0:3], v21, s[52:55], %s offen\n"
    assert overwritten(store % "s19" + "v_add_u32_e32 v0, s22, v54")[1]
    assert not overwritten(store % "0" + "v_add_u32_e32 v0, s22, v54")[1]
    assert not overwritten(store % "s19" + "v_add_u32_e32 v4, s22, v54")[1]
    assert not overwritten(store % "s19" + "s_nop 0\nv_add_u32_e32 v0, s22, v54")[1]


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not on PATH")
def test_nothing_overwrites_the_data_of_the_tiled_kernels_stores(tmp_path):
    out = tmp_path / "kernels.s"
    cmd = ["hipcc", "-O3", "--offload-arch=gfx950", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "--cuda-device-only", "-S", os.path.join(CSRC, "kernels_tiled.hip"), "-o", str(out)]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    stores, bad = overwritten(out.read_text())
    assert stores > 0 and not bad, bad


def test_the_deep_kernels_stores_have_no_scalar_offset():
    with open(os.path.join(CSRC, "train_deep_f32.h")) as f:
        text = f.read()
    calls = [arguments(text, m.end() - 1) for m in re.finditer(r"raw_buffer_store_b(?:96|128)\(", text)]
    assert calls and all(a[3] == "0" for a in calls), calls


def test_no_other_kernel_makes_such_stores():
    users = {os.path.basename(p) for p in glob.glob(os.path.join(CSRC, "*"))
             if p.endswith((".h", ".hip")) and re.search(r"buffer_store_(?:b96|b128|dwordx[34])", open(p).read())}
    assert users == {"train_deep_f32.h", "train_tiled_bf16.h"}
