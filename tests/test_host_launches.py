"""CPU tests of what a call asks of the HIP runtime: the library runs, in a process of its own, on the recording runtime of
host_runtime.c in place of the real one, so that its planning, streams, events and launches can be read back."""
import json
import os
import shutil
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2012_04201_amd", "libbbo_mlp.so")
pytestmark = pytest.mark.skipif(shutil.which("gcc") is None, reason="gcc not on PATH")

PRELUDE = '''
import ctypes as C, json, struct
rt = C.CDLL({runtime!r}, mode=C.RTLD_GLOBAL)
rt.hr_log.restype = C.c_char_p
L = C.CDLL({lib!r})
L.bbo_mlp_last_error.restype = C.c_char_p

def knob(name, value):
    C.c_int.in_dll(rt, name).value = value

def records(shapes, batch=32):
    out = b""
    for i, h in enumerate(shapes):
        out += struct.pack("<i4i4i7fQfifi", len(h), *(list(h) + [0] * (4 - len(h))), 0, 0, batch, 3,
                           1e-3, 0.0, 0.9, 0.9, 0.999, 1e-8, 0.0, i, 0.0, 0, 0.0, 0)
    return C.create_string_buffer(out, len(out))

P = C.c_void_p
def need(n, d, c, K, shapes, dtype=0):
    out = C.c_size_t(0)
    rc = L.bbo_mlp_workspace_bytes(C.c_int64(n), d, c, K, records(shapes), len(shapes), dtype, C.byref(out))
    assert rc == 0, L.bbo_mlp_last_error()
    return out.value

# (device pointers are numbers here: the recording runtime follows none)
def evaluate(n, d, c, K, shapes, workspace=1 << 40, dtype=0, stream=900):
    return L.bbo_mlp_cv_eval(P(4096), P(4096), C.c_int64(n), d, c, P(4096), K, records(shapes), len(shapes), dtype,
                             P(4096), P(4096), P(0), P(4096), C.c_size_t(workspace), P(stream))

def evaluate_static(n, d, c, K, shapes, dtype=0, stream=900):
    return L.bbo_mlp_cv_eval_static(P(4096), P(4096), C.c_int64(n), d, c, P(4096), K, records(shapes), len(shapes), dtype,
                                    P(4096), P(4096), P(0), P(stream))

def log():
    out = [l.split() for l in rt.hr_log().decode().splitlines()]
    rt.hr_reset()
    return out
'''


@pytest.fixture(scope="module")
def child(tmp_path_factory):
    if not os.path.exists(LIB):
        from paper_2012_04201_amd import build
        build.build_lib()
    runtime = str(tmp_path_factory.mktemp("rt") / "host_runtime.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-Wall", os.path.join(HERE, "host_runtime.c"), "-o", runtime], check=True)

    def run(body):
        code = PRELUDE.format(runtime=runtime, lib=LIB) + textwrap.dedent(body)
        res = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True)
        assert res.returncode == 0, res.stderr[-2000:]
        return json.loads(res.stdout)

    return run


MIXED = "[[20], [64], [100], [130], [], [40, 30], [300]]"


def unjoined(log, caller="900"):
    """Streams with a launch that the caller's stream is not made to wait for by the end of the call."""
    open_, marked = set(), {}
    for op, *a in log:
        if op == "launch" and a[0] != caller:
            open_.add(a[0])
            marked = {e: s - {a[0]} for e, s in marked.items()}
        elif op == "record":
            marked[a[0]] = {a[1]}
        elif op == "wait" and a[0] == caller:
            open_ -= marked.get(a[1], set())
        elif op == "sync":
            open_.discard(a[0])
    return open_


def test_a_call_joins_its_side_streams(child):
    log = child("rc = evaluate(300, 30, 3, 5, %s); assert rc == 0; print(json.dumps(log()))" % MIXED)
    assert len({l[1] for l in log if l[0] == "launch"}) == 4 and not unjoined(log)


@pytest.mark.parametrize("knob", ["hr_fail_launch", "hr_fail_record"])
def test_a_call_that_fails_half_way_leaves_no_stream_behind(child, knob):
    """An error return hands the workspace back to the caller: what is already running on the side streams has to be
    ordered before whatever the caller's stream does next."""
    logs = child("""
        out = []
        for k in range(1, 13):
            evaluate(300, 30, 3, 5, %s)
            log()
            knob("%s", k)
            rc = evaluate(300, 30, 3, 5, %s)
            knob("%s", 0)
            out.append([rc, log()])
        print(json.dumps(out))
    """ % (MIXED, knob, MIXED, knob))
    failed = [log for rc, log in logs if rc]
    assert len(failed) >= 5 and all(rc in (0, 4) for rc, _ in logs)
    assert any(l[0] == "launch" and l[1] != "900" for log in failed for l in log)
    for log in failed:
        assert not unjoined(log), log


@pytest.mark.parametrize("n,d,c,K,shapes,dtype", [
    (300, 30, 3, 5, eval(MIXED), 0), (150, 4, 3, 5, [[8], [40]], 0), (600, 24, 4, 3, [[40, 24], [], [300]], 1),
    (569, 30, 2, 5, [[50], [100], [150], [200]] * 40, 0)])
def test_the_allocation_free_entry_creates_nothing(child, n, d, c, K, shapes, dtype):
    """Its kernels follow each other on the caller's stream: no stream, event or host buffer is made or used, in a
    thread's first call as in any other."""
    log = child("rc = evaluate_static(%d, %d, %d, %d, %r, %d); assert rc == 0; print(json.dumps(log()))" %
                (n, d, c, K, shapes, dtype))
    assert {l[0] for l in log} == {"launch"} and {l[1] for l in log} == {"900"}


@pytest.mark.parametrize("n,d,c,K,dtype,widest,narrower", [
    (569, 30, 2, 5, 0, [224], [[50 + 3 * i % 175] for i in range(256)]),   # variants side by side need three times the room
    (569, 30, 2, 5, 0, [224], [[192]] * 256),                              # more workgroups a CU, more room in all
    (569, 13, 2, 5, 0, [224], [[10]] * 512),
    (1797, 64, 10, 5, 0, [256], [[20 + i % 236] for i in range(256)]),
    (569, 30, 2, 5, 0, [128, 128, 128], [[128, 128, 128], [64, 60, 64]] * 128),
    (1268, 43, 1, 4, 0, [46, 237, 155], [[46, 237, 155], [46, 237, 150], [46, 100, 100]] * 100),  # and larger records
    (600, 64, 10, 5, 1, [256, 256], [[256, 256], [256, 128], [64, 64], []] * 100),
    (569, 30, 2, 5, 0, [224], [[20], [100], [200], [224]] * 2)])
def test_a_workspace_for_the_widest_models_holds_a_mix_of_narrower_ones(child, n, d, c, K, dtype, widest, narrower):
    B = len(narrower)
    out = child("""
        n, d, c, K, dtype, widest, narrower, B = %r
        ws = need(n, d, c, K, [widest] * B, dtype)
        full = need(n, d, c, K, narrower, dtype)
        rcs, logs = [], []
        for room in (ws, full, 256):
            rcs.append(evaluate(n, d, c, K, narrower, room, dtype))
            logs.append(log())
        print(json.dumps([ws, full, rcs, logs]))
    """ % ((n, d, c, K, dtype, widest, narrower, B),))
    ws, full, rcs, (tight, roomy, none) = out
    assert rcs == [0, 0, 3] and none == []
    grids = lambda log: sorted((int(l[3]), int(l[4]), int(l[2])) for l in log if l[0] == "launch")
    streams = lambda log: {l[1] for l in log if l[0] == "launch"}
    for (t0, l0, g), (t1, l1, g1) in zip(grids(tight), grids(roomy)):  # the same launches, on half the workgroups or more
        assert (t0, l0) == (t1, l1) and g <= g1 <= 2 * g + 1
    assert len(grids(tight)) == len(grids(roomy))
    assert streams(tight) in (streams(roomy), {"900"}) and (ws < full or streams(tight) == streams(roomy))


@pytest.mark.parametrize("models,apart", [(2, True), (6, True), (7, False), (60, False)])
def test_workgroups_of_launches_side_by_side_get_a_cu_each(child, models, apart):
    """40, 120, 140 and 1200 workgroups in four launches: up to one for every second of 256 CUs, no CU has the LDS for two."""
    log = child("rc = evaluate(569, 30, 2, 5, [[50], [100], [150], [200]] * %d); assert rc == 0; print(json.dumps(log()))" % models)
    lds = [int(l[4]) for l in log if l[0] == "launch" and "k_train" in l[5]]
    assert len(lds) == 4 and (min(lds) * 2 > 160 * 1024) == apart
