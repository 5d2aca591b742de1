"""The host side of plans and rankers over a HIP runtime of host memory.  A plan whose growth fails for
want of memory is not loaded any more (nothing is launched on buffers that are gone) and can
be loaded again.  Maps and class tuples are given after whatever evaluates a batch.  A
ranker's buffers are not allocated anew for every size."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

HEAD = """
import ctypes, sys
import numpy as np
fake = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
fail, launches = ctypes.c_int.in_dll(fake, "fake_fail"), ctypes.c_int.in_dll(fake, "fake_launches")
import paper_2507_17087_amd as tm
import workloads as W
L, p = tm.lib(), ctypes.c_void_p()
out, best, pmap = np.zeros((400, 4), np.int64), np.zeros(1, np.int64), np.zeros(64, np.int32)
st = W.stencil((1, 1), 8)

def load(n):
    c = W.batch([W.candidate((8, 8), 2, 2, [])] * n)
    return L.tm_plan_load(p, c.ctypes.data, n, st.ctypes.data, 0, None)

def run():
    return L.tm_plan_run(p, out.ctypes.data, best.ctypes.data, None)
"""

GROWTH = HEAD + """
assert L.tm_plan_create(4, 1, ctypes.byref(p)) == tm.TM_OK
assert (load(4), run()) == (tm.TM_OK, tm.TM_OK) and launches.value > 0, L.tm_last_error()
fail.value = 100000
assert load(400) == tm.TM_ENOMEM
n = launches.value
codes = [run(), L.tm_plan_run_map(p, out.ctypes.data, best.ctypes.data, pmap.ctypes.data, 64, None),
         L.tm_plan_materialize(p, None, 0, pmap.ctypes.data, 64, None),
         L.tm_plan_run_stage(p, 1, out.ctypes.data, None, None),
         L.tm_search(p, None, np.array([0, 4], np.int64).ctypes.data, 1, 0, 1, 0.0, 0.0, best.ctypes.data, None, None)]
assert codes == [tm.TM_EINVAL] * 5 and launches.value == n, (codes, launches.value - n)
assert b"not loaded" in L.tm_last_error()
assert load(5) == tm.TM_OK and run() == tm.TM_OK and launches.value > n
fail.value = 0
assert load(400) == tm.TM_OK and run() == tm.TM_OK
assert L.tm_plan_destroy(p) == tm.TM_OK
print("done")
"""

READY = HEAD + """
tuples, seg = ctypes.c_int64(), np.array([0, 4], np.int64)
ways = {
    "run": run,
    "stage": lambda: L.tm_plan_run_stage(p, 1, out.ctypes.data, best.ctypes.data, None),
    "run_map": lambda: L.tm_plan_run_map(p, out.ctypes.data, best.ctypes.data, pmap.ctypes.data, 64, None),
    "search": lambda: L.tm_search(p, None, seg.ctypes.data, 1, 0, 1, 0.0, 0.0, best.ctypes.data, None, None),
    "autotune": lambda: L.tm_plan_autotune(p, out.ctypes.data, None, None, None),
}

def asked():
    return (L.tm_plan_materialize(p, None, 3, pmap.ctypes.data, 64, None),
            L.tm_plan_class_tuples(p, ctypes.byref(tuples), None))

OK, NO = (tm.TM_OK,) * 2, (tm.TM_EINVAL,) * 2
for name, way in ways.items():
    assert L.tm_plan_create(4, 1, ctypes.byref(p)) == tm.TM_OK
    assert asked() == NO and load(4) == tm.TM_OK and asked() == NO, name
    assert way() == tm.TM_OK and asked() == OK, (name, L.tm_last_error())
    assert L.tm_plan_set_launch(p, 1, 0, None) == tm.TM_OK and asked() == OK, name
    assert load(4) == tm.TM_OK and asked() == OK, name
    assert L.tm_plan_destroy(p) == tm.TM_OK
assert L.tm_plan_create(4, 100000, ctypes.byref(p)) == tm.TM_OK  # room for the tables
assert load(4) == tm.TM_OK and asked() == OK
assert L.tm_plan_destroy(p) == tm.TM_OK
assert L.tm_plan_create(4, 16, ctypes.byref(p)) == tm.TM_OK  # for the owner tables only
assert load(4) == tm.TM_OK and asked() == NO
assert L.tm_plan_destroy(p) == tm.TM_OK
print("done")
"""

SIZES = HEAD + """
allocs = ctypes.c_int.in_dll(fake, "fake_allocs")
feat, y = np.zeros((4096, 64), np.float32), np.zeros((4096, 2), np.float32)
grad = np.zeros(L.tm_ranker_param_count(), np.float32)
assert L.tm_ranker_create(1, ctypes.byref(p)) == tm.TM_OK
counts = []
for sizes in (range(1, 1025), range(1024, 0, -1), (4096, 4095, 1)):
    at = allocs.value
    for n in sizes:
        assert L.tm_ranker_forward(p, feat.ctypes.data, n, y.ctypes.data, None) == tm.TM_OK
        if n % 97 == 1:
            assert L.tm_ranker_grad(p, feat.ctypes.data, y.ctypes.data, n, grad.ctypes.data, None) == tm.TM_OK
    counts.append(allocs.value - at)
assert counts == [2, 0, 1], counts
assert L.tm_ranker_destroy(p) == tm.TM_OK
print("done")
"""


def over_host_memory(tmp_path, body):
    so = str(tmp_path / "fake_hip.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-w", "-o", so, os.path.join(HERE, "fake_hip.c")], check=True)
    p = subprocess.run([sys.executable, "-c", body, so], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert p.returncode == 0 and p.stdout.strip() == "done", p.stdout + p.stderr


def test_growth_without_memory(tmp_path):
    over_host_memory(tmp_path, GROWTH)


def test_maps_after_any_evaluation(tmp_path):
    over_host_memory(tmp_path, READY)


def test_buffers_of_many_sizes(tmp_path):
    over_host_memory(tmp_path, SIZES)
