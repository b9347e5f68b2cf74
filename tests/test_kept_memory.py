"""What becomes of the memory of destroyed trainers, on a stand-in for the HIP runtime (tests/hip_stub.cpp) that has
as much "device" memory as a test says.  Each test runs in a process of its own: the library keeps state."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2201_00194_amd", "libfamilyseer.so")

PRELUDE = """
import ctypes, sys
import numpy as np
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
stub.stub_used.restype = ctypes.c_size_t
stub.stub_budget.argtypes = [ctypes.c_size_t]
lib = ctypes.CDLL(sys.argv[2])
P, i32, f32 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_float
lib.fs_trainer_create.argtypes = [P, i32, P, i32, ctypes.c_int64, P, i32, P, P, P, f32, i32, i32, P]
lib.fs_trainer_destroy.argtypes = [P]
lib.fs_workspace_reserve.argtypes = [ctypes.c_size_t] * 2

class Params(ctypes.Structure):
    _fields_ = [("depth", i32)] + [(n, f32) for n in ("eta", "lam", "gain", "weight", "scale")]

def create(rows=1000, features=9, trees=64):
    x, off, y = np.zeros(rows * features, np.float32), np.arange(rows + 1, dtype=np.int32), np.zeros(rows, np.float32)
    cut_off, cuts = np.arange(features + 1, dtype=np.int32), np.zeros(features, np.float32)
    t = P()
    rc = lib.fs_trainer_create(ctypes.byref(t), features, x.ctypes.data, 0, rows, off.ctypes.data, rows, y.ctypes.data,
                               cut_off.ctypes.data, cuts.ctypes.data, 0.0, 4, trees, None)
    assert rc == 0, rc
    return t

def boost(*trainers, rounds=1):
    arr = (P * len(trainers))(*trainers)
    p = Params(4, 0.5, 1.0, 0.0, 1.0, 1024.0)
    return lib.fs_train_boost(len(trainers), arr, rounds, ctypes.byref(p), None)

def kept_after(*destroyed):
    before = stub.stub_used()
    for t in destroyed:
        lib.fs_trainer_destroy(t)
    assert stub.stub_used() == before, "nothing was kept"
    return before
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("stub") / "libstub.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", os.path.join(HERE, "hip_stub.cpp"), "-o", so], check=True)

    def run_code(code):
        done = subprocess.run([sys.executable, "-c", PRELUDE + code, so, LIB], capture_output=True, text=True, timeout=120)
        assert done.returncode == 0, done.stderr

    return run_code


@pytest.mark.parametrize("spare", [0, 50_000])
def test_a_reservation_takes_it_back(run, spare):
    """For the descriptors' buffers (2 x 21 KB) and, with those to be had, for the ring's slots (64 KB each)."""
    run(f"""
used = kept_after(create(trees=4000))
stub.stub_budget(used + {spare})
assert lib.fs_workspace_reserve(0, 0) == 0
assert stub.stub_used() < used
""")


def test_descriptors_of_a_batch_take_it_back(run):
    run("""
a, b = create(), create()
used = kept_after(a)
stub.stub_budget(used)
assert boost(b) == 0
stub.stub_budget(2 ** 63)
more = [create() for _ in range(20)]
gone = more.pop()
used = kept_after(gone)
stub.stub_budget(used)
assert boost(b, *more) == 0                  # more than the first allocation is for
""")


def test_only_what_works_in_it_is_waited_for(run):
    run("""
a, b = create(), create()
assert boost(a, b) == 0
used = kept_after(a)
waits = stub.stub_device_waits(), stub.stub_event_waits()
c = create()
assert stub.stub_used() == used
assert (stub.stub_device_waits(), stub.stub_event_waits()) == (waits[0], waits[1] + 1)
kept_after(c)                                # no call worked in it: nothing to wait for
d = create()
assert (stub.stub_device_waits(), stub.stub_event_waits()) == (waits[0], waits[1] + 1)
""")


def test_memory_that_a_graph_works_in_is_not_kept(run):
    run("""
a, b = create(), create()
assert boost(a, b) == 0
stub.stub_capturing(1)
assert boost(a) == 0
stub.stub_capturing(0)
used = stub.stub_used()
lib.fs_trainer_destroy(a)
assert stub.stub_used() < used
kept_after(b)
""")
