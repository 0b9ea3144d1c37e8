"""wnnc_set_tile and wnnc_set_split on a built tree, on the CPU: the library's
host code runs against a HIP runtime without a device (hip_host.cpp).

A changed task list is complete when the call returns (the header says that
the calls synchronize): the next operator may run on another stream, so no
operation may still be queued then.
"""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2405_16634_amd", "libwnnc.so")

PRELUDE = """
import ctypes, sys
host = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
host.host_launches.restype = ctypes.c_longlong
lib = ctypes.CDLL(sys.argv[2])
N = 25600
lib.wnnc_build.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int64, ctypes.c_void_p]
lib.wnnc_adjoint.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_float, ctypes.c_void_p]
for f in (lib.wnnc_set_tile, lib.wnnc_set_split):
    f.argtypes = [ctypes.c_void_p, ctypes.c_int]
lib.wnnc_destroy.argtypes = [ctypes.c_void_p]
lib.wnnc_last_error.restype = ctypes.c_char_p
P = (ctypes.c_float * (3 * N))()
s = (ctypes.c_float * N)()
out = (ctypes.c_float * (3 * N))()
def context(tile):
    h = ctypes.c_void_p()
    assert lib.wnnc_create(ctypes.byref(h), 0, None) == 0, lib.wnnc_last_error()
    assert lib.wnnc_set_tile(h, tile) == 0
    assert lib.wnnc_build(h, P, N, None) == 0, lib.wnnc_last_error()
    assert host.host_launches() > 0
    return h
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    if not os.path.exists(LIB):
        pytest.skip("libwnnc.so is not built")
    so = str(tmp_path_factory.mktemp("hip") / "libhip_host.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", os.path.join(HERE, "hip_host.cpp"), "-o", so],
                   check=True)

    def go(body):
        p = subprocess.run([sys.executable, "-c", PRELUDE + body, so, LIB], capture_output=True,
                           text=True, timeout=300)
        assert p.returncode == 0, p.stdout + p.stderr
        return p.stdout

    return go


def test_changed_tasks_are_complete_on_return(run):
    run("""
h = context(1)
for change, v in ((lib.wnnc_set_split, 64), (lib.wnnc_set_split, 0), (lib.wnnc_set_tile, 4),
                  (lib.wnnc_set_tile, 2), (lib.wnnc_set_tile, 1), (lib.wnnc_set_split, 256)):
    before = host.host_launches()
    assert change(h, v) == 0, lib.wnnc_last_error()
    assert host.host_launches() > before
    assert host.host_pending() == 0, (v, host.host_pending())
lib.wnnc_destroy(h)
""")


def test_a_failed_change_leaves_no_tasks_to_launch(run):
    """Every allocation that a change of tasks makes fails once: the call
    reports it, and the next operator is refused instead of launched on
    half-replaced tables; after another build everything works."""
    out = run("""
adjoint = lambda h: lib.wnnc_adjoint(h, ctypes.addressof(s), 0.002, ctypes.addressof(out))
failed = 0
for k in range(1, 40):
    h = context(4)
    host.host_fail_allocation(k)
    status = lib.wnnc_set_tile(h, 1)
    assert status == 0 or b"out of memory" in lib.wnnc_last_error()
    host.host_fail_allocation(0)
    before = host.host_launches()
    ran = adjoint(h)
    launched = host.host_launches() - before
    if status == 0:
        assert ran == 0 and launched > 0
        break
    failed += 1
    assert ran != 0 and launched == 0, (k, ran, launched)
    assert lib.wnnc_build(h, P, N, None) == 0, lib.wnnc_last_error()
    assert adjoint(h) == 0
    lib.wnnc_destroy(h)
else:
    raise AssertionError("the change never succeeded")
print("failed", failed)
""")
    assert int(out.split("failed")[1]) >= 8


def test_whole_walks_need_no_cuts(run):
    """Without split walks the tasks are the groups: no cuts are made, counted
    or read back."""
    run("""
h = context(1)
for change, v in ((lib.wnnc_set_split, 0), (lib.wnnc_set_tile, 4), (lib.wnnc_set_tile, 2)):
    before = host.host_launches()
    assert change(h, v) == 0, lib.wnnc_last_error()
    assert host.host_launches() - before == 3, (v, host.host_launches() - before)
lib.wnnc_destroy(h)
""")
