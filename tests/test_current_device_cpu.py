"""Calls on an object of another device than the calling thread's current one,
against a stand-in HIP runtime with two devices (tests/fake_hip.c): work goes
to the object's device, and the current device is the caller's again."""
import os
import subprocess
import sys

import pytest

import paper_1801_05857_amd as gx

HERE = os.path.dirname(os.path.abspath(__file__))

DUMP = r"""
import ctypes, sys
hip = ctypes.CDLL(None)
L = ctypes.CDLL(sys.argv[1])
vp, u64 = ctypes.c_void_p, ctypes.c_uint64
L.gx_table_create.argtypes = [ctypes.c_uint32, ctypes.c_uint32, u64, vp, ctypes.POINTER(vp)]
L.gx_table_dump.argtypes = [vp, vp, u64, ctypes.POINTER(u64)]
L.gx_table_destroy.argtypes = [vp]
dev = ctypes.c_int()
for own, cur, slots in ((1, 0, 1 << 17), (0, 1, 1 << 17), (1, 1, 1 << 17), (1, 0, 64)):
    assert hip.hipSetDevice(own) == 0
    t = vp()
    assert L.gx_table_create(1, 16, slots, None, ctypes.byref(t)) == 0
    assert hip.hipSetDevice(cur) == 0
    before = (ctypes.c_int * 2).in_dll(hip, "fake_mallocs")[1 - own]
    # (no kernel clears the table: a small one reads as 64 zero keys)
    buf = (ctypes.c_uint32 * 64)()
    n = u64(99)
    assert L.gx_table_dump(t, buf, 64, ctypes.byref(n)) == 0
    assert (ctypes.c_int * 2).in_dll(hip, "fake_mallocs")[1 - own] == before, "memory elsewhere"
    assert ctypes.c_int.in_dll(hip, "fake_wrong").value == 0, "launch elsewhere"
    assert hip.hipGetDevice(ctypes.byref(dev)) == 0 and dev.value == cur
    assert L.gx_table_destroy(t) == 0
print("launches", ctypes.c_int.in_dll(hip, "fake_launches").value)
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    if not os.path.exists(gx.LIB_PATH):
        from paper_1801_05857_amd import build

        build.build(force=False)
    so = tmp_path_factory.mktemp("fake") / "fake_hip.so"
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-o", str(so),
                           os.path.join(HERE, "fake_hip.c")])
    return str(so)


def test_dump_of_a_table_of_another_device(fake):
    env = dict(os.environ, LD_PRELOAD=fake)
    r = subprocess.run([sys.executable, "-c", DUMP, gx.LIB_PATH], capture_output=True, text=True,
                       timeout=120, env=env)
    assert r.returncode == 0, r.stdout + r.stderr
    assert int(r.stdout.split()[1]) >= 8  # the gathers and their heads were launched
