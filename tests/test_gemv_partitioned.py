"""The GEMV shape rules count the CUs of the device at hand: with a quarter of
them they choose a quarter of the work-groups (a stand-in for the HIP queries
is loaded before the library; no GPU)."""
from __future__ import annotations

import os
import subprocess
import sys

import pytest

STUB = """
#include <stdlib.h>
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int attr, int dev) { *v = atoi(getenv("CUS")); return 0; }
"""
PROBE = """
import ctypes, sys
class Config(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in ("block", "vec", "unroll", "grid", "increment", "rows", "split")]
lib, c = ctypes.CDLL(sys.argv[1]), Config()
for op, lines, k in ((3, 1, 10**8), (3, 40, 10**6), (3, 500, 5000), (4, 10**7, 3), (4, 10**6, 16), (4, 4096, 4096)):
    assert lib.bwla_get_config(op, 1, 0, ctypes.c_int64(lines), ctypes.c_int64(k), ctypes.byref(c)) == 0
    print(c.block * c.grid if lines == 500 else c.grid)
"""


def test_work_groups_follow_the_device(tmp_path):
    from paper_1409_0669_amd import build
    src, so = tmp_path / "stub.c", tmp_path / "stub.so"
    src.write_text(STUB)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(so), str(src)], check=True)

    def groups(cus):
        env = dict(os.environ, LD_PRELOAD=str(so), CUS=str(cus))
        env.pop("BWLA_TUNING", None)
        out = subprocess.run([sys.executable, "-c", PROBE, build.LIB], env=env, check=True, capture_output=True,
                             text=True).stdout
        return [int(v) for v in out.split()]

    whole, part = groups(256), groups(64)
    assert whole[0] == 256 and part[0] == 64  # one line of 400 MB: a slice per CU
    for w, p in zip(whole, part):
        assert w / 8 <= p <= w / 2, (whole, part)
