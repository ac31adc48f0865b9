"""Runs a few lines against libsas.so in a process whose HIP runtime is the
recorder (tests/hip_recorder.cpp): nothing runs, every launch is noted.

The lines see `sas` (the binding), `np`, `launches()` (the launches since it
was last called, as (kernel, grid, block) with grid and block the products of
their dimensions), `buffer(nbytes)` (address of 256-byte aligned host memory)
and leave their answer in `out`, which run() returns."""
import json
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

_BEFORE = r"""
import ctypes, json, re, sys, types
rec = ctypes.CDLL(%r, mode=ctypes.RTLD_GLOBAL)
rec.recorder_count.restype = ctypes.c_int64
rec.recorder_launch.restype = ctypes.c_char_p
sys.path.insert(0, %r)
sys.modules["torch"] = types.ModuleType("torch")  # no device memory is wanted of it
import numpy as np
from paper_2509_26279_amd import sas
lib = sas.load()
_held = []

def buffer(nbytes):
    _held.append(ctypes.create_string_buffer(nbytes + 256))
    return (ctypes.addressof(_held[-1]) + 255) // 256 * 256

def launches():
    d, got = (ctypes.c_uint32 * 6)(), []
    for i in range(rec.recorder_count()):
        name = rec.recorder_launch(ctypes.c_int64(i), d).decode()
        m = re.search(r"N_1(\d+)(k_\w+)", name)  # length and name
        got.append((m.group(2)[:int(m.group(1))], d[0] * d[1] * d[2], d[3] * d[4] * d[5]))
    rec.recorder_clear()
    return got
"""


def run(tmp_path, body):
    if shutil.which("g++") is None:
        pytest.skip("g++ not found")
    so = str(tmp_path / "hip_recorder.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-shared", "-fPIC", "-o", so,
                    os.path.join(HERE, "hip_recorder.cpp")], check=True)
    r = subprocess.run([sys.executable, "-c",
                        _BEFORE % (so, ROOT) + body + "\nprint(json.dumps(out))\n"],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    return json.loads(r.stdout.splitlines()[-1])
