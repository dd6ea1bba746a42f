"""Runs the library's host side without a device and returns what it would
have launched (tests/host_launch/recorder.cpp takes the place of the HIP
runtime).  ``script`` is the body of a Python program in which ``cq`` is the
binding module, ``L`` the loaded C library, ``C`` ctypes, and ``events()`` the
launches and uploads since the last call; what it assigns to ``out`` comes
back (through JSON).  Device pointers are made up: nothing reads them."""
import json
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "host_launch", "recorder.cpp")

PREAMBLE = """
import ctypes as C, json, sys
sys.path.insert(0, {root!r})
R = C.CDLL({lib!r}, mode=C.RTLD_GLOBAL)
R.recorder_events.restype = C.c_char_p
import paper_2205_05836_amd as cq
from paper_2205_05836_amd import _lib, api
L = _lib.lib()
def events():
    e = json.loads(R.recorder_events().decode())
    R.recorder_clear()
    return e
"""


def build(tmp):
    cxx = shutil.which("g++")
    if cxx is None or not os.path.isdir("/opt/rocm/include"):
        pytest.skip("no host C++ compiler or HIP headers")
    lib = os.path.join(str(tmp), "recorder.so")
    r = subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                        "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2205_05836_amd", "csrc"),
                        "-I", "/opt/rocm/include", SRC, "-o", lib], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    return lib


def run(lib, script, **env):
    code = PREAMBLE.format(root=ROOT, lib=lib) + script + "\nprint('\\n' + json.dumps(out))\n"
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=600,
                       env=dict(os.environ, CQ_AUTOTUNE="0", **env), cwd=ROOT)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-3000:]
    return json.loads(r.stdout.splitlines()[-1])
