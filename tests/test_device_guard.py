"""A step call allocates on the device of its simulation, whatever device its caller has made current since,
and leaves that device current (host code, built here with g++ over a fake device runtime)."""
import ctypes
import os
import re
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    out = os.path.join(tempfile.mkdtemp(), "libdevice_guard_test.so")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(rocm, "include"),
                    "-Wl,-Bsymbolic", "-o", out, os.path.join(ROOT, "tests", "device_guard_driver.cpp")], check=True)
    return ctypes.CDLL(out)


@pytest.mark.parametrize("before,dev", [(0, 0), (0, 1), (3, 1), (7, 0)])
def test_guard(lib, before, dev):
    after = ctypes.c_int(-1)
    assert lib.inside(before, dev, 0, ctypes.byref(after)) == dev and after.value == before
    assert lib.inside(dev, dev, 1, ctypes.byref(after)) == dev and after.value == dev  # no answer: left alone


def test_every_allocation_of_a_simulation_is_guarded():
    src = open(os.path.join(ROOT, "paper_1712_06121_amd", "csrc", "api.cpp")).read()
    calls = [m.start() for m in re.finditer(r"\bhipMalloc\(|\bhipMemGetInfo\(", src)]
    assert len(calls) == 2
    for at in calls:
        assert re.search(r"DeviceGuard on\((owner\.)?device\);[^}]*\Z", src[:at])
