"""The rule that cuts an ensemble's count passes into launches (host code, built here with g++): no
launch of 2^32 work-items or more, no more launches than that takes, every box once and in order."""
import ctypes
import os
import re
import subprocess
import tempfile

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1712_06121_amd", "csrc")


@pytest.fixture(scope="module")
def lib():
    out = os.path.join(tempfile.mkdtemp(), "liblaunch_groups_test.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-o", out,
                    os.path.join(ROOT, "tests", "launch_groups_driver.cpp")], check=True)
    return ctypes.CDLL(out)


def runs(lib, per, threads):
    per = np.asarray(per, np.uint32)
    first = np.zeros(len(per) + 1, np.int64)
    n = lib.runs(per.ctypes.data_as(ctypes.c_void_p), len(per), threads, first.ctypes.data_as(ctypes.c_void_p))
    return first[:n + 1].tolist()


# tiles of meshes of nm cells per side: (nm / 16)^3
@pytest.mark.parametrize("sides,want", [
    ([64], 1), ([64, 96, 128] * 40, 1), ([2048], 1), ([2048, 2048], 2), ([1024] * 15, 1), ([1024] * 16, 2),
    ([1024] * 15 + [1024 - 16], 1), ([64] + [2048] * 2 + [64], 2), ([2048, 64, 2048, 64, 2048], 3)])
def test_count_pass_runs(lib, sides, want):
    threads = lib.count_threads()
    per = [(nm // 16)**3 for nm in sides]
    first = runs(lib, per, threads)
    assert first[0] == 0 and first[-1] == len(per) and all(a < b for a, b in zip(first, first[1:]))
    blocks = [sum(per[a:b]) for a, b in zip(first, first[1:])]
    assert all(b * threads < 2**32 for b in blocks)
    assert len(blocks) == want
    for (a, b), n in zip(zip(first[1:], first[2:]), blocks):  # a run ends only where the next box is too much
        assert (n + per[a]) * threads >= 2**32


def test_the_kernel_and_the_rule_have_one_width():
    src = open(os.path.join(CSRC, "particles.hip")).read()
    assert re.search(r"constexpr int CNTH = kCountThreads;", src)
    assert re.search(r"k_count_boxes<X, V><<<g\.blocks, CNTH, 0, st>>>", src)
    assert re.search(r"box_runs\(per, \(uint64_t\)threads\)", src) and re.search(r": CNTH;", src)
