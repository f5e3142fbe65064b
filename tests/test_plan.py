"""The split of a channel's stages over workgroups (csrc/wbmm_plan.h, host
code that every call of a general kernel runs) against a search over every
split, and its time."""
import ctypes
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_02097_amd", "csrc")
SOURCE = r"""
#include <stdint.h>
#include <time.h>
#include "wbmm_plan.h"
extern "C" void plan(int64_t C, int64_t stages, int64_t slots, double ov, int64_t max_parts, int *spw, int *parts) {
  wbmm::gen_plan(C, stages, slots, ov, max_parts, spw, parts);
}
extern "C" double plan_seconds(int64_t C, int64_t stages, int64_t slots, double ov, int64_t max_parts, int n) {
  timespec a, b;
  volatile int sink = 0;
  clock_gettime(CLOCK_MONOTONIC, &a);
  for (int i = 0; i < n; ++i) {
    int spw, parts;
    wbmm::gen_plan(C, stages + (i & 1), slots, ov, max_parts, &spw, &parts);
    sink = sink + spw;
  }
  clock_gettime(CLOCK_MONOTONIC, &b);
  return ((b.tv_sec - a.tv_sec) + 1e-9 * (b.tv_nsec - a.tv_nsec)) / n;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, so = d / "plan.cpp", d / "plan.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I" + CSRC, str(src), "-o", str(so)], check=True)
    lib = ctypes.CDLL(str(so))
    i64 = ctypes.c_int64
    lib.plan.argtypes = [i64, i64, i64, ctypes.c_double, i64, ctypes.c_void_p, ctypes.c_void_p]
    lib.plan_seconds.argtypes = [i64, i64, i64, ctypes.c_double, i64, ctypes.c_int]
    lib.plan_seconds.restype = ctypes.c_double
    return lib


def cdiv(a, b):
    return -(-a // b)


def search(C, stages, slots, ov, max_parts):
    """Every number of workgroups up to the first beyond eight rounds."""
    best, plan = None, None
    for p in range(1, min(stages, max_parts) + 1):
        per = cdiv(stages, p)
        cost = cdiv(C * cdiv(stages, per), slots) * (per + ov)
        if best is None or cost < best - 1e-9:
            best, plan = cost, (per, cdiv(stages, per))
        if C * p > 8 * slots:
            break
    return plan


def test_split_is_the_best_one(lib):
    rng = random.Random(1)
    cases = [(1, 1, 256, 1.0, 1), (1, 1, 256, 3.0, 1 << 20), (256, 7, 256, 1.0, 1 << 20), (257, 7, 256, 1.5, 1 << 20),
             (1, 1 << 20, 512, 1.0, 1 << 20), (4000000, 3, 256, 1.0, 1 << 20)]
    cases += [(int(2 ** rng.uniform(0, 12)), int(2 ** rng.uniform(0, rng.choice([4, 8, 13]))),
               rng.choice([256, 512, 512, 304, 64, 1]), rng.choice([1.0, 1.5, 3.0]),
               rng.choice([1, 2, 3, 7, 10, 40, 1024, 1 << 20])) for _ in range(4000)]
    spw, parts = ctypes.c_int(), ctypes.c_int()
    for case in cases:
        lib.plan(*case, ctypes.byref(spw), ctypes.byref(parts))
        assert (spw.value, parts.value) == search(*case), case


def test_split_takes_no_time(lib):
    """Well below a launch (several microseconds), whatever the sizes: no
    search through thousands of splits."""
    for C in (1, 8, 96, 300, 100000):
        for stages in (1, 100, 4096, 1 << 20):
            t = min(lib.plan_seconds(C, stages, 512, 1.0, 1 << 20, 200) for _ in range(3))
            print("C %d, %d stages: %.2f us" % (C, stages, 1e6 * t))
            assert t < 2e-6, (C, stages)
