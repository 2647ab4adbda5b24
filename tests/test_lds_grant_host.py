"""Permission for large dynamic LDS (csrc/lds_grant.h), checked without a GPU: once per device, and asked for again
after a failure."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2310_18859_amd", "csrc")

SOURCE = r"""
#include "lds_grant.h"
// Launches on devices[0 .. n); the runtime's answers are answers[0 ..], one per time it is asked.
extern "C" int launches(const int *devices, int n, const int *answers, int *results)
{
    sida::LdsGrant grant;
    int asked = 0;
    for (int i = 0; i < n; ++i) results[i] = grant.on(devices[i], [&] { return answers[asked++]; });
    return asked;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("grant")
    src, so = str(d / "grant.cpp"), str(d / "grant.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-Wall", "-I" + CSRC, "-o", so, src], check=True)
    return ctypes.CDLL(so)


@pytest.mark.parametrize("devices,answers,want,asked", [
    ([0, 0, 0], [0], [0, 0, 0], 1),
    ([0, 1, 0, 7, 1, 63], [0, 0, 0, 0], [0] * 6, 4),                # every device is asked for
    ([0, 0, 0], [98, 98, 0], [98, 98, 0], 3),                       # a failure is not kept
    ([1, 0, 1, 0], [98, 0, 0], [98, 0, 0, 0], 3),                   # ... and is its device's own
    ([64, 64, 1000], [0, 0, 0], [0, 0, 0], 3),
])
def test_asked_once_per_device_and_again_after_a_failure(lib, devices, answers, want, asked):
    ints = lambda v: (ctypes.c_int * len(v))(*v)
    results = ints([-1] * len(devices))
    assert lib.launches(ints(devices), len(devices), ints(answers + [0]), results) == asked
    assert list(results) == want
