"""Loads that are to reach no memory (csrc/past_end.h), checked without a GPU: the offsets that the grouped GEMM's loads take
behind a workgroup's last tile are out of range by every reading of the range check, for every matrix and batch it accepts."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2310_18859_amd", "csrc")

SOURCE = r"""
#include "past_end.h"
using namespace sida;
extern "C" bool is_dropped(unsigned records, int lane, int scalar) { return dropped(records, lane, scalar); }
extern "C" int past_end() { return kPastEnd; }
extern "C" int token_scalar(int ahead) { return last_token_scalar(ahead); }
extern "C" int weight_scalar(int ahead) { return last_weight_scalar(ahead); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("past_end")
    src, so = str(d / "model.cpp"), str(d / "model.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-Wall", "-I" + CSRC, "-o", so, src], check=True)
    lib = ctypes.CDLL(so)
    lib.is_dropped.restype = ctypes.c_bool
    lib.is_dropped.argtypes = [ctypes.c_uint32, ctypes.c_int32, ctypes.c_int32]
    return lib


def reads(records, lane, scalar, clamped):
    """A load of 16 bytes reads something: the check as an unsigned comparison, with the records less the scalar offset
    held at 0 or wrapped round."""
    left = records - scalar
    return (lane & 0xffffffff) < ((max(left, 0) if clamped else left) & 0xffffffff)


@pytest.mark.parametrize("ahead", [2, 4])
@pytest.mark.parametrize("K", [128, 256, 384, 1024, 3072, 4096])
def test_loads_behind_the_last_tile_are_dropped(lib, K, ahead):
    if K % (64 * ahead):
        return
    past = lib.past_end()
    # K-steps left when the last tile's loads are all out: the scalar offsets count from 0 again
    token = [s * 128 for s in range(ahead)]
    weight = [s * 4096 + f * 1024 for s in range(ahead) for f in range(4)]
    assert max(token) == lib.token_scalar(ahead) and max(weight) == lib.weight_scalar(ahead)
    most_rows = (2**31 - 1) // (K * 2)                       # 32-bit byte offsets: larger batches are refused
    cases = [(rows * K * 2, s) for rows in (1, 2, 127, most_rows) for s in token]
    cases += [(n * K * 2, s) for n in (128, 256, 4096) for s in weight]
    for records, scalar in cases:
        assert lib.is_dropped(records, past, scalar), (records, scalar)
        assert not reads(records, past, scalar, True) and not reads(records, past, scalar, False)


def test_what_is_not_dropped_for_certain(lib):
    """An empty descriptor with a scalar offset, and a single row whose scalar offset runs on past it, are dropped only if
    the range check clamps."""
    for records, lane, scalar in [(0, 1008, 4096), (0, 0, 1), (128, lib.past_end(), 256)]:
        assert not lib.is_dropped(records, lane, scalar)
        assert reads(records, lane, scalar, False) and not reads(records, lane, scalar, True)
    assert lib.is_dropped(0, 0, 0) and not lib.is_dropped(4096, 1008, 2048) and not lib.is_dropped(4096, 0, -1)
