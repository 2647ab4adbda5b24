"""The heads that keep a layer's weights (csrc/heads_walk.h), checked without a GPU: every tile has a workgroup, the offsets of
their loads fit 32 signed bits, and the calls that take them."""
import ctypes
import os
import subprocess

import pytest

from test_gpu_hash_parts import NOT_WALKED, WALKED

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2310_18859_amd", "csrc")

SOURCE = r"""
#include "heads_walk.h"
using namespace sida;
extern "C" bool walks(int C, int E, int L, int N) { return heads_walk(C, E, L, N); }
extern "C" int waves(int E) { return heads_walk_waves(E); }
extern "C" int workgroups(int N, int L, int waves) { return heads_walk_workgroups(N, L, waves); }
extern "C" int tokens(int waves) { return heads_walk_tokens(waves); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("heads_walk")
    src, so = str(d / "walk.cpp"), str(d / "walk.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-Wall", "-I" + CSRC, "-o", so, src], check=True)
    lib = ctypes.CDLL(so)
    lib.walks.restype = ctypes.c_bool
    return lib


def launch(lib, E, L, N):
    """(workgroups of a layer, tiles, tokens of a tile)"""
    waves = lib.waves(E)
    tokens = lib.tokens(waves)
    return lib.workgroups(N, L, waves), -(-N // tokens), tokens


@pytest.mark.parametrize("E", [17, 64, 128, 129, 256])
@pytest.mark.parametrize("L", [1, 3, 6, 12, 31])
@pytest.mark.parametrize("C", [64, 128])
def test_offsets_of_the_loads_fit(lib, C, E, L):
    """A workgroup's last loads are those of the tile after the next one behind its last: 16 bytes, read as zeros."""
    low, high = 2048 if L * 2048 >= 32768 else 32768 // L + 1, 2**31 // (4 * C)
    assert lib.walks(C, E, L, low) and not lib.walks(C, E, L, high)
    while high - low > 1:
        mid = (low + high) // 2
        low, high = (mid, high) if lib.walks(C, E, L, mid) else (low, mid)
    groups, tiles, tokens = launch(lib, E, L, low)
    last = max(b + (tiles - 1 - b) // groups * groups for b in (0, groups - 1, (tiles - 1) % groups))
    assert last == tiles - 1
    assert ((last + 2 * groups) * tokens + tokens) * C * 4 <= 2**31 - 1
    assert low > 0.98 * 2**31 / (4 * C)                                     # and no more is refused than that takes


@pytest.mark.parametrize("E,L,N", [(17, 16, 2048), (64, 6, 8192), (128, 6, 8192), (128, 12, 2731), (250, 3, 2057), (256, 6, 8192),
                                   (129, 63, 2048), (20, 400, 2048), (100, 1, 100003)])
def test_every_tile_has_a_workgroup(lib, E, L, N):
    groups, tiles, _ = launch(lib, E, L, N)
    each = -(-tiles // groups)
    assert 1 <= groups <= tiles and groups * each >= tiles and (groups - 1) * each < tiles
    assert groups * L <= max(L, 768 if E <= 128 else 256)                   # all resident at a time


@pytest.mark.parametrize("C,E,L,N,want", [
    (128, 128, 6, 8192, True), (128, 128, 6, 5462, True), (128, 128, 6, 5461, False), (128, 16, 16, 8192, False),
    (128, 17, 16, 2048, True), (128, 17, 17, 2047, False), (128, 250, 3, 2048, True), (128, 250, 2, 3071, False),
    (128, 250, 2, 3072, True), (64, 128, 12, 2731, True),
    (64, 20, 400, 2048, False), (64, 20, 260, 2048, False), (64, 30, 260, 6144, False), (64, 60, 129, 2048, True), (64, 60, 14, 2600, True),
    (128, 20, 400, 2048, True), (64, 150, 52, 2048, True), (64, 250, 1, 6144, True),
])
def test_calls_that_walk(lib, C, E, L, N, want):
    assert lib.walks(C, E, L, N) == want


@pytest.mark.parametrize("C,L,E,n_seq,T", WALKED + NOT_WALKED)
def test_calls_of_the_gpu_test_walk_as_it_says(lib, C, L, E, n_seq, T):
    N, walked = n_seq * T, (C, L, E, n_seq, T) in WALKED
    groups, tiles, tokens = launch(lib, E, L, N)
    assert lib.walks(C, E, L, N) == walked and N >= 2048
    assert not walked or -(-tiles // groups) >= 3
