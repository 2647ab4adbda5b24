"""The hand-over between the workgroups of the hash function's recurrence, checked without a GPU: the code the
kernel runs (csrc/handover.h) is compiled for the host and its events are recorded."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2310_18859_amd", "csrc")

SOURCE = r"""
#include "handover.h"
using namespace sida;
// The walk of a posting layer over T steps as text: t/s/f = take, store, fetch a chunk; B = a barrier; P = a post.
extern "C" int walk(int T, char *out, int *chunk)
{
    int n = 0;
    auto put = [&](char what, int c) { out[n] = what; chunk[n++] = c; };
    walk_chunks<kSteps, true>(T, [&](int c) { put('t', c); }, [&](int c) { put('s', c); }, [&] { put('B', -1); },
                              [&](int c) { put('f', c); }, [&] { put('P', -1); }, [&] { put('B', -1); });
    return n;
}
extern "C" int steps_per_chunk() { return kSteps; }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("handover")
    src, so = str(d / "model.cpp"), str(d / "model.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wno-unknown-pragmas", "-I" + CSRC, "-o", so, src],
                   check=True)
    return ctypes.CDLL(so)


def walk(lib, T):
    out, chunk = ctypes.create_string_buffer(16 * T + 64), (ctypes.c_int * (16 * T + 64))()
    n = lib.walk(T, out, chunk)
    return [(out.raw[i:i + 1].decode(), chunk[i]) for i in range(n)]


@pytest.mark.parametrize("T", list(range(1, 34)) + [89, 125, 128, 333, 385, 4096])
def test_a_counted_chunk_has_arrived(lib, T):
    """Wavefronts run freely between two barriers.  Whatever their order, a count of (c + 1) * wavefronts is
    reached only when every wavefront has posted chunk c."""
    events, K = walk(lib, T), -(-T // lib.steps_per_chunk())
    intervals = [[]]
    for what, c in events:
        if what == "B":
            intervals.append([])
        else:
            intervals[-1].append((what, c))
    for wavefronts in (4, 8):
        posted = 0                                       # by every wavefront, at the start of the interval
        for ev in intervals:
            most = posted + sum(w == "P" for w, _ in ev)
            for slow in range(1, wavefronts):            # wavefronts still at the start, the others at the end
                count = slow * posted + (wavefronts - slow) * most
                assert count < (posted + 1) * wavefronts, f"chunk {posted} is taken for complete with {slow} wavefronts behind"
            posted = most
        assert posted == K
    # the order of one wavefront's events: a chunk is fetched, taken, walked, stored and posted, once each
    assert [c for w, c in events if w == "t"] == list(range(K)) and [c for w, c in events if w == "s"] == list(range(K))
    assert [c for w, c in events if w == "f"] == list(range(1, K))
    names = [w for w, _ in events]
    stored = [i for i, w in enumerate(names) if w == "s"]
    posts = [i for i, w in enumerate(names) if w == "P"]
    for c in range(K):
        assert stored[c] < posts[c] and (c + 1 == K or posts[c] < stored[c + 1])
        assert "B" in names[events.index(("t", c)):stored[c]]
