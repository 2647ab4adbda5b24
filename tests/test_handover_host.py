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
// The walk of a layer over T steps as text: t/s/f = take, store, fetch a chunk; S = a step, which ends with a
// barrier; B = a barrier of its own; P = a post.
template <bool POST>
int walk_of(int T, char *out, int *chunk)
{
    int n = 0;
    auto put = [&](char what, int c) { out[n] = what; chunk[n++] = c; };
    walk_chunks<kSteps, POST>(T, [&](int c) { put('t', c); }, [&](int c) { put('s', c); }, [&] { put('S', -1); },
                              [&](int c) { put('f', c); }, [&] { put('P', -1); }, [&] { put('B', -1); });
    return n;
}
extern "C" int walk(int T, bool post, char *out, int *chunk) { return post ? walk_of<true>(T, out, chunk) : walk_of<false>(T, out, chunk); }
extern "C" int steps_per_chunk() { return kSteps; }
extern "C" void role(int ticket, int n_seq, int *what, int *seq)
{
    const Role r = role_of(ticket, n_seq);
    *what = r.what;
    *seq = r.seq;
}
// Waits for 1, 2, .. n on a counter that shows values[0 .. count) and then the last one for ever; returns the
// peeks it took, and in *seen what it went on with.
extern "C" long long waits(int n, const int *values, int count, int *seen)
{
    long long peeks = 0;
    *seen = 0;
    for (int want = 1; want <= n; ++want) wait_for(want, *seen, [&] { return values[peeks++ < count ? peeks - 1 : count - 1]; });
    return peeks;
}
extern "C" int most_peeks() { return kMostPeeks; }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("handover")
    src, so = str(d / "model.cpp"), str(d / "model.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wno-unknown-pragmas", "-I" + CSRC, "-o", so, src],
                   check=True)
    lib = ctypes.CDLL(so)
    lib.waits.restype = ctypes.c_longlong
    return lib


def walk(lib, T, post=True):
    out, chunk = ctypes.create_string_buffer(16 * T + 64), (ctypes.c_int * (16 * T + 64))()
    n = lib.walk(T, ctypes.c_bool(post), out, chunk)
    return [(out.raw[i:i + 1].decode(), chunk[i]) for i in range(n)]


LENGTHS = list(range(1, 34)) + [89, 125, 128, 333, 385, 4096]


@pytest.mark.parametrize("post", [True, False])
@pytest.mark.parametrize("T", LENGTHS)
def test_every_chunk_is_walked_whole(lib, T, post):
    """Between take(c) and take(c + 1): the states of chunk c - 1 are stored before the first step, every time step of
    chunk c is made once, and chunk c + 1's inputs are asked for (they replace chunk c's, which take(c) has put away)."""
    events, steps = walk(lib, T, post), lib.steps_per_chunk()
    K = -(-T // steps)
    taken = [i for i, (w, _) in enumerate(events) if w == "t"]
    assert taken[0] == 0 and [events[i][1] for i in taken] == list(range(K))
    end_of_walk = max(i for i, (w, _) in enumerate(events) if w == "s")
    for c, (begin, end) in enumerate(zip(taken, taken[1:] + [end_of_walk])):
        part = events[begin + 1:end]
        names = [w for w, _ in part]
        assert names.count("S") == min(steps, T - c * steps)
        assert [e for e in part if e[0] == "s"] == [("s", c - 1)] * (c > 0)
        assert c == 0 or names[0] == "s"
        assert [e for e in part if e[0] == "f"] == [("f", c + 1)] * (c + 1 < K)
        assert names.count("P") == (post and c > 0) and "B" not in names
    # the last chunk's states leave after the last step (and after the post of those before them)
    assert events[end_of_walk] == ("s", K - 1) and [w for w, _ in events[end_of_walk + 1:]] == ["B", "P"] * post


@pytest.mark.parametrize("T", LENGTHS)
def test_a_counted_chunk_has_arrived(lib, T):
    """Wavefronts run freely between two barriers.  Whatever their order, a count of (c + 1) * wavefronts is
    reached only when every wavefront has posted chunk c."""
    events, K = walk(lib, T), -(-T // lib.steps_per_chunk())
    events = [("B" if w == "S" else w, c) for w, c in events]
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


@pytest.mark.parametrize("n_seq", [1, 2, 7, 85])
def test_every_ticket_is_a_role_of_a_sequence(lib, n_seq):
    """3 * n_seq tickets are all roles of all sequences, lower roles first; any other number stays in range."""
    def role(ticket):
        what, seq = ctypes.c_int(-1), ctypes.c_int(-1)
        lib.role(ticket, n_seq, ctypes.byref(what), ctypes.byref(seq))
        return what.value, seq.value
    assert [role(t) for t in range(3 * n_seq)] == [(w, s) for w in range(3) for s in range(n_seq)]
    for t in [-1, -2, -n_seq, -3 * n_seq - 1, -2**31, 2**31 - 1, 3 * n_seq, 0x7FC00000, -0x7FC00000]:
        what, seq = role(t)
        assert 0 <= what <= 2 and 0 <= seq < n_seq, t


def waits(lib, n, values):
    seen = ctypes.c_int(-1)
    peeks = lib.waits(n, (ctypes.c_int * len(values))(*values), len(values), ctypes.byref(seen))
    return peeks, seen.value


def test_a_wait_takes_what_arrives(lib):
    assert waits(lib, 3, [0, 0, 1, 1, 2, 3]) == (6, 3)
    assert waits(lib, 5, [0, 5]) == (2, 5)               # what has been seen is not looked at again
    assert waits(lib, 4, [2, 0, 0, 3, 4]) == (5, 4)      # a counter that was cleared meanwhile


@pytest.mark.parametrize("stuck", [0, 1, 3, -2**31])
def test_a_wait_for_what_never_arrives_ends_and_is_the_last(lib, stuck):
    """The counter stays below what is waited for: the wait gives up once, and no later wait looks at it again."""
    peeks, seen = waits(lib, 512, [stuck])
    assert peeks <= lib.most_peeks() + 4 and seen == 2**31 - 1
