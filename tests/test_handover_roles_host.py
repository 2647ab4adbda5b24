"""The four-role recurrence of the hash function (csrc/handover.h), checked without a GPU: tickets, counters and the progress
that layer 1's own gate pre-activations report; then whole calls with a thread for every wavefront, workgroups starting in
any order and few of them at a time."""
import ctypes
import subprocess

import pytest

from test_handover_host import CSRC

SOURCE = r"""
#include <atomic>
#include <condition_variable>
#include <mutex>
#include <random>
#include <thread>
#include <vector>
#include "handover.h"
using namespace sida;
extern "C" void role4(int ticket, int n_seq, int *what, int *seq)
{
    const Role r = role_of_four(ticket, n_seq);
    *what = r.what;
    *seq = r.seq;
}
extern "C" int lines(int seq, int *l1, int *g2, int *g1)
{
    *l1 = layer1_line(seq);
    *g2 = gates2_line(seq);
    *g1 = gates1_line(seq);
    return kLine;
}
extern "C" int words(int n_seq) { return counter_words(n_seq); }
extern "C" int there(int rounds, int tokens, int steps) { return chunks_there(rounds, tokens, steps); }
extern "C" int gate_tokens() { return kGateTokens; }
extern "C" int steps_per_chunk(bool narrow) { return narrow ? kStepsNarrow : kSteps; }

struct Barrier {
    std::mutex m;
    std::condition_variable cv;
    int n, waiting = 0, turn = 0;
    explicit Barrier(int count) : n(count) {}
    void operator()()
    {
        std::unique_lock<std::mutex> lk(m);
        const int mine = turn;
        if (++waiting == n) {
            waiting = 0;
            ++turn;
            cv.notify_all();
        } else {
            cv.wait(lk, [&] { return turn != mine; });
        }
    }
};

// One call of n_seq sequences of T steps with `wavefronts` per layer and at most `resident` workgroups at a time.  A token's
// number goes x -> layer 1's gates (100 + x) -> layer 1's state -> layer 2's gates -> layer 2's state, each step a fixed
// function; every wavefront reads and checks all of them.  Returns the number of values that were wrong, or waits given up.
template <int STEPS>
int call(int n_seq, int T, int wavefronts, int resident, unsigned seed)
{
    std::vector<std::atomic<int>> counters(counter_words(n_seq)), pre(n_seq * T), h1(n_seq * T), h2(n_seq * T);
    for (auto *v : {&counters, &pre, &h1, &h2})
        for (auto &a : *v) a = 0;
    std::atomic<int> bad{0};
    auto gates1 = [](int s, int t) { return 1000 * s + t + 1; };
    auto state1 = [&](int s, int t) { return 2 * gates1(s, t) + 1; };
    auto gates2 = [&](int s, int t) { return 3 * state1(s, t) + 1; };
    auto peek = [](std::atomic<int> &c) {
        static thread_local unsigned n = 0;
        if (++n % 64) std::this_thread::yield();
        else std::this_thread::sleep_for(std::chrono::microseconds(50));
        return c.load();
    };
    auto wait = [&](int want, int &seen, std::atomic<int> &c) {
        wait_for(want, seen, [&] { return peek(c); });
        if (seen == kGaveUp) ++bad;
    };
    auto gates = [&](int s, bool first) {                      // gates_ahead of the kernel, its wavefronts as one
        const int tokens = first ? kGateTokens : STEPS, rounds = (T + tokens - 1) / tokens;
        int seen = 0;
        for (int c = 0; c < rounds; ++c) {
            if (!first) wait((c + 1) * wavefronts, seen, counters[layer1_line(s)]);
            for (int t = c * tokens; t < T && t < (c + 1) * tokens; ++t) {
                if (!first && h1[s * T + t] != state1(s, t)) ++bad;
                pre[s * T + t] = first ? gates1(s, t) : gates2(s, t);
            }
            counters[first ? gates1_line(s) : gates2_line(s)] = chunks_there(c + 1, tokens, STEPS);
        }
    };
    auto layer = [&](int s, bool first) {
        Barrier barrier(wavefronts);
        auto wavefront = [&] {
            int seen = 0, t = 0;
            std::vector<int> next(STEPS), in(STEPS);
            auto fetch = [&](int c) {
                wait(c + 1, seen, counters[first ? gates1_line(s) : gates2_line(s)]);
                for (int i = 0; i < STEPS && c * STEPS + i < T; ++i) next[i] = pre[s * T + c * STEPS + i];
            };
            auto step = [&] {
                if (in[t % STEPS] != (first ? gates1(s, t) : gates2(s, t))) ++bad;
                ++t;
                barrier();
            };
            auto store = [&](int c) {
                for (int i = c * STEPS; i < T && i < (c + 1) * STEPS; ++i) (first ? h1 : h2)[s * T + i] = first ? state1(s, i) : 1;
            };
            auto post = [&] { counters[layer1_line(s)]++; };
            fetch(0);
            barrier();
            auto walk = [&](auto posts) {
                walk_chunks<STEPS, decltype(posts)::value>(T, [&](int) { in = next; }, store, step, fetch, post, barrier);
            };
            if (first) walk(std::true_type());
            else walk(std::false_type());
        };
        std::vector<std::thread> all;
        for (int w = 0; w < wavefronts; ++w) all.emplace_back(wavefront);
        for (auto &th : all) th.join();
    };
    std::atomic<int> started{0};
    auto slot = [&] {                                          // a compute unit: one workgroup after the other
        std::mt19937 rng(seed + started);
        while (started++ < 4 * n_seq) {
            std::this_thread::sleep_for(std::chrono::microseconds(rng() % 300));
            const Role r = role_of_four(counters[0]++, n_seq);
            if (r.what < 0 || r.what == 1) gates(r.seq, r.what < 0);
            else layer(r.seq, r.what == 0);
        }
    };
    std::vector<std::thread> slots;
    for (int i = 0; i < resident; ++i) slots.emplace_back(slot);
    for (auto &th : slots) th.join();
    for (auto &v : h2) bad += v != 1;
    return bad + (counters[0] != 4 * n_seq);
}
extern "C" int run_call(bool narrow, int n_seq, int T, int wavefronts, int resident, unsigned seed)
{
    return narrow ? call<kStepsNarrow>(n_seq, T, wavefronts, resident, seed) : call<kSteps>(n_seq, T, wavefronts, resident, seed);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("handover_roles")
    src, so = str(d / "model.cpp"), str(d / "model.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-pthread", "-Wall", "-Wno-unknown-pragmas", "-I" + CSRC, "-o", so, src],
                   check=True)
    return ctypes.CDLL(so)


@pytest.mark.parametrize("n_seq", [1, 2, 16, 64])
def test_four_roles(lib, n_seq):
    """4 * n_seq tickets are all roles of all sequences, layer 1's gates first; any other number stays in range."""
    def role(ticket):
        what, seq = ctypes.c_int(-9), ctypes.c_int(-9)
        lib.role4(ticket, n_seq, ctypes.byref(what), ctypes.byref(seq))
        return what.value, seq.value
    assert [role(t) for t in range(4 * n_seq)] == [(w, s) for w in range(-1, 3) for s in range(n_seq)]
    for t in [-1, -2, -n_seq, -3 * n_seq - 1, -2**31, 2**31 - 1, 4 * n_seq, 0x7FC00000, -0x7FC00000]:
        what, seq = role(t)
        assert -1 <= what <= 2 and 0 <= seq < n_seq, t


@pytest.mark.parametrize("n_seq", [1, 2, 64, 85])
def test_counters_have_lines_of_their_own(lib, n_seq):
    at, used = [ctypes.c_int() for _ in range(3)], [0]
    for s in range(n_seq):
        line = lib.lines(s, *map(ctypes.byref, at))
        used += [a.value for a in at]
    assert sorted(used) == list(range(0, lib.words(n_seq), line))      # the ticket's line, and three a sequence
    assert lib.words(n_seq) <= 64 * n_seq                              # fit the states of one token a sequence


@pytest.mark.parametrize("narrow", [False, True])
@pytest.mark.parametrize("T", list(range(1, 34)) + [89, 128, 333, 4096])
def test_reported_chunks_are_there(lib, narrow, T):
    """Layer 1's gates: a chunk is reported no sooner than all its tokens are stored, and every chunk in the end."""
    tokens, steps = lib.gate_tokens(), lib.steps_per_chunk(narrow)
    rounds, chunks = -(-T // tokens), -(-T // steps)
    for r in range(rounds + 1):
        stored = min(T, r * tokens)
        assert min(T, lib.there(r, tokens, steps) * steps) <= stored
    assert lib.there(rounds, tokens, steps) >= chunks


@pytest.mark.parametrize("narrow", [False, True])
@pytest.mark.parametrize("n_seq,T,wavefronts,resident", [
    (1, 1, 2, 1), (1, 40, 2, 4), (2, 33, 3, 1), (3, 17, 2, 12), (3, 64, 2, 5), (4, 9, 4, 3), (2, 8, 8, 2),
])
def test_whole_calls(lib, narrow, n_seq, T, wavefronts, resident):
    """Every state is made of its own inputs and every wait ends, also where one workgroup runs after the other."""
    for seed in range(3):
        assert lib.run_call(narrow, n_seq, T, wavefronts, resident, seed) == 0
