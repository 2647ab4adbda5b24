// How the workgroups of the LSTM recurrence (hash_fn.hip) hand chunks of time steps on to one another.
// Plain code for host and device: the protocol is checked without a GPU.
#pragma once

#if defined(__HIPCC__)
#define SIDA_HD __host__ __device__ __forceinline__
#else
#define SIDA_HD inline
#endif

namespace sida {

constexpr int kSteps = 8;        // time steps per chunk of the hand-over between the layers

// What a workgroup does, by the ticket it drew: layer 1 of a sequence (0), the gate pre-activations between
// the layers (1), layer 2 (2).  Any number is a valid ticket: the counters stand in the caller's workspace,
// and another call that uses it meanwhile (not allowed, and wrong results for both) may write over them.
struct Role {
    int what, seq;
};
SIDA_HD Role role_of(int ticket, int n_seq)
{
    const unsigned t = (unsigned)ticket, what = t / (unsigned)n_seq;
    return Role{what < 2u ? (int)what : 2, (int)(t % (unsigned)n_seq)};
}

// Waits until the counter that peek() reads has reached `want`; `seen` is the most that it has shown.  In a
// call that has its workspace to itself the counter gets there within microseconds: what is waited for is the
// next chunk of a workgroup that already runs.  Another call that clears or writes over the counter would be
// waited for without end, so a wait gives up after kMostPeeks (about a second), and every later one with it.
constexpr int kMostPeeks = 1 << 20, kGaveUp = 0x7fffffff;
template <class Peek>
SIDA_HD void wait_for(int want, int &seen, Peek &&peek)
{
    if (seen >= want) return;
    int left = kMostPeeks, now;
#pragma clang loop unroll(disable)
    while ((now = peek()) < want)
        if (--left == 0) {
            seen = kGaveUp;
            return;
        }
    seen = now;
}

// The walk of one wavefront of an LSTM layer's workgroup over a sequence of T time steps:
//   take(c)    chunk c's inputs go where the steps read them
//   store(c)   its part of chunk c's states starts on its way to memory
//   step()     one time step; ends with a barrier of the workgroup
//   fetch(c)   chunk c's inputs are asked for
//   post()     waits for its stores, then adds one to the count of posts of all wavefronts
//   barrier()  a barrier of the workgroup
// The reader takes a count of (c + 1) * wavefronts for "chunk c has arrived".  That holds only while no
// wavefront posts twice before all others have posted once: between any two posts stands a barrier.
// Inside the walk the steps bring it (the post of chunk c - 1 follows at most two steps of chunk c);
// the last chunk may end right after that post, hence the barrier in front of the final one.
// The store of a chunk's states gets two steps to complete, the loads of the next chunk's inputs the last two
// of a chunk: each step more is a step by which the second layer ends later.  Measured at both widths, also where
// the layers run one after the other and nobody follows, against three steps and the second half of a chunk
// (us a call, d = 768, 6 x 128 experts, one per token):
//             1 x 128          8 x 333          64 x 128         96 x 85 (layer after layer)
//   C = 128   112.8 -> 111.5   260.2 -> 258.6   168.2 -> 166.6   201.8 -> 201.4
//   C = 64     74.8 ->  73.9   166.9 -> 166.0   107.9 -> 106.9   123.8 -> 123.6
// Loads that nobody is waited for need no more than two steps (96 x 85 with loads after step 2: 201.8 and 123.8).
// Posts after one step are 0.5 us less at C = 128 and up to 1 us more at C = 64 (8 x 333); loads after step 7
// are within 0.5 us of these everywhere.
constexpr int kPostAfter = 2, kFetchAfter = kSteps - 2;
template <int STEPS, bool POST, class Take, class Store, class Step, class Fetch, class Post, class Barrier>
SIDA_HD void walk_chunks(int T, Take &&take, Store &&store, Step &&step, Fetch &&fetch, Post &&post, Barrier &&barrier)
{
    static_assert(kPostAfter <= kFetchAfter && kFetchAfter <= STEPS, "steps of a chunk");
    const int chunks = (T + STEPS - 1) / STEPS;
    for (int c = 0; c < chunks; ++c) {
        const int n = T - c * STEPS < STEPS ? T - c * STEPS : STEPS;
        take(c);
        if (c > 0) store(c - 1);
        if (n == STEPS) {                                      // written out: a step's addresses become constants
#pragma unroll
            for (int i = 0; i < kPostAfter; ++i) step();
            if (POST && c > 0) post();
#pragma unroll
            for (int i = kPostAfter; i < kFetchAfter; ++i) step();
            if (c + 1 < chunks) fetch(c + 1);
#pragma unroll
            for (int i = kFetchAfter; i < STEPS; ++i) step();
        } else {                                               // the last chunk
            int i = 0;
#pragma clang loop unroll(disable)
            for (; i < (n < kPostAfter ? n : kPostAfter); ++i) step();
            if (POST && c > 0) post();
#pragma clang loop unroll(disable)
            for (; i < n; ++i) step();
        }
    }
    store(chunks - 1);
    if (POST) {
        barrier();
        post();
    }
}

}  // namespace sida
