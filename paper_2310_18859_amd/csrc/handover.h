// How the workgroups of the LSTM recurrence (hash_fn.hip) hand chunks of time steps on to one another.
// Plain code for host and device: the protocol is checked without a GPU.
#pragma once

#if defined(__HIPCC__)
#define SIDA_HD __host__ __device__ __forceinline__
#else
#define SIDA_HD inline
#endif

namespace sida {

// Time steps per chunk of the hand-over between the layers, of layers 128 wide and of narrower ones.  Layer 2 ends about
// two chunks behind layer 1, so a short chunk ends earlier: eight steps and four, us a call, C = 128: 1 x 128 tokens
// 112.2 -> 107.5, 8 x 333 260.9 -> 254.2, 64 x 128 167.3 -> 161.9, 2 x 512 351.8 -> 344.1, 96 x 85 (layer after layer)
// 202.7 -> 201.3.  A chunk's own work is the same for any width; at C = 64, where a step is shorter, it makes 8 x 333
// tokens slower (167.9 -> 170.6; 1 x 128 74.0 -> 72.4).
constexpr int kSteps = 4, kStepsNarrow = 8;

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
// The same with layer 1's own gate pre-activations among the roles (-1), in front of the others.
SIDA_HD Role role_of_four(int ticket, int n_seq)
{
    return (unsigned)ticket < (unsigned)n_seq ? Role{-1, ticket} : role_of((int)((unsigned)ticket - (unsigned)n_seq), n_seq);
}

// Counters of one call: the tickets drawn, then per sequence a 64-byte line each for the progress of layer 1's states
// (chunks times wavefronts), of layer 2's inputs and of layer 1's inputs (chunks).
constexpr int kLine = 16;        // words
SIDA_HD constexpr int counter_words(int n_seq) { return kLine * (1 + 3 * n_seq); }
SIDA_HD constexpr int layer1_line(int seq) { return kLine * (1 + 3 * seq); }
SIDA_HD constexpr int gates2_line(int seq) { return layer1_line(seq) + kLine; }
SIDA_HD constexpr int gates1_line(int seq) { return layer1_line(seq) + 2 * kLine; }

// Gate pre-activations are made for some tokens at a time, whole chunks: layer 1's for kGateTokens, layer 2's for a chunk.
// Chunks there when `rounds` of them have been stored; the reader waits for c + 1 before it loads chunk c.
constexpr int kGateTokens = 8;
SIDA_HD constexpr int chunks_there(int rounds, int tokens, int steps) { return rounds * (tokens / steps); }

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
// The store of a chunk's states gets a quarter of a chunk to complete, the loads of the next chunk's inputs its last
// quarter: each step more is a step by which the second layer ends later.  Chunks of four steps, posts and loads after
// steps 1 and 3, 2 and 2, 1 and 2, 2 and 3 (C = 128, us a call, d = 768, 6 x 128 experts, one per token; 8 x 333 three):
//   1 x 128 107.5, 109.9, 108.1, 107.9;  8 x 333 254.2, 259.1, 256.6, 254.8;  64 x 128 161.9, 164.4, 162.7, 162.5
// Chunks of eight, after steps 2 and 6 and after 3 and 4: C = 64 1 x 128 73.9 and 74.8, 8 x 333 166.0 and 166.9, 64 x 128
// 106.9 and 107.9, 96 x 85 (layer after layer) 123.6 and 123.8; posts after one step up to 1 us more (8 x 333).
template <int STEPS>
constexpr int kPostAfter = STEPS / 4;
template <int STEPS>
constexpr int kFetchAfter = STEPS - STEPS / 4;
template <int STEPS, bool POST, class Take, class Store, class Step, class Fetch, class Post, class Barrier>
SIDA_HD void walk_chunks(int T, Take &&take, Store &&store, Step &&step, Fetch &&fetch, Post &&post, Barrier &&barrier)
{
    static_assert(kPostAfter<STEPS> <= kFetchAfter<STEPS> && kFetchAfter<STEPS> <= STEPS, "steps of a chunk");
    const int chunks = (T + STEPS - 1) / STEPS;
    for (int c = 0; c < chunks; ++c) {
        const int n = T - c * STEPS < STEPS ? T - c * STEPS : STEPS;
        take(c);
        if (c > 0) store(c - 1);
        if (n == STEPS) {                                      // written out: a step's addresses become constants
#pragma unroll
            for (int i = 0; i < kPostAfter<STEPS>; ++i) step();
            if (POST && c > 0) post();
#pragma unroll
            for (int i = kPostAfter<STEPS>; i < kFetchAfter<STEPS>; ++i) step();
            if (c + 1 < chunks) fetch(c + 1);
#pragma unroll
            for (int i = kFetchAfter<STEPS>; i < STEPS; ++i) step();
        } else {                                               // the last chunk
            int i = 0;
#pragma clang loop unroll(disable)
            for (; i < (n < kPostAfter<STEPS> ? n : kPostAfter<STEPS>); ++i) step();
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
