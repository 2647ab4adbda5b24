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

// The walk of one wavefront of an LSTM layer's workgroup over a sequence of T time steps:
//   take(c)    chunk c's inputs go where the steps read them
//   store(c)   its part of chunk c's states starts on its way to memory
//   step()     one time step; ends with a barrier of the workgroup
//   fetch(c)   chunk c's inputs are asked for
//   post()     waits for its stores, then adds one to the count of posts of all wavefronts
//   barrier()  a barrier of the workgroup
// The reader takes a count of (c + 1) * wavefronts for "chunk c has arrived".  That holds only while no
// wavefront posts twice before all others have posted once: between any two posts stands a barrier.
// Inside the walk the steps bring it (the post of chunk c - 1 follows at most three steps of chunk c);
// the last chunk may end right after that post, hence the barrier in front of the final one.
// The store of a chunk's states gets three steps to complete, the loads of the next chunk's inputs get the
// second half of a chunk.
template <int STEPS, bool POST, class Take, class Store, class Step, class Fetch, class Post, class Barrier>
SIDA_HD void walk_chunks(int T, Take &&take, Store &&store, Step &&step, Fetch &&fetch, Post &&post, Barrier &&barrier)
{
    const int chunks = (T + STEPS - 1) / STEPS;
    for (int c = 0; c < chunks; ++c) {
        const int n = T - c * STEPS < STEPS ? T - c * STEPS : STEPS;
        take(c);
        if (c > 0) store(c - 1);
        int i = 0;
#pragma clang loop unroll(disable)
        for (; i < (n < 3 ? n : 3); ++i) step();
        if (POST && c > 0) post();
#pragma clang loop unroll(disable)
        for (; i < (n < STEPS / 2 ? n : STEPS / 2); ++i) step();
        if (c + 1 < chunks) fetch(c + 1);
#pragma clang loop unroll(disable)
        for (; i < n; ++i) step();
    }
    store(chunks - 1);
    if (POST) {
        barrier();
        post();
    }
}

}  // namespace sida
