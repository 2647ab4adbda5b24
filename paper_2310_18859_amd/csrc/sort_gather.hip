// K-a: token -> expert stable counting sort and permute-gather.
//
// Any implementation that invokes only the experts that have tokens (Section 2.3) must bring the
// rows of one expert together.  The order is fixed as (expert id, token index) so that the result
// is unique: perm[offsets[e] + j] is the j-th smallest token index routed to expert e.
//
// By size of the call: one workgroup (sort_one, up to 4096 tokens), one launch of independent
// workgroups (sort_chunks, up to 65536 tokens), or three small launches (one workgroup doing the
// whole sort was measured at 20 us for 16384 tokens: the ballot ranking is VALU-bound on a single
// compute unit):
//   sort_hist   one wavefront per chunk of 256 tokens: LDS histogram of the chunk
//   sort_scan   one workgroup: per-expert totals, exclusive scan over experts (offsets), the
//               first output row of every (chunk, expert) pair, and the grouped FFN's token-tile
//               descriptors
//   sort_rank   one wavefront per chunk: rank of a token among equal ids = (tokens of that id in
//               earlier chunks) + (earlier rounds of this chunk) + (lower lanes of this round, by
//               wavefront ballots over the 8 id bits)
// plus the row gather (gather_rows, 16-byte accesses) when it is not folded into the first GEMM.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include "kernels.h"

namespace sida {

namespace {

constexpr int kChunk = 256;      // tokens that a wavefront ranks (4 rounds of 64); sort_one up to 512 tokens takes 64
constexpr int kMaxE = 256;

// The jobs of a launch, by value; row y of the grid does job y.
struct SortJobs {
    SortJob job[kSortJobs];
};
#define SIDA_SORT_JOB(j)                                    \
    const int32_t *__restrict__ ids = (j).ids;              \
    const float *__restrict__ alpha = (j).alpha;            \
    int32_t *__restrict__ counts = (j).counts;              \
    int32_t *__restrict__ offsets = (j).offsets;            \
    int32_t *__restrict__ perm = (j).perm;                  \
    int32_t *__restrict__ inv = (j).inv;                    \
    float *__restrict__ gate_perm = (j).gate_perm;          \
    TileDesc *__restrict__ tiles = (j).tiles;               \
    const LayerTable &tbl = (j).tbl

__device__ __forceinline__ int clamp_id(int k, int E) { return k < 0 ? 0 : (k >= E ? E - 1 : k); }

__global__ __launch_bounds__(64) void sort_hist(const int32_t *__restrict__ ids, int T, int E,
                                                int32_t *__restrict__ block_hist)
{
    __shared__ int hist[kMaxE];
    const int lane = threadIdx.x;
    for (int e = lane; e < E; e += 64) hist[e] = 0;
    __syncthreads();
    const int base = blockIdx.x * kChunk;
#pragma unroll
    for (int r = 0; r < kChunk / 64; ++r) {
        const int t = base + r * 64 + lane;
        if (t < T) atomicAdd(&hist[clamp_id(ids[t], E)], 1);
    }
    __syncthreads();
    for (int e = lane; e < E; e += 64) block_hist[(size_t)blockIdx.x * E + e] = hist[e];
}

// One workgroup of 1024 threads: thread (p, e) owns expert e over quarter p of the chunks, so the
// walks over the chunks are short and their loads are issued 8 at a time.  Also expands the
// layer's expert table into the token-tile descriptors of the grouped FFN (thread i: entry i).
__global__ __launch_bounds__(1024) void sort_scan(int32_t *__restrict__ block_hist, int n_chunks, int E, int T,
                                                  int32_t *__restrict__ counts, int32_t *__restrict__ offsets,
                                                  const LayerTable tbl, TileDesc *__restrict__ tiles, int max_tiles)
{
    __shared__ int part[4][kMaxE];
    __shared__ int s_off[kMaxE + 1];
    __shared__ int s_wsum[4];
    const int tid = threadIdx.x, e = tid & 255, p = tid >> 8;
    const int per = (n_chunks + 3) / 4;
    const int b0 = p * per, b1 = min(n_chunks, b0 + per);

    int sum = 0;
    if (e < E)
        for (int b = b0; b < b1; b += 8) {
            int v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = b + i < b1 ? block_hist[(size_t)(b + i) * E + e] : 0;
#pragma unroll
            for (int i = 0; i < 8; ++i) sum += v[i];
        }
    part[p][e] = sum;
    __syncthreads();

    const int lane = tid & 63, wv = tid >> 6;
    int total = 0, incl = 0;
    if (tid < 256) {
        total = part[0][e] + part[1][e] + part[2][e] + part[3][e];
        if (e >= E) total = 0;
        incl = total;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_up(incl, o, 64);
            if (lane >= o) incl += v;
        }
        if (lane == 63) s_wsum[wv] = incl;
    }
    __syncthreads();
    if (tid < 256) {
        for (int i = 0; i < wv; ++i) incl += s_wsum[i];
        const int excl = incl - total;
        if (e < E) {
            counts[e] = total;
            offsets[e] = excl;
            s_off[e] = excl;
            if (e == E - 1) {
                offsets[E] = T;
                s_off[E] = T;
            }
        }
    }
    __syncthreads();

    // first output row of (chunk b, expert e) for this thread's chunks
    if (e < E) {
        int run = s_off[e];
        for (int q = 0; q < p; ++q) run += part[q][e];
        for (int b = b0; b < b1; b += 8) {
            int v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = b + i < b1 ? block_hist[(size_t)(b + i) * E + e] : 0;
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (b + i < b1) {
                    block_hist[(size_t)(b + i) * E + e] = run;
                    run += v[i];
                }
        }
    }

    if (tbl.n > 0) {
        int ex = 0, slot = 0, off = 0, cnt = 0, n_t = 0;
        if (tid < tbl.n) {
            ex = tbl.expert[tid];
            slot = tbl.slot[tid];
            off = s_off[ex];
            cnt = s_off[ex + 1] - off;
            n_t = (cnt + tbl.tile_m - 1) / tbl.tile_m;
        }
        __syncthreads();                                        // s_wsum is reused
        int inc2 = n_t;
        if (tid < 256) {
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int v = __shfl_up(inc2, o, 64);
                if (lane >= o) inc2 += v;
            }
            if (lane == 63) s_wsum[wv] = inc2;
        }
        __syncthreads();
        if (tid < 256) {
            for (int i = 0; i < wv; ++i) inc2 += s_wsum[i];
            int at = inc2 - n_t;
            for (int k = 0; k < n_t && at < max_tiles; ++k, ++at) {
                TileDesc td;
                td.slot = slot;
                td.row0 = off + k * tbl.tile_m;
                td.rows = min(tbl.tile_m, cnt - k * tbl.tile_m);
                td.expert = ex;
                tiles[at] = td;
            }
        }
    }
}

__global__ __launch_bounds__(64) void sort_rank(const int32_t *__restrict__ ids, int T, int E,
                                                const int32_t *__restrict__ block_base,
                                                int32_t *__restrict__ perm, int32_t *__restrict__ inv,
                                                const float *__restrict__ alpha, float *__restrict__ gate_perm)
{
    __shared__ int next_row[kMaxE];
    const int lane = threadIdx.x;
    for (int e = lane; e < E; e += 64) next_row[e] = block_base[(size_t)blockIdx.x * E + e];
    __syncthreads();
    const unsigned long long below = (1ull << lane) - 1ull;
    const int base = blockIdx.x * kChunk;
#pragma unroll
    for (int r = 0; r < kChunk / 64; ++r) {
        const int t = base + r * 64 + lane;
        const bool live = t < T;
        const int k = live ? clamp_id(ids[t], E) : 0;
        // lanes of this round that hold the same id
        unsigned long long same = __ballot(live);
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
            const unsigned long long b = __ballot((k >> bit) & 1);
            same &= ((k >> bit) & 1) ? b : ~b;
        }
        if (live) {
            const int ahead = __popcll(same & below);
            const int row = next_row[k] + ahead;
            perm[row] = t;
            inv[t] = row;
            if (alpha) gate_perm[row] = alpha[t];
        }
        __syncthreads();               // every lane has read next_row before anyone advances it
        if (live && (same & below) == 0) next_row[k] += __popcll(same);
        __syncthreads();
    }
}

// The whole sort in one workgroup for layer calls of up to 4096 tokens (from one or two sequences
// per batch, the paper's serving regime, upwards): wavefront w owns chunk w of ROUNDS * 64 tokens,
// the per-chunk histograms and bases live in LDS, and the three launches above shrink to one.
// Same results.  Up to 512 tokens a chunk is one round for each of the eight wavefronts: with chunks of
// 256 tokens one or two of them rank four rounds in a row, as three or four still do from 513 to 1024
// tokens.  Kernel time with gate values and 128 experts, before the one-round chunks and the early loads ->
// now: 256 tokens 5.0 -> 3.4 us, 512 5.1 -> 3.6, 513 5.2 -> 4.4, 1024 5.2 -> 4.5, 2048 5.6 -> 4.8, 2049
// 5.7 -> 5.6, 4096 6.8 -> 6.5; 8, 64 and 256 experts alike, but for 8 experts and 2049 tokens, 5.7 -> 5.9.  A layer
// of 8 experts and 256 tokens, one call behind another, 26.1 -> 23.8 us.  The three launches took 17-19 us with their gaps at 4096 tokens.
constexpr int kOneT = 4096;      // most tokens the single-workgroup sort takes

template <int NWV, int ROUNDS>
__global__ __launch_bounds__(NWV * 64) void sort_one(const SortJobs jobs, int T, int E, int max_tiles)
{
    SIDA_SORT_JOB(jobs.job[blockIdx.y]);
    constexpr int kTokens = ROUNDS * 64;           // of a wavefront
    __shared__ int hist[NWV][kMaxE];               // per-chunk histogram, then first output row of (chunk, expert)
    __shared__ int s_off[kMaxE + 1];
    __shared__ int s_wsum[4];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    // Everything that is read from memory is asked for here, so that its latency is paid once: a sort of one or two
    // sequences is little else (gate values and the expert table looked at where they are used: 2 us more).
    int my_id[ROUNDS];
    float my_alpha[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const int t = wv * kTokens + r * 64 + lane;
        my_id[r] = t < T ? ids[t] : 0;
        my_alpha[r] = alpha && t < T ? alpha[t] : 0.f;
    }
    int ex = 0, slot = 0;
    if (tid < tbl.n) {
        ex = tbl.expert[tid];
        slot = tbl.slot[tid];
    }
    for (int i = tid; i < NWV * kMaxE; i += NWV * 64) (&hist[0][0])[i] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        my_id[r] = wv * kTokens + r * 64 + lane < T ? clamp_id(my_id[r], E) : -1;
        if (my_id[r] >= 0) atomicAdd(&hist[wv][my_id[r]], 1);
    }
    __syncthreads();

    // expert totals -> offsets (threads 0..255: one expert each), then the bases of every chunk
    int total = 0, incl = 0;
    if (tid < 256) {
        if (tid < E)
            for (int c = 0; c < NWV; ++c) total += hist[c][tid];
        incl = total;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_up(incl, o, 64);
            if (lane >= o) incl += v;
        }
        if (lane == 63) s_wsum[wv] = incl;
    }
    __syncthreads();
    if (tid < 256) {
        for (int i = 0; i < wv; ++i) incl += s_wsum[i];
        const int excl = incl - total;
        if (tid < E) {
            counts[tid] = total;
            offsets[tid] = excl;
            s_off[tid] = excl;
            if (tid == E - 1) {
                offsets[E] = T;
                s_off[E] = T;
            }
            int run = excl;
            for (int c = 0; c < NWV; ++c) {
                const int v = hist[c][tid];
                hist[c][tid] = run;
                run += v;
            }
        }
    }
    __syncthreads();

    // token tiles of the grouped FFN (as in sort_scan)
    if (tbl.n > 0) {
        int off = 0, cnt = 0, n_t = 0;
        if (tid < tbl.n) {
            off = s_off[ex];
            cnt = s_off[ex + 1] - off;
            n_t = (cnt + tbl.tile_m - 1) / tbl.tile_m;
        }
        int inc2 = n_t;
        if (tid < 256) {
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int v = __shfl_up(inc2, o, 64);
                if (lane >= o) inc2 += v;
            }
        }
        __syncthreads();                                        // s_wsum is reused
        if (tid < 256 && lane == 63) s_wsum[wv] = inc2;
        __syncthreads();
        if (tid < 256) {
            for (int i = 0; i < wv; ++i) inc2 += s_wsum[i];
            int at = inc2 - n_t;
            for (int k = 0; k < n_t && at < max_tiles; ++k, ++at) {
                TileDesc td;
                td.slot = slot;
                td.row0 = off + k * tbl.tile_m;
                td.rows = min(tbl.tile_m, cnt - k * tbl.tile_m);
                td.expert = ex;
                tiles[at] = td;
            }
        }
    }

    // ranks: wavefront w walks its chunk in rounds of 64 tokens (LDS accesses of one wavefront
    // execute in program order, so the reads of a round precede its updates)
    const unsigned long long below = (1ull << lane) - 1ull;
    int *next_row = hist[wv];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const int t = wv * kTokens + r * 64 + lane;
        const bool live = my_id[r] >= 0;
        const int k = live ? my_id[r] : 0;
        unsigned long long same = __ballot(live);
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
            const unsigned long long b = __ballot((k >> bit) & 1);
            same &= ((k >> bit) & 1) ? b : ~b;
        }
        int row = 0;
        if (live) row = next_row[k] + __popcll(same & below);
        __builtin_amdgcn_wave_barrier();
        if (live && (same & below) == 0) next_row[k] += __popcll(same);
        __builtin_amdgcn_wave_barrier();
        if (live) {
            perm[row] = t;
            inv[t] = row;
            if (alpha) gate_perm[row] = my_alpha[r];
        }
    }
}

// The whole sort in ONE launch for calls between kOneT and kChunksT tokens, without any exchange
// between workgroups: workgroup c (one per chunk of kFineChunk tokens) histograms ALL ids itself - those
// before its chunk and the rest separately, 64 KiB of L2-resident ids at 16384 tokens - which gives
// it the expert totals (hence the offsets) and the number of tokens of every expert in earlier
// chunks, i.e. the first output row of each of its (chunk, expert) pairs; its first wavefront
// then ranks the chunk's tokens as sort_rank does.  Workgroup 0 also writes counts, offsets and the
// token tiles.  Same results as the three launches (17 us at 16384 tokens) in about half the time.
constexpr int kChunksT = 65536;
constexpr int kFineChunk = 128;                    // two ranking rounds per workgroup
constexpr int kIdLoads = 8;                        // 16-byte id loads in flight per thread
__global__ __launch_bounds__(256) void sort_chunks(const SortJobs jobs, int T, int E, int max_tiles)
{
    SIDA_SORT_JOB(jobs.job[blockIdx.y]);
    __shared__ int s_rest[kMaxE];                  // tokens per expert from this chunk on
    __shared__ int s_before[kMaxE];                // ... in earlier chunks, then the next output row
    __shared__ int s_off[kMaxE + 1];
    __shared__ int s_wsum[4];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int my0 = blockIdx.x * kFineChunk;
    s_rest[tid] = 0;
    s_before[tid] = 0;
    __syncthreads();
    // four ids per load, kIdLoads loads in flight per thread
    const int n4 = T >> 2;
    const int4 *ids4 = reinterpret_cast<const int4 *>(ids);
    for (int base = tid; base < n4; base += 256 * kIdLoads) {
        int4 v[kIdLoads];
#pragma unroll
        for (int u = 0; u < kIdLoads; ++u) v[u] = ids4[min(base + u * 256, n4 - 1)];   // unconditional loads
#pragma unroll
        for (int u = 0; u < kIdLoads; ++u)
            if (base + u * 256 < n4) {
                int *h = (base + u * 256) * 4 < my0 ? s_before : s_rest;   // chunks start at multiples of 4
                atomicAdd(&h[clamp_id(v[u].x, E)], 1);
                atomicAdd(&h[clamp_id(v[u].y, E)], 1);
                atomicAdd(&h[clamp_id(v[u].z, E)], 1);
                atomicAdd(&h[clamp_id(v[u].w, E)], 1);
            }
    }
    if (tid < (T & 3)) {                           // the last T % 4 ids
        const int t = (n4 << 2) + tid;
        atomicAdd(&(t < my0 ? s_before : s_rest)[clamp_id(ids[t], E)], 1);
    }
    __syncthreads();

    // expert totals -> offsets (thread e: expert e), then this chunk's first row per expert
    const int before = s_before[tid];
    int total = tid < E ? before + s_rest[tid] : 0, incl = total;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
    }
    if (lane == 63) s_wsum[wv] = incl;
    __syncthreads();
    for (int i = 0; i < wv; ++i) incl += s_wsum[i];
    const int excl = incl - total;
    if (tid < E) {
        s_off[tid] = excl;
        if (tid == E - 1) s_off[E] = T;
        s_before[tid] = excl + before;             // next output row of (this chunk, expert tid)
        if (blockIdx.x == 0) {
            counts[tid] = total;
            offsets[tid] = excl;
            if (tid == E - 1) offsets[E] = T;
        }
    }
    __syncthreads();

    // token tiles of the grouped FFN (as in sort_scan), by workgroup 0
    if (blockIdx.x == 0 && tbl.n > 0) {
        int ex = 0, slot = 0, off = 0, cnt = 0, n_t = 0;
        if (tid < tbl.n) {
            ex = tbl.expert[tid];
            slot = tbl.slot[tid];
            off = s_off[ex];
            cnt = s_off[ex + 1] - off;
            n_t = (cnt + tbl.tile_m - 1) / tbl.tile_m;
        }
        int inc2 = n_t;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_up(inc2, o, 64);
            if (lane >= o) inc2 += v;
        }
        __syncthreads();                           // s_wsum is reused
        if (lane == 63) s_wsum[wv] = inc2;
        __syncthreads();
        for (int i = 0; i < wv; ++i) inc2 += s_wsum[i];
        int at = inc2 - n_t;
        for (int k = 0; k < n_t && at < max_tiles; ++k, ++at) {
            TileDesc td;
            td.slot = slot;
            td.row0 = off + k * tbl.tile_m;
            td.rows = min(tbl.tile_m, cnt - k * tbl.tile_m);
            td.expert = ex;
            tiles[at] = td;
        }
    }

    // ranks: the first wavefront walks the chunk in rounds of 64 tokens (LDS accesses of one
    // wavefront execute in program order, so the reads of a round precede its updates)
    if (wv != 0) return;
    int *next_row = s_before;
    const unsigned long long below = (1ull << lane) - 1ull;
    int my_id[kFineChunk / 64];
#pragma unroll
    for (int r = 0; r < kFineChunk / 64; ++r) {
        const int t = my0 + r * 64 + lane;
        my_id[r] = t < T ? clamp_id(ids[t], E) : -1;
    }
#pragma unroll
    for (int r = 0; r < kFineChunk / 64; ++r) {
        const int t = my0 + r * 64 + lane;
        const bool live = my_id[r] >= 0;
        const int k = live ? my_id[r] : 0;
        unsigned long long same = __ballot(live);
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
            const unsigned long long b = __ballot((k >> bit) & 1);
            same &= ((k >> bit) & 1) ? b : ~b;
        }
        int row = 0;
        if (live) row = next_row[k] + __popcll(same & below);
        __builtin_amdgcn_wave_barrier();
        if (live && (same & below) == 0) next_row[k] += __popcll(same);
        __builtin_amdgcn_wave_barrier();
        if (live) {
            perm[row] = t;
            inv[t] = row;
            if (alpha) gate_perm[row] = alpha[t];
        }
    }
}

// Rows of d*2 bytes moved as 16-byte pieces.  A workgroup takes kGatherRows consecutive output rows:
// their source rows go to LDS first, then the rows' pieces are dealt to the 256 threads as one flat
// range (no lane idles whatever the row length - 96 pieces at d = 768), kGatherUnroll independent
// loads in flight per thread.
constexpr int kGatherRows = 8, kGatherUnroll = 4;
__global__ __launch_bounds__(256) void gather_rows(const uint4 *__restrict__ x, const int32_t *__restrict__ perm,
                                                   int T, int vec_per_row, uint4 *__restrict__ x_perm, int k)
{
    __shared__ int src_row[kGatherRows];
    const int row0 = blockIdx.x * kGatherRows;
    const int rows = min(kGatherRows, T - row0);
    if ((int)threadIdx.x < rows) {
        const int t = perm[row0 + threadIdx.x];
        src_row[threadIdx.x] = k == 1 ? t : t / k;            // row r belongs to token perm[r] / k
    }
    __syncthreads();
    const int n = rows * vec_per_row;                         // pieces of this workgroup
    uint4 *dst = x_perm + (size_t)row0 * vec_per_row;         // its output rows are one contiguous range
    for (int base = threadIdx.x; base < n; base += 256 * kGatherUnroll) {
        uint4 v[kGatherUnroll];
#pragma unroll
        for (int u = 0; u < kGatherUnroll; ++u) {             // unconditional loads (past the end: the last piece again)
            const int j = min(base + u * 256, n - 1);
            const int r = j / vec_per_row, i = j - r * vec_per_row;
            v[u] = x[(size_t)src_row[r] * vec_per_row + i];
        }
#pragma unroll
        for (int u = 0; u < kGatherUnroll; ++u)
            if (base + u * 256 < n) dst[base + u * 256] = v[u];
    }
}

}  // namespace

bool sort_in_one_launch(int32_t T) { return T <= kChunksT; }

int launch_sort(const SortJob *jobs, int32_t n, int32_t T, int32_t E, int32_t max_tiles, hipStream_t st)
{
    if (n < 1 || n > kSortJobs || (n > 1 && T > kChunksT)) return (int)hipErrorInvalidValue;
    // sort_chunks reads ids 16 bytes at a time: a job whose ids are off that boundary takes three launches of its own
    const auto joins = [&](const SortJob &j) {
        return T <= kOneT || (T <= kChunksT && (reinterpret_cast<uintptr_t>(j.ids) & 15u) == 0);
    };
    SortJobs a;
    int32_t m = 0;
    for (int32_t i = 0; i < n; ++i)
        if (joins(jobs[i])) a.job[m++] = jobs[i];
    if (m > 0) {
        if (T <= 8 * 64) hipLaunchKernelGGL((sort_one<8, 1>), dim3(1, m), dim3(512), 0, st, a, T, E, max_tiles);
        else if (T <= 8 * kChunk) hipLaunchKernelGGL((sort_one<8, kChunk / 64>), dim3(1, m), dim3(512), 0, st, a, T, E, max_tiles);
        else if (T <= kOneT) hipLaunchKernelGGL((sort_one<16, kChunk / 64>), dim3(1, m), dim3(1024), 0, st, a, T, E, max_tiles);
        else hipLaunchKernelGGL(sort_chunks, dim3((T + kFineChunk - 1) / kFineChunk, m), dim3(256), 0, st, a, T, E, max_tiles);
    }
    const int n_chunks = (T + kChunk - 1) / kChunk;
    for (int32_t i = 0; i < n; ++i) {
        const SortJob &j = jobs[i];
        if (joins(j)) continue;
        hipLaunchKernelGGL(sort_hist, dim3(n_chunks), dim3(64), 0, st, j.ids, T, E, j.block_hist);
        hipLaunchKernelGGL(sort_scan, dim3(1), dim3(1024), 0, st, j.block_hist, n_chunks, E, T, j.counts, j.offsets, j.tbl,
                           j.tiles, max_tiles);
        hipLaunchKernelGGL(sort_rank, dim3(n_chunks), dim3(64), 0, st, j.ids, T, E, j.block_hist, j.perm, j.inv, j.alpha,
                           j.gate_perm);
    }
    return (int)hipGetLastError();
}

int launch_gather(const void *x, const int32_t *perm, int32_t T, int32_t d, void *x_perm, hipStream_t st,
                  const LaunchEvents *ev, int32_t k)
{
    const int vec_per_row = d / 8;
    hipExtLaunchKernelGGL(gather_rows, dim3((T + kGatherRows - 1) / kGatherRows), dim3(256), 0, st, ev ? ev->start : nullptr,
                          ev ? ev->stop : nullptr, 0, (const uint4 *)x, perm, T, vec_per_row, (uint4 *)x_perm, k);
    return (int)hipGetLastError();
}

}  // namespace sida
