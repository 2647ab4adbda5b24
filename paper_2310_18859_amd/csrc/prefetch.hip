// Expert prefetch: brings the missing experts of one wave from pinned host memory into their pool
// slots (Section 3.1: the activated experts are loaded ahead of the forward pass), in the slot
// layout the grouped FFN reads (kernels.h).
//
// One hipMemcpyAsync per expert pays a fixed cost per copy: with 9.4 MB experts the copy engine
// reaches about 45 GB/s where a single large copy reaches 57 GB/s.  A kernel that reads the pinned
// blocks over the host link itself has no per-expert cost; 256 KiB in flight saturate the
// link (57 GB/s measured), one launch per wave, and it writes the slot layout directly.  The
// kernel runs on a few compute units of its own (sida_streams_create): a grouped GEMM that shares
// a compute unit with lanes waiting on host-link reads is slowed by them.
// With the copy engine the host block lands in the slot as it is and a second, in-place kernel
// re-orders it.
#include <hip/hip_runtime.h>

#include "kernels.h"

namespace sida {

namespace {

constexpr int kTilePieces = 32 * 16;      // 32 rows by 16 pieces: 8 KiB of the host block, and of the slot
constexpr int kCopyWorkgroups = 16;
constexpr int kCopyWavefronts = 32;       // of the whole grid: 8 KiB in flight in each
constexpr int kCopyWaves = 4;             // of a workgroup, at most
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Bound by the host link.  A wavefront moves a tile of 32 rows by 16 pieces (16 bytes each) at a time: 256
// bytes of four rows per load, eight loads in flight, turned around in LDS so that the tile is written as
// the 8 KiB run that it is in the slot.  The wavefronts of the grid walk the experts of the wave together,
// tile after tile: neighbours read neighbouring runs, and all end at the same time whatever the number of
// experts.
// Whole-line writes are what counts: with 16-byte writes scattered over the slot (linear reads, no LDS) the
// rate depends on how little the writes of one wavefront meet the reads of another - 45 to 56 GB/s, down to
// 25 on 8 compute units - and no number of loads in flight mends it.
// 9.4 MB experts on 16 compute units, scattered 16-byte writes before and now: 1 expert 49.1 -> 52.6 GB/s, 3
// 53.6 -> 55.8, 8 53.8 -> 56.8, 16 54.1 -> 57.1, 64 52.7 -> 57.3; on 8 compute units 24 to 46 -> 52.5 to 57.1.
// One large copy by the copy engine: 57.6.
__global__ __launch_bounds__(64 * kCopyWaves) void copy_experts(const CopyTable tbl, int tiles_in, int tiles, int kpr_in,
                                                               int kpr_out)
{
    __shared__ u32x4 lds[kCopyWaves][kTilePieces];
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    u32x4 *tile = lds[wave];
    const int waves = blockDim.x / 64, total = tbl.n * tiles;
    for (int c = __builtin_amdgcn_readfirstlane(blockIdx.x * waves + wave); c < total; c += gridDim.x * waves) {
        const int e = c / tiles, t = c - e * tiles;
        const bool second = t >= tiles_in;
        const int first = second ? tiles_in : 0, kpr = second ? kpr_out : kpr_in;
        const int stripe = (t - first) / (kpr / 16), piece = (t - first) % (kpr / 16) * 16;
        const u32x4 *__restrict__ src = static_cast<const u32x4 *>(tbl.src[e]) + (size_t)first * kTilePieces
                                        + (size_t)(stripe * 32 + lane / 16) * kpr + piece + lane % 16;
        u32x4 *__restrict__ dst = static_cast<u32x4 *>(tbl.dst[e]) + (size_t)t * kTilePieces + lane;
        u32x4 v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = src[(size_t)(i * 4) * kpr];
        // piece p of row r at 32 p + (r ^ p): sixteen lanes take the sixteen 16-byte bank groups both ways
#pragma unroll
        for (int i = 0; i < 8; ++i) tile[lane % 16 * 32 + ((i * 4 + lane / 16) ^ lane % 16)] = v[i];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // plain stores: a wave's experts (150 MB at the bench workload) stay in the 256 MB Infinity Cache
        // until the wave's GEMMs read them
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int p = i * 2 + lane / 32;
            dst[i * 64] = tile[p * 32 + (lane % 32 ^ p)];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// In-place re-ordering of slots that hold plain copies of host blocks: one workgroup per stripe of
// 32 rows (the same bytes in both layouts).  Every thread reads its pieces, the workgroup waits
// for all reads, then every thread writes: nothing is overwritten before it was read.
constexpr int kRelayoutThreads = 1024;
constexpr int kRelayoutPieces = 32 * (kMaxRelayoutK / 8) / kRelayoutThreads;   // per thread, at most

__global__ __launch_bounds__(kRelayoutThreads) void relayout_slots(const CopyTable tbl, int stripes_in, int kpr_in,
                                                                   int kpr_out, size_t pieces_in)
{
    u32x4 *slot = static_cast<u32x4 *>(tbl.dst[blockIdx.y]);
    const bool second = (int)blockIdx.x >= stripes_in;
    const int stripe = second ? blockIdx.x - stripes_in : blockIdx.x;
    const int kpr = second ? kpr_out : kpr_in;
    u32x4 *base = slot + (second ? pieces_in : 0) + (size_t)stripe * 32 * kpr;
    const int n = 32 * kpr;                                   // pieces of the stripe
    u32x4 v[kRelayoutPieces];
#pragma unroll
    for (int i = 0; i < kRelayoutPieces; ++i) {
        const int j = i * kRelayoutThreads + threadIdx.x;     // row-major piece (r, p) = (j / kpr, j % kpr)
        v[i] = base[j < n ? j : n - 1];                       // unconditional loads
    }
    __syncthreads();                                          // waits for this thread's loads, then for everyone's
#pragma unroll
    for (int i = 0; i < kRelayoutPieces; ++i) {
        const int j = i * kRelayoutThreads + threadIdx.x;
        if (j < n) {
            const int r = j / kpr, p = j - r * kpr;
            base[p * 32 + r] = v[i];
        }
    }
}

}  // namespace

int launch_expert_copy(const CopyTable &tbl, int32_t d, int32_t F, hipStream_t st)
{
    if (tbl.n <= 0) return 0;
    // 256 KiB in flight keep the link full (a round trip takes some 3 us).  More of them only slow the GEMMs
    // that run beside the copy, which share the L2s with them: GEMM 1 of a wave takes 35 us beside 16
    // workgroups of 256 threads, 41 beside 32, 45 beside 64.  One workgroup per compute unit of the stream,
    // up to 16; where it has 8, four wavefronts in each (two: 53 GB/s).
    const int cus = stream_compute_units(st), grid = cus < kCopyWorkgroups ? cus : kCopyWorkgroups;
    const int tiles_in = (int)((size_t)F * d / 8 / kTilePieces);    // d and F are multiples of 128
    hipLaunchKernelGGL(copy_experts, dim3(grid), dim3(64 * (kCopyWavefronts / grid)), 0, st, tbl, tiles_in, 2 * tiles_in,
                       d / 8, F / 8);
    return (int)hipGetLastError();
}

int launch_slot_relayout(const CopyTable &tbl, int32_t d, int32_t F, hipStream_t st)
{
    if (tbl.n <= 0) return 0;
    if (d > kMaxRelayoutK || F > kMaxRelayoutK) return (int)hipErrorInvalidValue;
    hipLaunchKernelGGL(relayout_slots, dim3(F / 32 + d / 32, tbl.n), dim3(kRelayoutThreads), 0, st, tbl, F / 32, d / 8, F / 8,
                       (size_t)F * d / 8);
    return (int)hipGetLastError();
}

}  // namespace sida
