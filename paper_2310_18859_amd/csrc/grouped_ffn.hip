// K-b: grouped expert FFN on bf16 MFMA (gfx950).
//
// For every expert e of a wave, with its tokens in rows [offsets[e], offsets[e+1]) of x_perm:
//     h      = relu(x_perm_e * W_in[e]^T)      (GEMM 1, [rows, d] x [F, d]^T, ReLU, bf16 out)
//     y_perm = h * W_out[e]^T                  (GEMM 2, [rows, F] x [d, F]^T, bf16 out)
// which is the expert MLP f_i of Eq. 1 (Section 2.1) invoked only for experts that have tokens
// (Section 2.3).  Expert weights are read from the pool slot named by the wave table.
//
// Operand paths.  The two operands of a tile take different routes into the matrix cores:
//  * weights go global -> registers.  A pool slot holds an expert in MFMA-fragment order (see
//    kernels.h, "slot layout"): the 32 weight rows x 16 K values one 32x32x16 MFMA takes as its
//    first operand are 1 KiB of consecutive memory, lane l's 16 bytes at offset 16*l, so a
//    wavefront fetches a fragment with one fully coalesced 16-byte-per-lane load and nothing of
//    the weights passes through LDS.  Every weight fragment is used by exactly one wavefront;
//  * token rows go global -> LDS directly (buffer_load ... lds, no register staging) through a
//    ring of NB+1 stages of BM rows x 64 K values and are read as fragments by all wavefronts.
// Both run NB K-steps ahead of the MFMAs, across tile boundaries too: the weights in NB rotating
// register buffers (a buffer is refilled right after the MFMAs that consumed it), the tokens in
// the ring.  All loads use buffer descriptors (32-bit offsets; reads past a descriptor's end
// return zeros instead of faulting) - and, deliberately, no FLAT-encoded LDS loads: with those in
// flight the compiler must wait for ALL outstanding loads at every use of a loaded register.
//
// Tiling: a workgroup of NWV = 4 wavefronts computes BM tokens x (NWV*NS*32) weight rows; wavefront w
// owns NS stripes of 32 weight rows and all BM token rows, i.e. NS x BM/32 accumulator blocks of
// 32x32 (fp32).  Two workgroups share a compute unit (8 wavefronts, two per SIMD), so that one's
// result stores and tile switch overlap the other's MFMAs.  One LDS fragment read feeds NS MFMAs.
// Experts with few tokens take another kernel, or another role beside it in the same launch (stream_tile).
//
// LDS token tile layout: row r of a stage is 128 bytes; its 16-byte piece c is stored at piece
// position c ^ (r/2 & 7).  A direct-to-LDS load writes lane i's 16 bytes at offset 16*i of the
// instruction's 1 KiB window (8 rows), so lane i fetches the global piece that belongs at position i%8 of
// its row; the fragment reads (32 rows, same logical piece) then touch all 16 places of 256 bytes per 16
// rows, which LDS reads at a time, and are bank-conflict free without padding (with r & 7, rows 8 apart
// met: half of the LDS cycles were conflicts).
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <type_traits>

#include <cstddef>
#include <mutex>
#include <unordered_map>

#include "kernels.h"
#include "past_end.h"
#include "tile_order.h"

namespace sida {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;

// Waits until at most N of this wavefront's vector memory operations are outstanding (they
// complete in issue order).  Operations the kernel issues beyond the ones a count is derived
// from only make a wait stricter, never too weak.
template <int N>
__device__ __forceinline__ void wait_loads()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Raw buffer descriptor over [base, base + bytes).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000);
}
// 16 bytes per lane straight into LDS: lane i's piece lands at lds_dst + 16*i.
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t r, int voffset, int soffset, void *lds_dst)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)lds_dst, 16, voffset, soffset, 0, 0);
}
// One dword per lane into LDS: lane i's word lands at lds_dst + 4*i.
__device__ __forceinline__ void load_word_to_lds(__amdgpu_buffer_rsrc_t r, int voffset, void *lds_dst)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)lds_dst, 4, voffset, 0, 0, 0);
}
// STREAM: the non-temporal cache policy, for data that is read once (it is not kept in L2 at the
// expense of data that is read again).
template <bool STREAM>
__device__ __forceinline__ bf16x8 load_frag(__amdgpu_buffer_rsrc_t r, int voffset, int soffset)
{
    return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, voffset, soffset, STREAM ? 2 : 0));
}

// 16 bytes per lane out; lanes whose offset is past the descriptor's end write nothing.  The whole offset goes through the
// lanes' register: with part of it in a scalar register the compiler takes the registers of the 16 bytes as free in the
// next instruction, and a vector instruction there changed bytes that were still to be stored (seen as wrong rows where
// the store met a cold address translation).  Without, it keeps them for the wait state that such a store needs.
template <bool STREAM>
__device__ __forceinline__ void store_row_piece(__amdgpu_buffer_rsrc_t r, bf16x8 v, int offset)
{
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(i32x4, v), r, offset, 0, STREAM ? 2 : 0);
}

// FUSE selects what the token rows are addressed through:
//   kPlain    A rows and C rows are the tile's rows row0 .. row0+rows-1 (x_perm -> h -> y_perm);
//   kGather   A is x in token order: row r of the tile is read from x[perm[row0 + r] / top_k]
//             (GEMM 1 without a separate gather pass);
//   kScatter  C is y in token order: row r of the tile is scaled by gate_perm[row0 + r] (fp32
//             product of the bf16-rounded result, one more rounding to bf16 - the arithmetic of
//             the separate combine pass) and written to y[perm[row0 + r]] (GEMM 2 without a
//             separate combine pass; top-1 routing writes every y row exactly once).
// The row maps are fetched into a small private LDS buffer per wavefront with direct loads, a
// whole tile ahead of their use, so that no register-returning load has to be waited for.
enum { kPlain = 0, kGather = 1, kScatter = 2 };

constexpr int kWaves = 4;        // wavefronts per workgroup
constexpr int kFewStripes = 2;   // weight stripes per workgroup of a few-token tile beside larger ones
constexpr int kStreamLdsBytes = 32 * 1024;   // LDS of a few-token tile: kWaves parts of 64 x 32 sums

struct GemmArgs {
    const __bf16 *A;             // token rows [a_rows, K]
    __bf16 *C;                   // results [.., N]
    const char *pool;
    size_t expert_bytes, w_off;  // W_in at offset 0 of a slot, W_out behind it
    const TileDesc *tiles;
    int m_tiles, m_tall, gm, nw, N, K;      // gm x nw: block of the tile order (tile_order.h)
    int m_few, few_rows;         // few-token tiles behind the m_tiles others, and their rows
    int big_wgs;                 // workgroups that walk the m_tiles tiles
    uint32_t a_bytes, c_bytes;   // bytes of A and C
    const int32_t *perm;         // fused modes: row maps, `map_len` entries
    const float *gate_perm;
    int map_len, top_k;
};

// ---- experts with few tokens ----------------------------------------------------------------------
// An expert with few tokens is a stream of weights: one pass over W for at most 64 rows.  What counts is
// that every compute unit has enough of it in flight all the time and the same share of it.  One workgroup
// takes a token tile of at most 64 rows and NS stripes of 32 weight rows, and its four wavefronts split the
// sum over K, so that
//  * a wavefront's weights are one linear run, loaded D steps of 32 K values ahead into registers, with no
//    barrier before the end of the sum - where four partial sums meet in LDS - and
//  * a launch is many short workgroups (an expert's second GEMM: d/32 of them), which the hardware deals out
//    as others end: no workgroup's share of tiles is larger than another's.
// Token rows are loaded whole 64-byte pieces at a time (16 rows per load) and turned around in LDS, within
// the wavefront: loaded as matrix operands, 16 bytes of another row in every lane, each lane is a cache
// access of its own, and from about 8 rows on those bound the launch (128 experts x 23 tokens: 147 us; 113
// this way).  Rows past the tile's end are outside the buffer descriptor: no request.
// Measured against the 64-row tiles of the kernel below: 52 experts x 2.5 tokens 46 / 44 -> 39 / 40 us per
// GEMM (6.1 TB/s of weights), 128 x 12: 107 / 99 -> 95 / 97 us, 8 x 8: 11 / 14 -> 10 / 8 us.
// Sums in four parts are no less exact: outputs of layers of 21 to 1111 tokens (384 to 1024 columns) against sums in 64
// bits rounded to bf16 at the same places, relative 2-norms, 1.2e-4 walked and 0.8e-4 streamed (medians of 12);
// against 64 bits throughout, where the roundings to bf16 decide, 2.87e-3 both.
template <int NS, int MI, int D, bool RELU, int FUSE, bool ONCE>
__device__ __forceinline__ void stream_tile(const GemmArgs &g, const i32x4 &td, int stripe, f32x4 *red)
{
    constexpr int W = kWaves;
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int N = g.N, K = g.K, row0 = td.y, rows = td.z;
    const int n = K / (32 * W), k0 = wv * n;                    // this wavefront's steps of 32 K values
    const __amdgpu_buffer_rsrc_t w_rsrc = make_rsrc(g.pool + (size_t)td.x * g.expert_bytes + g.w_off, (uint32_t)N * (uint32_t)K * 2u);
    const __amdgpu_buffer_rsrc_t a_rsrc = make_rsrc(g.A, g.a_bytes);
    constexpr int kT = 2 * MI;
    int src[kT], dst[MI];
    float gate[MI];
#pragma unroll
    for (int j = 0; j < kT; ++j) {
        src[j] = row0 + min(j * 16 + (lane >> 2), rows - 1);
        if (FUSE == kGather) src[j] = g.perm[src[j]];
    }
#pragma unroll
    for (int m = 0; m < MI; ++m) {
        const int r = row0 + min(m * 32 + (lane & 31), rows - 1);
        dst[m] = r;
        if (FUSE == kScatter) {
            dst[m] = g.perm[r];
            gate[m] = g.gate_perm[r];
        }
    }
    bf16x8 w[D][2][NS], t[D][kT];
    auto load_w = [&](int i, int f) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int s = 0; s < NS; ++s)
                w[i][j][s] = load_frag<ONCE>(w_rsrc, lane * 16, (stripe * NS + s) * (32 * K * 2) + (k0 + f) * 2048 + j * 1024);
    };
    int tok_v[kT];
    auto find_rows = [&]() {
#pragma unroll
        for (int j = 0; j < kT; ++j) {
            if (FUSE == kGather && g.top_k != 1) src[j] /= g.top_k;
            // rows past the end are out of the descriptor's range: zeros, no request
            tok_v[j] = j * 16 + (lane >> 2) < rows ? src[j] * K * 2 + (lane & 3) * 16 : kPastEnd;
        }
    };
    auto load_t = [&](int i, int f) {
#pragma unroll
        for (int j = 0; j < kT; ++j) t[i][j] = load_frag<false>(a_rsrc, tok_v[j], (k0 + f) * 64);
    };
    f32x16 acc[NS][MI];
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int m = 0; m < MI; ++m)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[s][m][r] = 0.f;
    // token rows of a step, turned around in LDS: row r is 64 bytes, piece p at position p ^ (r/4 & 3)
    char *turn = reinterpret_cast<char *>(red) + wv * (MI * 4096);
    const int put_at = (lane >> 2) * 64 + (((lane & 3) ^ ((lane >> 4) & 3)) * 16);
    int get_at[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) get_at[j] = (lane & 31) * 64 + (((j * 2 + half) ^ ((lane >> 2) & 3)) * 16);
    auto multiply = [&](int i) {
        char *slot = turn + (i & 1) * (MI * 2048);
#pragma unroll
        for (int j = 0; j < kT; ++j) *reinterpret_cast<bf16x8 *>(slot + j * 1024 + put_at) = t[i][j];
#pragma unroll
        for (int m = 0; m < MI; ++m)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const bf16x8 x = *reinterpret_cast<const bf16x8 *>(slot + m * 2048 + get_at[j]);
#pragma unroll
                for (int s = 0; s < NS; ++s) acc[s][m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[i][j][s], x, acc[s][m], 0, 0, 0);
            }
    };
    // Loads run D steps ahead.  Tiles of at most 32 rows load every step once: with the last step loaded again where
    // D steps ahead are past the end, K = 1024 cost 12 loads for 8 steps (64 experts x 16 tokens, 1024 x 4096: first
    // GEMM 106 us, 93 this way; 200 x 24 tokens, 384 x 1536: 67 and 54).  A load under a branch is waited for as if it
    // had not been made, too early for the loads behind it; hence no branch in the loop, and a sum of at most D steps
    // written out for each length.  Taller tiles (D = 3) do repeat the last step: at most two loads too many, and the
    // form without them is slower (8 experts x 48 tokens, second GEMM: 10.1 us against 11.2).
    auto start = [&](auto steps) {
#pragma unroll
        for (int i = 0; i < decltype(steps)::value; ++i) load_w(i, min(i, n - 1));
        find_rows();
#pragma unroll
        for (int i = 0; i < decltype(steps)::value; ++i) load_t(i, min(i, n - 1));
        __builtin_amdgcn_sched_barrier(0);                      // all in flight before the first product
    };
    if constexpr (MI > 1) {
        start(std::integral_constant<int, D>());
        int f = 0;
#pragma clang loop unroll(disable)
        for (; f + D < n; f += D) {
#pragma unroll
            for (int i = 0; i < D; ++i) {
                multiply(i);
                const int at = min(f + D + i, n - 1);
                load_w(i, at);
                load_t(i, at);
            }
        }
#pragma unroll
        for (int i = 0; i < D; ++i)
            if (i == 0 || f + i < n) multiply(i);
    } else if (n <= D) {
        auto short_sum = [&](auto steps) {
            if (n != decltype(steps)::value) return;
            start(steps);
#pragma unroll
            for (int i = 0; i < decltype(steps)::value; ++i) multiply(i);
        };
        static_assert(MI > 1 || D == 6, "lengths written out");
        short_sum(std::integral_constant<int, 6>());
        short_sum(std::integral_constant<int, 5>());
        short_sum(std::integral_constant<int, 4>());
        short_sum(std::integral_constant<int, 3>());
        short_sum(std::integral_constant<int, 2>());
        short_sum(std::integral_constant<int, 1>());
    } else {
        start(std::integral_constant<int, D>());
        int f = 0;
#pragma clang loop unroll(disable)
        for (; f + 2 * D <= n; f += D) {
#pragma unroll
            for (int i = 0; i < D; ++i) {
                multiply(i);
                load_w(i, f + D + i);
                load_t(i, f + D + i);
            }
        }
        const int left = n - f;                                 // D .. 2 D - 1
#pragma unroll
        for (int i = 0; i < D; ++i) {
            multiply(i);
            if (D + i < left) {
                load_w(i, f + D + i);
                load_t(i, f + D + i);
            }
        }
#pragma unroll
        for (int i = 0; i < D - 1; ++i)
            if (D + i < left) multiply(i);
    }
    // Where the results go is looked at here and no earlier: a wait for these loads, the kernel's first, would be a
    // wait in front of the sum.
    if (FUSE == kScatter)
#pragma unroll
        for (int m = 0; m < MI; ++m) asm volatile("" : "+v"(dst[m]), "+v"(gate[m]));
    // The parts of the sum meet in LDS, stripe by stripe.  A lane holds 4 x 4 consecutive output columns
    // 8q + 4*half .. of its token; wavefront q sums column group q.
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        if (s) __syncthreads();
#pragma unroll
        for (int m = 0; m < MI; ++m)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                red[((wv * MI + m) * 4 + q) * 64 + lane] = f32x4{acc[s][m][4 * q], acc[s][m][4 * q + 1], acc[s][m][4 * q + 2], acc[s][m][4 * q + 3]};
        __syncthreads();
#pragma unroll
        for (int m = 0; m < MI; ++m) {
            const int q = wv, token = m * 32 + (lane & 31);
            f32x4 v = red[(m * 4 + q) * 64 + lane];
#pragma unroll
            for (int p = 1; p < W; ++p) v += red[((p * MI + m) * 4 + q) * 64 + lane];
            bf16x4 o;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float e = v[j];
                if (RELU) e = e > 0.f ? e : 0.f;
                o[j] = (__bf16)e;
                if (FUSE == kScatter) o[j] = (__bf16)(gate[m] * (float)o[j]);
            }
            if (token < rows) *reinterpret_cast<bf16x4 *>(g.C + (size_t)dst[m] * N + (stripe * NS + s) * 32 + q * 8 + half * 4) = o;
        }
    }
}

// Workgroup `block` of the few-token tiles: which tile and stripe.  Workgroup b runs on XCD b % 8 (round-robin
// dispatch); the stripes of a token tile stay on one XCD, so that its rows are fetched into one L2.  Tiles
// are dealt to the XCDs in turn, back and forth (they come with the most tokens first), and the stripes of
// the last, incomplete round to all XCDs.
template <int NS, bool RELU, int FUSE, bool ONCE>
__device__ __forceinline__ void stream_block(const GemmArgs &g, int block, f32x4 *red)
{
    const int stripes = g.N / (32 * NS), rounds = g.m_few >> 3;
    const int xcd = block & 7, local = block >> 3;
    int mt = local / stripes, stripe = local - mt * stripes;
    if (mt < rounds) {
        mt = mt * 8 + ((mt & 1) ? 7 - xcd : xcd);
    } else {
        const int j = (local - rounds * stripes) * 8 + xcd;
        mt = rounds * 8 + j / stripes;
        stripe = j % stripes;
        if (mt >= g.m_few) return;
    }
    typedef const __attribute__((address_space(4))) i32x4 *ConstTiles;
    const i32x4 td = ((ConstTiles)(uintptr_t)(g.tiles + g.m_tiles))[mt];   // slot, row0, rows, expert
    if (td.z > 32) stream_tile<NS, 2, 3, RELU, FUSE, ONCE>(g, td, stripe, red);
    else stream_tile<NS, 1, 6, RELU, FUSE, ONCE>(g, td, stripe, red);
}

template <int NS, bool RELU, int FUSE, bool ONCE>
__global__ __launch_bounds__(kWaves * 64, NS == 1 ? 3 : 2) void stream_gemm_nt(const GemmArgs g)
{
    __shared__ f32x4 red[kStreamLdsBytes / sizeof(f32x4)];
    stream_block<NS, RELU, FUSE, ONCE>(g, blockIdx.x, red);
}

// Persistent workgroups: two per compute unit, each walks its tiles t = b, b+G, ...
//
// (tile, K-step) is ONE stream of steps: the loads run NB steps ahead of the MFMAs (K/64 is a
// multiple of NB), also across
// tile boundaries (the last NB steps of a tile already fetch the next one; behind a workgroup's last tile
// they ask for nothing, see point_nowhere).
// Per step a wavefront executes: one s_waitcnt, one s_barrier, its share of the token loads, and
// per 16 K values BM/32 LDS fragment reads, NS*BM/32 MFMAs and NS weight-fragment loads.
//
// ONCE: the weights of single-tile experts are streamed past L2's replacement (worth_streaming), and so are the results,
// which would push the many-token experts' weights and the token rows out of the L2s.  128 experts, 16384 tokens, GEMMs
// 155.6 / 160.1 -> 153.2 / 159.0 us, layers of 128 experts x 4096 tokens 4 % faster; but with 16 experts x 4096 tokens,
// whose weights the Infinity Cache holds, 5 % slower, and 7 % with 64 experts x 8192 tokens of 384 x 1536.
// Narrow tiles (NS = 1) take part, though their row pieces are 64 bytes, half a line, and the halves leave apart (second GEMM
// of 128 experts, 16384 tokens: 30.3 MB written for 25.2): with the default policy for theirs, us a pass of all layers, 64 experts
// x 1111 tokens 652 -> 667, 64 x 8192 1039 -> 1045, 128 x 16384 1843 -> 1870, three experts per token 1904 -> 1910.
template <int BM, int NS, int NB, bool RELU, int FUSE, bool ONCE>
__global__ __launch_bounds__(kWaves * 64, 2) void grouped_gemm_nt(const GemmArgs g)
{
    constexpr int NWV = kWaves, BN = NWV * NS * 32;
    constexpr int TS = NB + 1;                                  // token ring stages
    constexpr int kStageBytes = BM * 128;
    constexpr int kRingBytes = TS * kStageBytes;
    constexpr int QN = BM / 8;                                  // direct loads (1 KiB = 8 rows) per stage
    constexpr int TL = QN / NWV;                                // ... per wavefront
    constexpr int MI = BM / 32;
    constexpr int KS = 4;                                       // MFMA K sub-steps per K-step of 64
    constexpr int kOutCols = NS * 32;                           // output columns of a wavefront
    constexpr int kOutPitch = kOutCols * 2 + 16;                // staging row pitch in bytes
    constexpr int LPR = kOutCols * 2 / 16;                      // lanes per output-row segment
    constexpr int RPI = 64 / LPR;                               // rows per store instruction
    constexpr int STORES = MI * (32 / RPI);                     // result stores per thread per tile
    constexpr int kStepOps = TL + KS * NS;                      // loads per thread per K-step
    constexpr int kBase = (NB - 1) * kStepOps;                  // at the start of a K-step, everything issued NB steps ago must have landed
    constexpr int kStage = NWV * 32 * kOutPitch;                // result staging, 32 rows per wavefront
    constexpr int kSide = FUSE == kPlain ? 0 : (FUSE == kGather ? 256 : 2 * BM * 4);   // row maps, per wavefront
    static_assert(QN % NWV == 0 && TL * 8 <= 64, "token loads per wavefront");
    static_assert(kBase + STORES + 4 <= 63, "vmcnt range");
    static_assert(kRingBytes + kStage + NWV * kSide <= 80 * 1024, "two workgroups per compute unit");
    static_assert(kRingBytes + kStage >= kStreamLdsBytes, "the few-token tiles' LDS");

    extern __shared__ __attribute__((aligned(1024))) char lds[];
    if ((int)blockIdx.x >= g.big_wgs) {
        f32x4 *red = reinterpret_cast<f32x4 *>(lds);
        stream_block<kFewStripes, RELU, FUSE, ONCE>(g, (int)blockIdx.x - g.big_wgs, red);
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    char *stg = lds + kRingBytes + wv * (32 * kOutPitch);
    char *side = lds + kRingBytes + kStage + wv * kSide;        // this wavefront's row maps (FUSE != kPlain)
    const int N = g.N, K = g.K;
    const int n_tiles_n = N / BN;
    const int total = g.m_tiles * n_tiles_n;
    const int G = g.big_wgs, wg = blockIdx.x;
    if (wg >= total) return;
    const int n = (total - wg + G - 1) / G;                     // tiles of this workgroup
    const int nkk = K / (64 * NB);
    const int stripe_bytes = 32 * K * 2;
    const __amdgpu_buffer_rsrc_t c_rsrc = make_rsrc(g.C, g.c_bytes);

    struct Coord {
        int row0, rows, nt;
        bool once;                                              // the expert's only token tile: its weights are read once
    };
    auto locate = [&](int i, Coord *c) {                        // i-th tile of this workgroup; returns its pool slot
        int mt, nt;
        map_tile(wg + i * G, g.m_tiles, g.m_tall, n_tiles_n, g.gm, g.nw, &mt, &nt);
        // The descriptors were written by an earlier launch: read through the constant address space, a
        // scalar load.  (As a vector load its result is waited for with vmcnt(0), which also waits for
        // every prefetched tile load in flight - once per tile.)  The values are uniform, so descriptors
        // and offsets built from them stay in scalar registers.
        static_assert(sizeof(TileDesc) == 16 && offsetof(TileDesc, slot) == 0 && offsetof(TileDesc, row0) == 4 &&
                      offsetof(TileDesc, rows) == 8, "a tile descriptor is read as four ints");
        typedef const __attribute__((address_space(4))) i32x4 *ConstTiles;
        const i32x4 td = ((ConstTiles)(uintptr_t)g.tiles)[mt];  // slot, row0, rows, expert
        *c = Coord{td.y, td.z, nt, ONCE && mt >= g.m_tall};
        return td.x;
    };

    // ---- load side.  Direct load q of a stage fills token rows 8q .. 8q+7 (1 KiB): lane l covers
    // row l/8 of that window and stores at piece position l%8, so it fetches logical piece
    // (l%8) ^ (row/2 & 7).  Wavefront w issues loads w*TL .. w*TL+TL-1 of every stage, i.e. token
    // rows 8*TL*w .. 8*TL*(w+1)-1, and the NS*4 fragments of its own weight stripes.
    const int sub_row = lane >> 3;
    static_assert(TL % 2 == 0, "a wavefront's rows start at a multiple of 16");
    const int first_row = wv * TL * 8 + sub_row;
    const int piece = ((lane & 7) ^ (sub_row >> 1)) * 16;       // of load 0; 64 bytes on or back in every other load
    const __amdgpu_buffer_rsrc_t a_rsrc = make_rsrc(g.A, g.a_bytes);
    const __amdgpu_buffer_rsrc_t map_rsrc = make_rsrc(g.perm, FUSE == kPlain ? 0u : (uint32_t)g.map_len * 4u);
    const __amdgpu_buffer_rsrc_t gate_rsrc = make_rsrc(g.gate_perm, FUSE == kScatter ? (uint32_t)g.map_len * 4u : 0u);
    __amdgpu_buffer_rsrc_t w_rsrc = make_rsrc(g.pool, 0);
    int tok_v[TL], w_at[NS], w_v = lane * 16;                   // byte offsets: per lane, of the stripes, in a fragment
    int tok_s = 0, w_s = 0;                                     // running K offsets (uniform)
    bool w_once = false;                                        // cache policy of the weight loads (uniform)
    // kGather: perm of this wavefront's 8*TL token rows of a tile (rows past its end repeat the last one) -> side
    auto fetch_rows_in = [&](const Coord &c) {
        load_word_to_lds(map_rsrc, (c.row0 + min(wv * TL * 8 + (lane & (TL * 8 - 1)), c.rows - 1)) * 4, side);
    };
    auto point = [&](const Coord &c, int slot) {
#pragma unroll
        for (int j = 0; j < TL; ++j) {
            const int ra = min(first_row + j * 8, c.rows - 1);  // rows past the end re-read the last one
            int src = c.row0 + ra;
            if (FUSE == kGather) {                              // row ra of the tile is one of token src / top_k
                src = reinterpret_cast<const int *>(side)[j * 8 + sub_row];
                if (g.top_k != 1) src /= g.top_k;
            }
            tok_v[j] = src * K * 2 + (piece ^ ((j & 1) * 64));
        }
        w_rsrc = make_rsrc(g.pool + (size_t)slot * g.expert_bytes + g.w_off, (uint32_t)N * (uint32_t)K * 2u);
#pragma unroll
        for (int s = 0; s < NS; ++s) w_at[s] = (c.nt * (BN / 32) + wv * NS + s) * stripe_bytes;
        tok_s = 0;
        w_s = 0;
        w_once = c.once;
    };
    // Behind a workgroup's last tile: loads past the descriptors' ends (past_end.h), which ask for nothing, so that the loop
    // has no data-dependent branch around a load.  (The last tile's first steps fetched once more were two steps of 512
    // workgroups: 42 / 35 MB of the 898 / 909 that missed L2 at 128 experts, 16384 tokens.)
    auto point_nowhere = [&]() {
        constexpr uint32_t kRow = 64 * NB * 2;                  // bytes of a row of either operand, at least: K is a multiple of 64 NB
        static_assert(dropped(kRow, kPastEnd, last_token_scalar(NB)) && dropped(INT32_MAX, kPastEnd, 0) &&
                      dropped(BN * kRow, kPastEnd, last_weight_scalar(NB)), "nothing is loaded");
#pragma unroll
        for (int j = 0; j < TL; ++j) tok_v[j] = kPastEnd;
#pragma unroll
        for (int s = 0; s < NS; ++s) w_at[s] = 0;
        w_v = kPastEnd;
        tok_s = 0;
        w_s = 0;
    };
    int wr_off = 0;                                             // ring offset of the stage filled next
    auto issue_tokens = [&]() {
#pragma unroll
        for (int j = 0; j < TL; ++j) load_to_lds(a_rsrc, tok_v[j], tok_s, lds + wr_off + (wv * TL + j) * 1024);
        tok_s += 128;
        wr_off = wr_off + kStageBytes == kRingBytes ? 0 : wr_off + kStageBytes;
    };
    bf16x8 w[NB][KS][NS];                                       // weight fragments of NB K-steps
    // The weight fragments of one K-step into buffer b.  Weights of an expert with one token tile are
    // read by this tile's workgroups only: streamed past L2's replacement, they leave the token tiles
    // and the many-token experts' weights in place.  (A uniform branch around two equal sets of loads.)
    auto issue_weights = [&](bf16x8 (&wb)[KS][NS]) {
        if (ONCE && w_once) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int s = 0; s < NS; ++s) wb[ks][s] = load_frag<true>(w_rsrc, w_v, w_at[s] + w_s + ks * 1024);
        } else {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int s = 0; s < NS; ++s) wb[ks][s] = load_frag<false>(w_rsrc, w_v, w_at[s] + w_s + ks * 1024);
        }
        w_s += 4096;
    };

    // ---- compute side
    const int frag_row = lane & 31, half = lane >> 5;
    // fragment ks of a 32-row block is at stage + block + (x_at ^ 32 ks): stages and blocks are whole rows
    const int x_at = frag_row * 128 + ((half ^ ((frag_row >> 1) & 7)) * 16);
    f32x16 acc[NS][MI];
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < NS; ++i)
#pragma unroll
            for (int j = 0; j < MI; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    };
    int rd_off = 0;                                             // ring offset of the stage multiplied next

    // Result stores.  A lane holds D[n][m] with m = lane&31 and n = 8*(r/4) + 4*(lane>>5) + r%4, i.e.
    // 8-byte runs of 32 different token rows.  Each wavefront turns its 32-row blocks around through
    // its private staging area and then stores 16 bytes per lane, consecutive lanes covering whole
    // output-row segments (LDS operations of one wavefront execute in order: no barrier between
    // its writes and reads).
    // kScatter: perm and gate_perm of the tile's BM rows -> side[0 .. BM), side[BM .. 2 BM)
    auto fetch_rows_out = [&](const Coord &c) {
#pragma unroll
        for (int i = 0; i < BM / 64; ++i) {
            const int r = (c.row0 + min(i * 64 + lane, c.rows - 1)) * 4;
            load_word_to_lds(map_rsrc, r, side + i * 256);
            load_word_to_lds(gate_rsrc, r, side + BM * 4 + i * 256);
        }
    };
    auto store_tile = [&](const Coord &c) {
        const int seg = lane % LPR, srow = lane / LPR;
#pragma unroll
        for (int im = 0; im < MI; ++im) {
            float gate = 1.f;
            if (FUSE == kScatter) gate = reinterpret_cast<const float *>(side + BM * 4)[im * 32 + frag_row];
#pragma unroll
            for (int in = 0; in < NS; ++in)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    bf16x4 o;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        float v = acc[in][im][q * 4 + j];
                        if (RELU) v = v > 0.f ? v : 0.f;
                        o[j] = (__bf16)v;
                        if (FUSE == kScatter) o[j] = (__bf16)(gate * (float)o[j]);
                    }
                    *reinterpret_cast<bf16x4 *>(stg + frag_row * kOutPitch + (in * 32 + q * 8 + half * 4) * 2) = o;
                }
#pragma unroll
            for (int i = 0; i < 32 / RPI; ++i) {
                const int r = i * RPI + srow;
                const int m = im * 32 + r;
                const bf16x8 v = *reinterpret_cast<const bf16x8 *>(stg + r * kOutPitch + seg * 16);
                // of the row, what differs between lanes (kPlain: all of it but srow is uniform)
                const int lane_row = FUSE == kScatter ? reinterpret_cast<const int *>(side)[m] : srow;
                const int base_row = FUSE == kScatter ? 0 : c.row0 + im * 32 + i * RPI;
                // rows past the tile's end are stored out of range: nothing is written, but every thread issues all its
                // stores and the waits count them
                const int at = lane_row * N * 2 + seg * 16 + (base_row * N + c.nt * BN + wv * kOutCols) * 2;
                store_row_piece<ONCE>(c_rsrc, v, m < c.rows ? at : kPastEnd);
            }
        }
    };

    Coord cc, nc;
    int slot = locate(0, &cc);
    nc = cc;
    if (FUSE == kGather) {                                      // the first tile's row map is needed at once
        fetch_rows_in(cc);
        wait_loads<0>();
    }
    point(cc, slot);
#pragma unroll
    for (int b = 0; b < NB; ++b) {                              // K-steps 0 .. NB-1 of the first tile
        issue_tokens();
        issue_weights(w[b]);
    }
    clear();

    for (int t = 0; t < n; ++t) {
        int next_slot = slot;
        if (t + 1 < n) next_slot = locate(t + 1, &nc);          // used from the last NB steps of this tile on
        // row maps: of the next tile's token rows (read by point() below), or of this tile's result
        // rows (read by store_tile()); the previous reads of the buffer are behind this wavefront
        if (FUSE == kGather) fetch_rows_in(nc);
        if (FUSE == kScatter) fetch_rows_out(cc);
        const int live = (cc.rows + 31) >> 5;                   // 32-row blocks of this tile that hold tokens
#pragma clang loop unroll(disable)
        for (int kk = 0; kk < nkk; ++kk) {
            if (kk == nkk - 1) {                                // all loads of this tile have been issued
                if (FUSE == kGather && nkk == 1) wait_loads<0>();   // else a wait of an earlier step covered the row map
                if (t + 1 < n) point(nc, next_slot);
                else point_nowhere();
            }
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                // result stores of the previous tile may still be outstanding during a tile's first steps
                if (t > 0 && kk == 0) wait_loads<kBase + STORES>();
                else wait_loads<kBase>();
                __builtin_amdgcn_s_barrier();                   // everyone's token rows of this step are in LDS, and
                                                                // everyone is done reading the stage refilled next
                issue_tokens();
                // A fragment of the next 32-row block is read as soon as its predecessor has been multiplied, so
                // that LDS answers behind the products.  Blocks past the tile's end are not multiplied (the
                // first of them is read, to no effect).  Full tiles gain from it (GEMM 1 / 2, read ahead and not:
                // 8 experts x 2048 rows 84.3 / 81.6 and 85.6 / 83.7 us, of 1024 x 4096 139.9 / 147.0 and 143.3 /
                // 157.9), partly filled ones do not (64 experts, 8192 tokens, Zipf(1.2) 90.3 / 88.6 and 90.0 / 89.2).
                const int st = rd_off + x_at;
                bf16x8 xf[KS];
                auto read = [&](int im, int ks) { xf[ks] = *reinterpret_cast<const bf16x8 *>(lds + (st ^ (ks * 32)) + im * 4096); };
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) read(0, ks);
#pragma unroll
                for (int im = 0; im < MI; ++im)
                    if (im == 0 || im < live) {
#pragma unroll
                        for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
                            for (int s = 0; s < NS; ++s)
                                acc[s][im] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[b][ks][s], xf[ks], acc[s][im], 0, 0, 0);
                            if (im + 1 < MI) read(im + 1, ks);
                        }
                    }
                issue_weights(w[b]);
                rd_off = rd_off + kStageBytes == kRingBytes ? 0 : rd_off + kStageBytes;
            }
        }
        if (FUSE == kScatter && nkk == 1) wait_loads<0>();      // as above, for this tile's row maps
        store_tile(cc);
        clear();
        cc = nc;
        slot = next_slot;
    }
    wait_loads<0>();                                            // the last prefetches still write LDS
}

// Compute units the stream's kernels may run on (streams can be created with a compute-unit mask,
// see sida_streams_create), rounded down to a multiple of the 8 XCDs; cached per stream.
std::mutex g_cu_mu;
std::unordered_map<hipStream_t, int> g_cu_cache;

}  // namespace

int stream_compute_units(hipStream_t st)
{
    std::lock_guard<std::mutex> lk(g_cu_mu);
    auto &cache = g_cu_cache;
    auto it = cache.find(st);
    if (it != cache.end()) return it->second;
    int dev = 0, total = 256;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess && prop.multiProcessorCount > 0)
        total = prop.multiProcessorCount;
    int cus = total;
    uint32_t mask[16] = {};
    if (hipExtStreamGetCUMask(st, 16, mask) == hipSuccess) {
        int bits = 0;
        for (int i = 0; i < 16; ++i) bits += __builtin_popcount(mask[i]);
        if (bits > 0 && bits < total) cus = bits;
    } else {
        (void)hipGetLastError();
    }
    cus = cus >= 8 ? cus / 8 * 8 : 8;
    cache[st] = cus;
    return cus;
}

namespace {

// Weights that only one token tile reads are streamed past L2's replacement - when there are more of them
// than stay in the 256 MB Infinity Cache from one pass to the next anyway (measured: a 128-token batch
// over 52 experts, second GEMM 47 -> 43.5 us; 8 experts that are read again and again, 12 -> 14 us).
bool worth_streaming(const GemmArgs &a) { return (int64_t)(a.m_tiles - a.m_tall + a.m_few) * a.N * a.K * 2 > (int64_t)128 << 20; }

// One GEMM of the pair as one launch: BM token rows per tile, 4*NS*32 weight rows, NB K-steps ahead.  The workgroups of
// few-token tiles stand behind the persistent ones, which may take all workgroup slots: a launch's last round of walked
// tiles leaves slots free, and the stream fills them.  (With half of the slots for the persistent workgroups as soon as
// there are few-token tiles, 64 experts, 8192 tokens, those of at most 32 streamed, all layers: 997 -> 1100 us, with three quarters 1027.)
template <int BM, int NS, int NB, bool RELU, int FUSE, bool ONCE>
int launch_as(const GemmArgs &a, hipStream_t st, const LaunchEvents *ev)
{
    constexpr int kLdsBytes = (NB + 1) * BM * 128 + kWaves * 32 * (NS * 64 + 16) +
                              kWaves * (FUSE == kPlain ? 0 : (FUSE == kGather ? 256 : 2 * BM * 4));
    static LdsGrant grant;
    const int rc = allow_lds(grant, reinterpret_cast<const void *>(&grouped_gemm_nt<BM, NS, NB, RELU, FUSE, ONCE>), kLdsBytes);
    if (rc) return rc;
    GemmArgs g = a;
    const int n_tiles_n = a.N / (kWaves * NS * 32);
    g.gm = tile_group_height(a.m_tiles, a.m_tall, a.K > a.N);
    g.nw = tile_block_width(n_tiles_n, g.gm);
    const int total = a.m_tiles * n_tiles_n;
    const int cap = 2 * stream_compute_units(st);            // two workgroups per compute unit
    g.big_wgs = total < cap ? (total + 7) / 8 * 8 : cap;     // multiple of 8 XCDs
    const int few_wgs = (a.m_few * (a.N / (32 * kFewStripes)) + 7) / 8 * 8;
    hipExtLaunchKernelGGL((grouped_gemm_nt<BM, NS, NB, RELU, FUSE, ONCE>), dim3(g.big_wgs + few_wgs), dim3(kWaves * 64), kLdsBytes, st,
                          ev ? ev->start : nullptr, ev ? ev->stop : nullptr, 0, g);
    return (int)hipGetLastError();
}

// Tile shape of a launch.  BM = 64 or 128 token rows as the layer's descriptors say, weight rows by gemm_tiles_wide().
// A launch that leaves
// workgroup slots idle streams every tile's weights through few registers per compute unit, so
// narrow 64-row tiles also fetch four K-steps ahead instead of two where the K loop allows it (with
// 128-row tiles four steps ahead, one workgroup per compute unit, change nothing: 96 tiles of K = 3072
// 34 us either way).
template <int BM, bool RELU, int FUSE>
int launch_width(const GemmArgs &a, hipStream_t st, const LaunchEvents *ev)
{
    const bool wide = gemm_tiles_wide(a.m_tiles, a.m_tall, a.m_few > 0, a.N, a.K, 2 * (int64_t)stream_compute_units(st));
    const bool once = worth_streaming(a);
    if (wide) return once ? launch_as<BM, 2, 2, RELU, FUSE, true>(a, st, ev) : launch_as<BM, 2, 2, RELU, FUSE, false>(a, st, ev);
    if constexpr (BM == kGemmTileSmall)
        if (a.K % 256 == 0) return once ? launch_as<BM, 1, 4, RELU, FUSE, true>(a, st, ev) : launch_as<BM, 1, 4, RELU, FUSE, false>(a, st, ev);
    return once ? launch_as<BM, 1, 2, RELU, FUSE, true>(a, st, ev) : launch_as<BM, 1, 2, RELU, FUSE, false>(a, st, ev);
}

// A launch of few-token tiles only.  One stripe per workgroup keeps most workgroups going; two, which
// fetch the token rows half as often, are faster from 16 rows per tile on if that leaves at least 160
// workgroups (128 experts x 23 tokens: 113 / 113 -> 112 / 106 us; 8 x 32 tokens, second GEMM, 96
// workgroups: 9.4 -> 11.6 us).
template <int NS, bool RELU, int FUSE>
int launch_stream_as(const GemmArgs &a, hipStream_t st, const LaunchEvents *ev)
{
    const int grid = (a.m_few * (a.N / (32 * NS)) + 7) / 8 * 8;
    if (worth_streaming(a))
        hipExtLaunchKernelGGL((stream_gemm_nt<NS, RELU, FUSE, true>), dim3(grid), dim3(kWaves * 64), 0, st, ev ? ev->start : nullptr,
                              ev ? ev->stop : nullptr, 0, a);
    else
        hipExtLaunchKernelGGL((stream_gemm_nt<NS, RELU, FUSE, false>), dim3(grid), dim3(kWaves * 64), 0, st, ev ? ev->start : nullptr,
                              ev ? ev->stop : nullptr, 0, a);
    return (int)hipGetLastError();
}

template <bool RELU, int FUSE>
int launch_shape(const GemmArgs &a, int tile_m, hipStream_t st, const LaunchEvents *ev)
{
    if (a.m_tiles + a.m_few <= 0) {                          // nothing to launch: keep the events usable
        if (ev) {
            (void)hipEventRecord(ev->start, st);
            (void)hipEventRecord(ev->stop, st);
        }
        return 0;
    }
    if (a.m_tiles == 0) {
        if (a.few_rows > 16 * a.m_few && a.m_few * (a.N / 64) >= 160) return launch_stream_as<2, RELU, FUSE>(a, st, ev);
        return launch_stream_as<1, RELU, FUSE>(a, st, ev);
    }
    if (tile_m == kGemmTileSmall) return launch_width<kGemmTileSmall, RELU, FUSE>(a, st, ev);
    return launch_width<kGemmTileM, RELU, FUSE>(a, st, ev);
}

}  // namespace

int allow_lds(LdsGrant &grant, const void *kernel, int bytes)
{
    int device = -1;
    const hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return (int)e;
    return grant.on(device, [&] { return (int)hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes); });
}

void forget_stream(hipStream_t st)
{
    std::lock_guard<std::mutex> lk(g_cu_mu);
    g_cu_cache.erase(st);
}

int launch_ffn_gemm1(const void *x_perm, void *h, const char *pool, size_t expert_bytes, const TileDesc *tiles,
                     int32_t m_tiles, int32_t m_tall, int32_t m_few, int32_t few_rows, int32_t d, int32_t F, hipStream_t st,
                     const LaunchEvents *ev, int32_t a_rows, const int32_t *perm, int32_t map_len, int32_t top_k,
                     int32_t tile_m)
{
    GemmArgs a{};
    a.A = (const __bf16 *)x_perm;
    a.C = (__bf16 *)h;
    a.pool = pool;
    a.expert_bytes = expert_bytes;
    a.w_off = 0;
    a.tiles = tiles;
    a.m_tiles = m_tiles;
    a.m_tall = m_tall;
    a.m_few = m_few;
    a.few_rows = few_rows;
    a.N = F;
    a.K = d;
    a.a_bytes = (uint32_t)((size_t)a_rows * d * 2);
    a.c_bytes = (uint32_t)((size_t)map_len * F * 2);
    a.perm = perm;
    a.map_len = map_len;
    a.top_k = top_k;
    return perm ? launch_shape<true, kGather>(a, tile_m, st, ev) : launch_shape<true, kPlain>(a, tile_m, st, ev);
}

int launch_ffn_gemm2(const void *h, void *y_perm, const char *pool, size_t expert_bytes, const TileDesc *tiles,
                     int32_t m_tiles, int32_t m_tall, int32_t m_few, int32_t few_rows, int32_t d, int32_t F, hipStream_t st,
                     const LaunchEvents *ev, int32_t a_rows, const int32_t *perm, const float *gate_perm, int32_t tile_m)
{
    GemmArgs a{};
    a.A = (const __bf16 *)h;
    a.C = (__bf16 *)y_perm;
    a.pool = pool;
    a.expert_bytes = expert_bytes;
    a.w_off = (size_t)F * (size_t)d * 2;                     // W_out follows W_in in a slot
    a.tiles = tiles;
    a.m_tiles = m_tiles;
    a.m_tall = m_tall;
    a.m_few = m_few;
    a.few_rows = few_rows;
    a.N = d;
    a.K = F;
    a.a_bytes = (uint32_t)((size_t)a_rows * F * 2);
    a.c_bytes = (uint32_t)((size_t)a_rows * d * 2);
    a.perm = perm;
    a.gate_perm = gate_perm;
    a.map_len = a_rows;
    a.top_k = 1;                                             // scattering is only defined for one expert per token
    return perm ? launch_shape<false, kScatter>(a, tile_m, st, ev) : launch_shape<false, kPlain>(a, tile_m, st, ev);
}

// ---- token-tile descriptors ----------------------------------------------------------------
namespace {

// One workgroup; thread i owns table entry i.
__global__ __launch_bounds__(256) void build_tiles(const LayerTable tbl, const int32_t *__restrict__ offsets,
                                                   TileDesc *__restrict__ tiles, int max_tiles)
{
    __shared__ int s_wsum[4];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    int e = 0, slot = 0, off = 0, cnt = 0, n_t = 0;
    if (tid < tbl.n) {
        e = tbl.expert[tid];
        slot = tbl.slot[tid];
        off = offsets[e];
        cnt = offsets[e + 1] - off;
        n_t = (cnt + tbl.tile_m - 1) / tbl.tile_m;
    }
    int incl = n_t;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
    }
    if (lane == 63) s_wsum[wv] = incl;
    __syncthreads();
    for (int i = 0; i < wv; ++i) incl += s_wsum[i];
    int at = incl - n_t;
    for (int k = 0; k < n_t && at < max_tiles; ++k, ++at) {
        TileDesc t;
        t.slot = slot;
        t.row0 = off + k * tbl.tile_m;
        t.rows = min(tbl.tile_m, cnt - k * tbl.tile_m);
        t.expert = e;
        tiles[at] = t;
    }
}

}  // namespace

int launch_build_tiles(const LayerTable &tbl, const int32_t *offsets, TileDesc *tiles, int32_t max_tiles,
                       hipStream_t st)
{
    hipLaunchKernelGGL(build_tiles, dim3(1), dim3(256), 0, st, tbl, offsets, tiles, max_tiles);
    return (int)hipGetLastError();
}

}  // namespace sida
