// The hash function of the hash-building thread (Section 3.4.2): predicts, for every token of a
// sequence and every MoE layer, the experts to activate and their scaling factors, from the token
// embeddings alone - a fully connected layer that compresses the embedding, a 2-layer LSTM, an
// attention layer over the LSTM's output sequence whose weights go through SparseMax, a residual
// connection, and one linear head per MoE layer (Algorithm 1, right column: k <- h_l(X)[s]).
// Readings where the paper gives no detail: compressed width = LSTM hidden width C; standard LSTM
// cell (gates input, forget, cell, output), zero initial state; dot-product scores without scaling;
// the residual adds the token's own compressed embedding; alpha = SoftMax probability of the
// expert within its layer's head; the k largest are kept, ties to the lower expert id.
//
// All values and sums are fp32 (rounded to bf16 they would move the predicted probabilities by more than the parity
// bound).  Four or five launches per call:
//   hash_dense      c0 = x W_in^T + b, and again for layer 1's gate pre-activations (or in the next launch)
//   hash_recurrence both LSTM layers at once, layer 2 a few steps behind layer 1
//   hash_attention  scores, SparseMax, weighted sum and residual, for blocks of 16 queries
//   hash_heads      logits, SoftMax and the k best, for blocks of tokens and a MoE layer each (or hash_heads_walk)
// The contractions run on the fp32 matrix instruction (v_mfma_f32_16x16x4_f32, twice the rate of
// scalar-per-lane fp32 multiply-adds), or on the bf16 one with the values in exact parts (hash_dense, Parts); with the
// weights as the first operand a lane ends up with four consecutive output units of one token.  The recurrence is a chain of matrix-vector products,
// where 15 of the instruction's 16 columns would idle, and stays on the vector units.
// It is what bounds a call: 0.53 us a time step at C = 128, see lstm_layer.  Measured against one launch per layer and
// stage on the vector units (d = 768, C = 128, 6 x 128 experts; calls of perf/cases.py, inputs changing): 1 sequence of
// 128 tokens 375 -> 107 us, 8 of 333 tokens (top-3) 1059 -> 243 us, 64 of 128 tokens 609 -> 136 us.
#include <hip/hip_runtime.h>

#include <cfloat>
#include <mutex>
#include <type_traits>
#include <utility>

#include "handover.h"
#include "heads_walk.h"
#include "kernels.h"

namespace sida {

namespace {

// Scratch of sida_hash_forward_static: the intermediates of one call (8*C floats per token) live
// here instead of in a caller's workspace.  Every GPU the library runs on holds its own copy of
// the array, at its own address, until the process ends.  In host code the array's name is only a
// stand-in for the symbol: the device address comes from hipGetSymbolAddress, once per device.
static __device__ __align__(256) unsigned char scratch[kHashStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float *g_scratch_ptr[kMaxDevices] = {};

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
typedef __attribute__((ext_vector_type(4))) int i32x4;

// ---- fp32 matrix products -----------------------------------------------------------------------
// D[16 x 16] += A[16 x 4] B[4 x 16]: lane l gives A[l % 16][l / 16] and B[l / 16][l % 16] and holds
// D[4 * (l / 16) + i][l % 16].  The order of the K values is free, so four instructions take 16
// consecutive K values with lane group g = l / 16 at 4g .. 4g+3: one 16-byte load per operand.
__device__ __forceinline__ f32x4 mfma4(const f32x4 &a, const f32x4 &b, f32x4 d)
{
#pragma unroll
    for (int j = 0; j < 4; ++j) d = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], b[j], d, 0, 0, 0);
    return d;
}
// The loads above stay above: a wavefront has them all in flight (the compiler would rather save registers).
__device__ __forceinline__ void loads_issued() { __builtin_amdgcn_sched_barrier(0); }
__device__ __forceinline__ f32x4 load4(const float *p) { return *reinterpret_cast<const f32x4 *>(p); }
// Parameters, which the caller may hand over at the address of any float.
__device__ __forceinline__ f32x4 load4_param(const float *p)
{
    typedef f32x4 __attribute__((aligned(4))) f32x4_any;
    return *reinterpret_cast<const f32x4_any *>(p);
}

// ---- exchange between lanes ---------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ int dpp(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ float quad(float v)                 // value of another lane of the quad (or row, below)
{
    return __builtin_bit_cast(float, dpp<CTRL>(__builtin_bit_cast(int, v)));
}
// Reductions over the 16 lanes of a row: lane ^ 1, lane ^ 2, then mirrored halves (their quads agree) and
// mirrored rows; f(v, value of the other lane).
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kHalfMirror = 0x141, kMirror = 0x140;
__device__ __forceinline__ float row_sum(float v)
{
    v += quad<kXor1>(v);
    v += quad<kXor2>(v);
    v += quad<kHalfMirror>(v);
    return v + quad<kMirror>(v);
}
__device__ __forceinline__ float row_max(float v)
{
    v = fmaxf(v, quad<kXor1>(v));
    v = fmaxf(v, quad<kXor2>(v));
    v = fmaxf(v, quad<kHalfMirror>(v));
    return fmaxf(v, quad<kMirror>(v));
}

// ---- exchange between workgroups of one launch --------------------------------------------------
// Values that another workgroup reads while both run are stored and loaded at agent scope (past the
// L2, which is not coherent between XCDs), through buffer descriptors with the sc1 bit.
constexpr int kAgent = 16;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000);
}
template <int POLICY>
__device__ __forceinline__ float load_f32(__amdgpu_buffer_rsrc_t r, int byte)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, byte, 0, POLICY));
}
template <int POLICY>
__device__ __forceinline__ void store_f32(__amdgpu_buffer_rsrc_t r, int byte, float v)
{
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), r, byte, 0, POLICY);
}
__device__ __forceinline__ int peek(const int *flag)
{
    return __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void publish(int *flag, int v)
{
    __hip_atomic_store(flag, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <int N>
__device__ __forceinline__ void wait_memory()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// Workgroup barrier that orders LDS accesses only: global loads stay in flight across it.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// ---- operand tiles in LDS -----------------------------------------------------------------------
// Rows of 32 values, loaded straight into LDS with whole lines per request.  (Fetched as matrix operands,
// 16 bytes of a different row in every lane, each lane is a cache access of its own: the dense stages
// were bound by those, 64 per load, at 45 % of the matrix rate.)  Within a step of 32 values lane
// group g multiplies values 8g .. 8g+7, its two 16-byte pieces of an fp32 row, or the one of a bf16 row.
// A row's pieces are stored exclusive-or'ed with the row number, so that neither the lane-linear writes
// nor the reads of one piece of 16 rows meet in a bank.
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t r, int voffset, char *dst)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)dst, 16, voffset, 0, 0, 0);
}
template <typename T>
struct TileRow {                                               // T = float
    static constexpr int kBytes = 128, kRowsPerLoad = 8;
    static __device__ __forceinline__ int row(int lane) { return lane >> 3; }
    static __device__ __forceinline__ int piece(int lane, int row) { return (lane & 7) ^ (row & 7); }
    static __device__ __forceinline__ void read(const char *tile, int row, int g, float (&v)[8])
    {
        const char *p = tile + row * kBytes;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const f32x4 q = *reinterpret_cast<const f32x4 *>(p + (((2 * g + h) ^ (row & 7)) * 16));
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * h + e] = q[e];
        }
    }
};
template <>
struct TileRow<__bf16> {
    static constexpr int kBytes = 64, kRowsPerLoad = 16;
    static __device__ __forceinline__ int row(int lane) { return lane >> 2; }
    static __device__ __forceinline__ int piece(int lane, int row) { return (lane & 3) ^ ((row >> 1) & 3); }
    static __device__ __forceinline__ void read(const char *tile, int row, int g, bf16x8 &v)
    {
        v = *reinterpret_cast<const bf16x8 *>(tile + row * kBytes + ((g ^ ((row >> 1) & 3)) * 16));
    }
};
// v = hi + mid + lo, exactly from 2^-109 on (bf16 has 8 of the 24 bits and ends at 2^-133).  hi and mid are rounded to
// nearest, so mid is at most 2^-8 and lo at most 2^-17 of v's power of two, of either sign.  (Cut, at the same number of
// instructions, they were up to 2^-7 and 2^-15 and of v's sign.)  An infinite v, or one that rounds to infinity, has a part
// that is NaN, see any_overflow.
__device__ __forceinline__ void split3(const float (&v)[8], bf16x8 &hi, bf16x8 &mid, bf16x8 &lo)
{
    i32x4 h, m, l;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        f32x2 rest{v[2 * e], v[2 * e + 1]};
        auto take = [&] {                                      // the pair rounded, and what is left of it
            const unsigned int pair = __builtin_bit_cast(unsigned int, __builtin_convertvector(rest, bf16x2));
            rest[0] -= __builtin_bit_cast(float, pair << 16);
            rest[1] -= __builtin_bit_cast(float, pair & 0xffff0000u);
            return (int)pair;
        };
        h[e] = take();
        m[e] = take();
        l[e] = take();
    }
    hi = __builtin_bit_cast(bf16x8, h);
    mid = __builtin_bit_cast(bf16x8, m);
    lo = __builtin_bit_cast(bf16x8, l);
}
// The product of 16 x 32 and 32 x 16 fp32 values on the bf16 matrix instruction: of the nine products of their parts all
// but mid lo, lo mid and lo lo, which are together at most 2^-24 of the whole and of either sign; small ones first.  96
// clocks instead of 256, and 44 vector instructions to split the values of an operand: worth it where an operand meets two
// others (2 x 2 tiles of a wavefront; the layers' gate pre-activations and the heads of 2048 tokens and more: 64 x 128
// tokens 151.1 -> 146.3 us a call, 8 x 333 247.7 -> 246.7, 96 x 85 190.9 -> 184.2).  The longer sums of the instruction are
// rounded less often: alpha against 64 bits is nearer by another 10 to 22 % in 14 batches of such sizes (2-norms, relative).
struct Parts {
    bf16x8 hi, mid, lo;
};
__device__ __forceinline__ Parts parts_of(const float (&v)[8])
{
    Parts p;
    split3(v, p.hi, p.mid, p.lo);
    return p;
}
__device__ __forceinline__ f32x4 mfma_parts(const Parts &a, const Parts &b, f32x4 d)
{
    d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.lo, b.hi, d, 0, 0, 0);
    d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.hi, b.lo, d, 0, 0, 0);
    d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.mid, b.mid, d, 0, 0, 0);
    d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.mid, b.hi, d, 0, 0, 0);
    d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.hi, b.mid, d, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.hi, b.hi, d, 0, 0, 0);
}
// Infinities do not go through parts (they leave NaN behind, and parts that are 0 make NaN of an infinite factor): a sum
// that comes out infinite or NaN is made again on the fp32 instruction, and that one counts.  One that comes out
// finite had finite parts only.
template <int TU, int TT>
__device__ __forceinline__ bool any_overflow(const f32x4 (&d)[TU][TT])    // in any lane
{
    float none = 0.f;                                          // NaN once a value was infinite or NaN
#pragma unroll
    for (int i = 0; i < TU; ++i)
#pragma unroll
        for (int m = 0; m < TT; ++m)
#pragma unroll
            for (int e = 0; e < 4; ++e) none = fmaf(d[i][m][e], 0.f, none);
    return __any(none != none);
}
__device__ __forceinline__ f32x4 where_overflowed(f32x4 d, const f32x4 &other)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) d[e] = __builtin_isfinite(d[e]) ? d[e] : other[e];
    return d;
}
// A piece whose address is a multiple of its values' size only.
__device__ __forceinline__ void copy_piece(const float *p, char *dst)
{
    *reinterpret_cast<f32x4 *>(dst) = f32x4{p[0], p[1], p[2], p[3]};
}
__device__ __forceinline__ void copy_piece(const __bf16 *p, char *dst)
{
    *reinterpret_cast<bf16x8 *>(dst) = bf16x8{p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7]};
}
// The loads of one wavefront for tiles of ROWS rows of a [rows, k] matrix, shared by SHARE wavefronts.
// Every wavefront issues kLoads per tile (a tile of fewer loads is loaded twice over, with the same
// bytes); rows and columns past the end repeat the last ones.  DIRECT: the matrix starts at a 16-byte
// boundary, as a load into LDS wants it; otherwise the values go through registers.
template <typename T, int ROWS, int SHARE, bool DIRECT>
struct TileLoader {
    static constexpr int kAll = ROWS / TileRow<T>::kRowsPerLoad, kLoads = (kAll + SHARE - 1) / SHARE;
    static_assert(ROWS % TileRow<T>::kRowsPerLoad == 0 && (kAll % SHARE == 0 || kAll < SHARE), "whole loads");
    __amdgpu_buffer_rsrc_t rsrc;
    const T *base;
    int row_at[kLoads], piece[kLoads], dst[kLoads], last;
    __device__ __forceinline__ TileLoader(const T *first_row, int rows_left, int k, int lane, int share)
    {
        const int rows = min(rows_left, ROWS);
        rsrc = make_rsrc(first_row, (uint32_t)rows * (uint32_t)k * (uint32_t)sizeof(T));
        base = first_row;
        last = k * (int)sizeof(T) - 16;
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const int q = (share * kLoads + i) % kAll, row = q * TileRow<T>::kRowsPerLoad + TileRow<T>::row(lane);
            row_at[i] = min(row, rows - 1) * k * (int)sizeof(T);
            piece[i] = TileRow<T>::piece(lane, row) * 16;
            dst[i] = __builtin_amdgcn_readfirstlane(q) * 1024;
        }
    }
    __device__ __forceinline__ void issue(int step, char *tile) const
    {
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const int at = row_at[i] + min(step * TileRow<T>::kBytes + piece[i], last);
            if constexpr (DIRECT) load_to_lds(rsrc, at, tile + dst[i]);
            else copy_piece(base + at / (int)sizeof(T), tile + dst[i] + (threadIdx.x & 63) * 16);
        }
    }
};
// All but the last N of this wavefront's tile loads have arrived.
template <int N, bool DIRECT>
__device__ __forceinline__ void tiles_arrived()
{
    if (DIRECT) wait_memory<N>();
    else asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

// ---- dense stages -------------------------------------------------------------------------------
// out[n, u] = bias_a[u] + bias_b[u] + sum_i in[n, i] w[u, i] for n_tokens tokens and `units` units (w is
// [units, k], k a multiple of 8; bias_b may be null): the compressed embedding and layer 1's gate
// pre-activations.  A wavefront makes TU x TT tiles of 16 units x 16 tokens; a workgroup is 4 =
// WU (units) x WT (tokens) x KS (parts of the sum) wavefronts.  Operands run NB - 1 stages of G * 32
// values ahead in a ring of NB stages, shared by the workgroup's wavefronts or (KS > 1) each wavefront
// its own.
//  * Small batches are bound by the latency of their loads and by what one compute unit can fetch
//    (128 tokens: 33 us when 8 workgroups of 16 tokens read all weights each): one tile per wavefront
//    and the long sum over d_model in four parts, so that the operands of a wavefront are in flight at
//    once and the weights are spread over 64 workgroups.
//  * Large ones by the matrix units: 4 or 2 x 2 tiles per wavefront.
// Embeddings are bf16, so their product with fp32 weights goes through the bf16 matrix instruction, of 16 times the rate:
// a weight is the sum of three bf16 values, exactly, every product is exact, and the sums are fp32 as before.  (The
// instruction does not normalise embeddings below 2^-126: their products keep fewer bits, 20 at 2^-130.)  8192 tokens
// of 768: 64 x 128 tokens 162.0 -> 152.1 us a call (1 x 4 tiles, so that a weight is split once per workgroup), 8 x 333
// 254.4 -> 249.5, 32 x 200 at C = 64 135.3 -> 125.4.  alpha against 64 bits over eight batches of 2060 to 8192 tokens, d of
// 256 to 2056 (2-norm, relative): 0.44e-6 - 1.07e-6 before, 0.31e-6 - 0.84e-6 this way, smaller in each.
// Also clears the counters of the recurrence behind it.
template <int TU, int TT, int WU, int WT, int KS, int G, int NB, typename IN, bool DIRECT>
__global__ __launch_bounds__(256) void hash_dense(const IN *__restrict__ in, const float *__restrict__ w,
                                                  const float *__restrict__ bias_a, const float *__restrict__ bias_b, int k,
                                                  int units, int n_tokens, float *__restrict__ out,
                                                  int *__restrict__ counters, int n_counters)
{
    static_assert(WU * WT * KS == 4 && (KS == 1 || (KS == 4 && TU * TT == 1)), "wavefronts of a workgroup");
    constexpr int kShare = KS == 1 ? 4 : 1;
    constexpr bool kSplit = std::is_same<IN, __bf16>::value;   // the weights, into three bf16 parts
    constexpr bool kParts = kSplit || TU * TT > 1;             // ... or both operands
    constexpr int WR = WU * TU * 16, XR = WT * TT * 16;        // rows staged together
    constexpr int kW = WR * TileRow<float>::kBytes, kStep = kW + XR * TileRow<IN>::kBytes, kStage = G * kStep;
    typedef TileLoader<float, WR, kShare, DIRECT> LoadW;
    typedef TileLoader<IN, XR, kShare, DIRECT> LoadX;
    constexpr int kStageLoads = G * (LoadW::kLoads + LoadX::kLoads);
    __shared__ __attribute__((aligned(1024))) char ring[(4 / kShare) * NB * kStage];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), col = lane & 15, g = lane >> 4;
    if (blockIdx.y == 0)
        for (int i = blockIdx.x * 256 + tid; i < n_counters; i += gridDim.x * 256) counters[i] = 0;
    const int part = KS == 1 ? 0 : wv, wu = KS == 1 ? wv % WU : 0, wt = KS == 1 ? wv / WU : 0;
    const int n0 = blockIdx.x * XR, u0 = blockIdx.y * WR;
    const int steps = (k + 31) / 32, per = (steps + KS - 1) / KS, first = part * per, last = min(steps, first + per);
    const LoadW load_w(w + (size_t)u0 * k, units - u0, k, lane, wv % kShare);
    const LoadX load_x(in + (size_t)n0 * k, n_tokens - n0, k, lane, wv % kShare);
    char *mine = ring + (KS == 1 ? 0 : wv * NB * kStage);
    f32x4 acc[TU][TT] = {};
    const int end = min(k, last * 32);                         // of this wavefront's part of the sum
    auto issue = [&](int s, int slot) {                        // past the end: the last values again, unused
#pragma unroll
        for (int h = 0; h < G; ++h) {
            load_w.issue(s + h, mine + slot * kStage + h * kStep);
            load_x.issue(s + h, mine + slot * kStage + h * kStep + kW);
        }
    };
    if (first < last) {
#pragma unroll
        for (int b = 0; b < NB - 1; ++b) issue(first + b * G, b);
        int slot = 0;
        for (int s = first; s < last; s += G) {
            tiles_arrived<(NB - 2) * kStageLoads, DIRECT>();
            if (KS == 1) __builtin_amdgcn_s_barrier();         // everyone's part of this stage is here, and the slot
                                                               // filled next has been read by everyone
            issue(s + (NB - 1) * G, slot == 0 ? NB - 1 : slot - 1);
            const char *tile = mine + slot * kStage;
            slot = slot + 1 == NB ? 0 : slot + 1;
            float a[G][TU][8];
            typename std::conditional<kSplit, bf16x8, float[8]>::type b[G][TT];
#pragma unroll
            for (int h = 0; h < G; ++h) {
#pragma unroll
                for (int i = 0; i < TU; ++i) TileRow<float>::read(tile + h * kStep, (wu * TU + i) * 16 + col, g, a[h][i]);
#pragma unroll
                for (int m = 0; m < TT; ++m) TileRow<IN>::read(tile + h * kStep + kW, (wt * TT + m) * 16 + col, g, b[h][m]);
            }
            if ((s + G) * 32 > end)                            // past the end of the sum
#pragma unroll
                for (int h = 0; h < G; ++h)
#pragma unroll
                    for (int i = 0; i < TU; ++i)
#pragma unroll
                        for (int e = 0; e < 8; ++e) a[h][i][e] = (s + h) * 32 + 8 * g < end ? a[h][i][e] : 0.f;
#pragma unroll
            for (int h = 0; h < G; ++h) {
                if constexpr (kSplit) {
#pragma unroll
                    for (int i = 0; i < TU; ++i) {
                        bf16x8 part[3];
                        split3(a[h][i], part[2], part[1], part[0]);
#pragma unroll
                        for (int q = 0; q < 3; ++q)
#pragma unroll
                            for (int m = 0; m < TT; ++m)
                                acc[i][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(part[q], b[h][m], acc[i][m], 0, 0, 0);
                    }
                } else if constexpr (kParts) {
                    Parts pa[TU], pb[TT];
#pragma unroll
                    for (int i = 0; i < TU; ++i) pa[i] = parts_of(a[h][i]);
#pragma unroll
                    for (int m = 0; m < TT; ++m) pb[m] = parts_of(b[h][m]);
#pragma unroll
                    for (int i = 0; i < TU; ++i)
#pragma unroll
                        for (int m = 0; m < TT; ++m) acc[i][m] = mfma_parts(pa[i], pb[m], acc[i][m]);
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e)
#pragma unroll
                        for (int m = 0; m < TT; ++m)
#pragma unroll
                            for (int i = 0; i < TU; ++i)
                                acc[i][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[h][i][e], b[h][m][e], acc[i][m], 0, 0, 0);
                }
            }
        }
        tiles_arrived<0, DIRECT>();                            // the last loads still write LDS
        if (kParts && any_overflow(acc)) {
#pragma unroll 1
            for (int t = 0; t < TU * TT; ++t) {
                const int i = t / TT, m = t % TT;
                f32x4 d[1][1] = {acc[0][0]};                   // a token that is NaN is in one tile of four
#pragma unroll
                for (int j = 1; j < TU * TT; ++j)
                    if (j == t) d[0][0] = acc[j / TT][j % TT];
                if (!any_overflow(d)) continue;
                const float *row = w + (size_t)(u0 + (wu * TU + i) * 16 + col) * k;
                const IN *token = in + (size_t)min(n0 + (wt * TT + m) * 16 + col, n_tokens - 1) * k;
                f32x4 again = {};
#pragma unroll 1
                for (int s = first * 32; s < end; s += 32) {   // four such steps at a time were not faster
                    float a[8] = {}, b[8] = {};
                    const int at = s + 8 * g;
                    if (at < end) {
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            a[e] = row[at + e];
                            b[e] = (float)token[at + e];
                        }
                    }
#pragma unroll
                    for (int e = 0; e < 8; ++e) again = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], again, 0, 0, 0);
                }
#pragma unroll
                for (int j = 0; j < TU * TT; ++j)
                    if (j == t) acc[j / TT][j % TT] = where_overflowed(acc[j / TT][j % TT], again);
            }
        }
    }
    if (KS > 1) {                                              // the parts of the sum meet in the first wavefront
        __shared__ f32x4 parts[KS][64];
        parts[part][lane] = acc[0][0];
        __syncthreads();
        if (part) return;
#pragma unroll
        for (int q = 1; q < KS; ++q) acc[0][0] += parts[q][lane];
    }
#pragma unroll
    for (int i = 0; i < TU; ++i) {
        const int u = u0 + (wu * TU + i) * 16 + 4 * g;
        f32x4 bias = load4_param(bias_a + u);
        if (bias_b) bias += load4_param(bias_b + u);
#pragma unroll
        for (int m = 0; m < TT; ++m) {
            const int n = n0 + (wt * TT + m) * 16 + col;
            if (n < n_tokens) *reinterpret_cast<f32x4 *>(out + (size_t)n * units + u) = acc[i][m] + bias;
        }
    }
}

// ---- the recurrence -----------------------------------------------------------------------------
// Sigmoid and tanh by one straight line for both, told apart by three constants per lane, since the step of the
// recurrence is bound by the instructions it issues: exponential by v_exp_f32, reciprocal with one Newton step, and a
// Taylor polynomial of tanh below 1/4, where 2 / (1 + e) - 1 cancels (its next term, 1382/155925 x^11, is below 2^-26 of
// tanh there).  Errors are about 2 units in the last place of 1; of a tanh just above 1/4 that is up to 7 of its own.
// The sums in parts make up for it: alpha against 64 bits, over nine batches of 29 to 8192 tokens, 0.56e-6 - 1.13e-6 with
// tanhf and sums in index order, 0.34e-6 - 1.05e-6 this way, smaller in each (2-norms, relative).
// lane:  sigmoid(v) = 1 / (1 + exp(-v)),  tanh(v) = 2 / (1 + exp(-2v)) - 1.
struct GateKind {
    float scale, gain, small;      // of the exponent (base 2), of the reciprocal, bound of the polynomial
};
__device__ __forceinline__ GateKind gate_kind(bool is_tanh)
{
    constexpr float kLog2e = 1.44269504f;
    return is_tanh ? GateKind{-2.f * kLog2e, 2.f, 0.25f} : GateKind{-kLog2e, 1.f, 0.f};
}
__device__ __forceinline__ float gate_value(float v, const GateKind &k)
{
    // an exponent of at most 126 keeps the Newton step away from infinity; NaN goes through
    const float e = 1.f + __builtin_amdgcn_exp2f(__builtin_elementwise_minimum(v * k.scale, 126.f));
    const float r = __builtin_amdgcn_rcpf(e);
    const float n = fmaf(fmaf(-e, r, 1.f), r, r);
    const float q = v * v;
    const float t = v * fmaf(q, fmaf(q, fmaf(q, fmaf(q, 62.f / 2835.f, -17.f / 315.f), 2.f / 15.f), -1.f / 3.f), 1.f);
    return fabsf(v) < k.small ? t : fmaf(k.gain, n, 1.f - k.gain);
}

// v of the quad's lane 1 * x + v * v of the quad's lane 2: forget gate * state + input gate * cell gate, in lane 0.  Two
// instructions (the compiler makes the second a move and a multiply-add).
__device__ __forceinline__ float next_cell(float v, float x)
{
    // A value from another lane may be read two instructions after it was written.  The compiler sees to that in its
    // own code, not in front of this; the wait stays here, also where what it put in front has waited already.
    float cell;
    asm("s_nop 1\n\t"
        "v_mul_f32_dpp %0, %1, %1 quad_perm:[2,2,2,2] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_fmac_f32_dpp %0, %1, %2 quad_perm:[1,1,1,1] row_mask:0xf bank_mask:0xf bound_ctrl:1"
        : "=&v"(cell) : "v"(v), "v"(x));
    return cell;
}

template <int C>
constexpr int kChunk = C == 128 ? kSteps : kStepsNarrow;       // time steps handed over together

template <int C>
struct RecurrenceLds {
    static constexpr int kSeg = C / 8, kSegPitch = kSeg + 4;   // the eight segments start in different banks
    static constexpr int kRow = 8 * kSegPitch;
    // Where a unit's state stands in a row.  Four units that are loaded together stand one on, in a circle, so that a
    // unit's state comes into a register of odd number where its weights' is even, and the other way round.
    static __device__ __forceinline__ int place(int unit) { return (unit / kSeg) * kSegPitch + (unit % kSeg & ~3) + ((unit + 1) & 3); }
    float h[2 * kChunk<C>][kRow];                               // the state after each step of two chunks
    float pre[kChunk<C>][4 * C];                                // gate pre-activations of a chunk; a thread reads what it wrote
    static constexpr int kInPitch = C + 16;
    float in[2][kGateTokens * kInPitch];                        // tokens of which gate pre-activations are made
    int ticket;
};

// One LSTM layer over one sequence of T steps, by a workgroup of 4C threads.  Eight threads share the
// eight gate rows of two units: each holds an eighth of the columns of all eight in registers, so that a
// step reads only an eighth of the state per thread from LDS (with a whole gate row per thread the
// 8 x 32 broadcast reads of 16 bytes took longer than the multiply-adds: 1.05 us a step at C = 128; with
// quarters 0.65 us).  Slot j of lane l of the eight is row j ^ l, so that seven adds of permuted lanes
// leave row l's sum in lane l; thread 4u+s then has gate s of unit u, the four gates meet in quad permutes
// too, and a step has one barrier and no global access: pre-activations come and states go a chunk of
// steps at a time.
// What a step at C = 128 is bound by, 1270 cycles: a wavefront issues one instruction of any kind in 4.1 cycles, 190 of them,
// and waits for the barrier and its first state from LDS (240); two wavefronts per SIMD multiply side by side (128 each in
// 526 cycles), but sums of permuted lanes and exponentials keep the SIMD to themselves, and the second wavefront ends 160
// later.  Registers stand in two banks, of even and of odd numbers, and a pair of multiply-adds of two wavefronts gets
// four operands from each: one whose three are all even (or odd) makes the other wavefront wait for four cycles.
// 66 of a step's were, when a unit's weights and state came out of 16-byte loads in the same order; with place() 2
// are, and a step takes 1284 cycles instead of 1308 (bits unchanged); both products of the cell in one piece 1270.
// Whole chunks are written out (addresses become offsets; the kernel's code grows to 17 - 21 KB), lane 0
// of a quad alone carries the cell's state, and sums of permuted lanes are one instruction each, with the
// same bits.  One taken back at a time, us a call, and all three in front (1 x 128, 8 x 333, 96 x 85 tokens; of an earlier build):
// 112.8, 260.2, 201.8; chunks walked in a loop 115.9, 267.7, 205.5; the state in every lane 113.2, 260.9, 202.8;
// the sum with a permuted value more 113.0, 260.7, 201.8.
// Tried on it without gain: the own wavefront's columns ahead of the barrier, rows finished one after the other so that sums meet behind
// products, 32 columns a lane in four accumulators, and the two wavefronts of a SIMD half a step apart with two barriers a
// step (1254 to 1480 cycles).
//   WAIT   pre arrives in chunks from another workgroup (progress in *arrived)
//   POST   out is handed on to another workgroup (progress in *done: wavefronts x chunks)
template <int C, bool WAIT, bool POST>
__device__ __forceinline__ void lstm_layer(const float *__restrict__ pre, const float *__restrict__ w_hh, int T,
                                           float *__restrict__ out, const int *arrived, int *done, RecurrenceLds<C> &lds)
{
    constexpr int kSeg = RecurrenceLds<C>::kSeg, kSegPitch = RecurrenceLds<C>::kSegPitch, kRow = RecurrenceLds<C>::kRow;
    constexpr int kSteps = kChunk<C>;
    const int tid = threadIdx.x, u = tid >> 2, s = tid & 3;
    const int l8 = tid & 7;
    float w[8][kSeg];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int id = j ^ l8;                                 // gate id & 3 of unit 2 * (tid / 8) + (id >> 2)
        const float *row = w_hh + (size_t)((id & 3) * C + (tid >> 3) * 2 + (id >> 2)) * C + l8 * kSeg;
#pragma unroll
        for (int i = 0; i < kSeg; i += 4) {
            const f32x4 v = load4_param(row + i);
            w[j][i] = v[0];
            w[j][i + 1] = v[1];
            w[j][i + 2] = v[2];
            w[j][i + 3] = v[3];
        }
    }
    const __amdgpu_buffer_rsrc_t pre_rsrc = make_rsrc(pre, (uint32_t)T * 4 * C * 4);
    const __amdgpu_buffer_rsrc_t out_rsrc = make_rsrc(out, (uint32_t)T * C * 4);
    const int my_gate = (s * C + u) * 4;
    // this unit's place in a row of the state; the quad's other lanes write to the row's unused places
    const int h_out = s == 0 ? RecurrenceLds<C>::place(u) : (u % 8) * kSegPitch + kSeg + s;
    if (tid < kRow) lds.h[2 * kSteps - 1][tid] = 0.f;          // "the step before the first"
    int seen = 0, ahead = 0;
    float next[kSteps];
    auto fetch = [&](int c) {                                  // past the end: zeros (the descriptor ends there)
        if (WAIT) {
            seen = max(seen, __builtin_amdgcn_readfirstlane(ahead));
            wait_for(c + 1, seen, [&] { return __builtin_amdgcn_readfirstlane(peek(arrived)); });
        }
#pragma unroll
        for (int i = 0; i < kSteps; ++i) next[i] = load_f32<WAIT ? kAgent : 0>(pre_rsrc, (c * kSteps + i) * 4 * C * 4 + my_gate);
        if (WAIT) ahead = peek(arrived);                       // looked at when the next chunk is due
    };
    // chunk c's states, from LDS to global memory (past the end: dropped)
    auto store_chunk = [&](int c) {
        constexpr int kOwn = kSteps / 4;
        static_assert(kOwn == 1 || kOwn == 2, "states of a chunk per thread");
        const int step = kOwn * tid / C, unit = kOwn * tid % C, at = ((c * kSteps + step) * C + unit) * 4;
        const float *from = lds.h[(c & 1) * kSteps + step];
        if constexpr (kOwn == 1) store_f32<POST ? kAgent : 0>(out_rsrc, at, from[RecurrenceLds<C>::place(unit)]);
        else {
            const f32x2 v{from[RecurrenceLds<C>::place(unit)], from[RecurrenceLds<C>::place(unit + 1)]};
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), out_rsrc, at, 0, POST ? kAgent : 0);
        }
    };
    // a wavefront's part of one more chunk of states has left for good
    auto post = [&]() {
        wait_memory<0>();
        if ((tid & 63) == 0) __hip_atomic_fetch_add(done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    fetch(0);
    lds_barrier();
    const GateKind mine = gate_kind(s == 2), of_cell = gate_kind(true);
    float cell = 0.f;
    const float *h_in = &lds.h[2 * kSteps - 1][l8 * kSegPitch];
    float *row = nullptr;
    const float *z_in = nullptr;
    auto step = [&]() {
        float acc[8] = {};
        acc[0] = *z_in;
#pragma unroll
        for (int k = 0; k < kSeg; k += 4) {
            const f32x4 hv = load4(h_in + k);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[j] = fmaf(w[j][k + e], hv[(e + 1) & 3], acc[j]);   // see place()
        }
        // lane ^ 7 (mirrored halves) holds the row in the slot ^ 7; then the quad
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] += quad<kHalfMirror>(acc[j ^ 7]);
        const float z = (acc[0] + quad<kXor1>(acc[1])) + quad<kXor2>(acc[2] + quad<kXor1>(acc[3]));
        const float a = gate_value(z, mine);
        cell = next_cell(a, cell);                             // the state of the quad's lane 0; what the others hold is not read
        row[h_out] = quad<0xFF>(a) * gate_value(cell, of_cell);
        h_in = row + l8 * kSegPitch;
        row += kRow;
        z_in += 4 * C;
        lds_barrier();
    };
    auto take = [&](int c) {
#pragma unroll
        for (int i = 0; i < kSteps; ++i) lds.pre[i][tid] = next[i];
        row = lds.h[(c & 1) * kSteps];
        z_in = &lds.pre[0][tid];
    };
    walk_chunks<kSteps, POST>(T, take, store_chunk, step, fetch, post, lds_barrier);
}

// D[4 x 64] += A[4 x 16] B[16 x 64] as 16 instructions of 16 4x4 blocks: lane l gives A[l % 4][l / 4]
// (every instruction broadcasts one column of it to all blocks) and B[0..15][l], and holds D[0..3][l].
template <int... J>
__device__ __forceinline__ void mfma_rows(float a, const float *b, f32x4 &even, f32x4 &odd, std::integer_sequence<int, J...>)
{
    ((((J & 1) ? odd : even) = __builtin_amdgcn_mfma_f32_4x4x1f32(a, b[J], (J & 1) ? odd : even, 4, J, 0)), ...);
}

// A layer's gate pre-activations for one sequence, some tokens at a time.  FIRST: layer 1's, of the compressed embeddings,
// which are all there: eight tokens at a time, ahead of layer 1.  Else layer 2's, a chunk at a time as layer 1
// finishes them; they replace layer 1's in `pre`: layer 1 has consumed a token's before it hands the
// token on.  A thread keeps its gate row of W_ih in registers, the tokens are the rows of a matrix
// product of few rows (blocks of 4: a 16-row product took 3.4 us a chunk and held layer 2 up, 5 us
// between chunks), and the results leave in whole lines.
template <int C, bool FIRST>
__device__ __forceinline__ void gates_ahead(const float *__restrict__ x, const float *__restrict__ w_ih,
                                            const float *__restrict__ b_ih, const float *__restrict__ b_hh, int T,
                                            float *__restrict__ pre, const int *arrived, int *done, RecurrenceLds<C> &lds)
{
    constexpr int kPitch = RecurrenceLds<C>::kInPitch;
    constexpr int kTokens = FIRST ? kGateTokens : kChunk<C>, kBlocks = kTokens / 4, kPolicy = FIRST ? 0 : kAgent;
    static_assert(kTokens % 4 == 0 && kTokens <= kGateTokens && kTokens % kChunk<C> == 0 && kTokens * C / 4 <= 4 * C, "whole blocks and chunks");
    const int tid = threadIdx.x, lane = tid & 63;
    const __amdgpu_buffer_rsrc_t x_rsrc = make_rsrc(x, (uint32_t)T * C * 4);
    const __amdgpu_buffer_rsrc_t pre_rsrc = make_rsrc(pre, (uint32_t)T * 4 * C * 4);
    auto load = [&](int c) {                                   // 16 bytes per thread; past the end: zeros
        return __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(x_rsrc, (c * kTokens * C + tid * 4) * 4, 0, kPolicy));
    };
    const bool loads = tid < kTokens * C / 4;
    i32x4 v = {};
    if (FIRST && loads) v = load(0);
    float w[C];                                                // row tid
#pragma unroll
    for (int k = 0; k < C; k += 4) {
        const f32x4 q = load4_param(w_ih + (size_t)tid * C + k);
#pragma unroll
        for (int e = 0; e < 4; ++e) w[k + e] = q[e];
    }
    const float bias = b_ih[tid] + b_hh[tid];
    const int rounds = (T + kTokens - 1) / kTokens;
    int seen = 0;
    for (int c = 0; c < rounds; ++c) {
        if (!FIRST) wait_for((c + 1) * (C / 16), seen, [&] { return __builtin_amdgcn_readfirstlane(peek(arrived)); });
        float *in = lds.in[c & 1];
        if (loads) {
            if (!FIRST) v = load(c);
            *reinterpret_cast<i32x4 *>(in + (tid / (C / 4)) * kPitch + (tid % (C / 4)) * 4) = v;
            if (FIRST) v = load(c + 1);
        }
        lds_barrier();
        f32x4 even[kBlocks], odd[kBlocks];
#pragma unroll
        for (int q = 0; q < kBlocks; ++q) {
            even[q] = f32x4{bias, bias, bias, bias};
            odd[q] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        const float *ip = in + (lane & 3) * kPitch + (lane >> 2);
#pragma unroll
        for (int k = 0; k < C / 16; ++k)
#pragma unroll
            for (int q = 0; q < kBlocks; ++q)
                mfma_rows(ip[q * 4 * kPitch + k * 16], w + k * 16, even[q], odd[q], std::make_integer_sequence<int, 16>());
#pragma unroll
        for (int q = 0; q < kBlocks; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i)                        // past the end: dropped
                store_f32<kAgent>(pre_rsrc, ((c * kTokens + q * 4 + i) * 4 * C + tid) * 4, even[q][i] + odd[q][i]);
        wait_memory<0>();
        lds_barrier();
        if (tid == 0) publish(done, chunks_there(c + 1, kTokens, kChunk<C>));
    }
}

// Both LSTM layers of every sequence in one launch of 3 or 4 workgroups per sequence: the gate pre-activations of
// layer 1 (GATES; else a launch before has made them), layer 1, the gate pre-activations between the layers, layer 2; each
// works behind the one before, chunk by chunk, so that a call takes T plus about 20 steps (30 at C = 64, whose chunks are
// longer) instead of 2T.  A workgroup takes its role by ticket: first all of the first role, and so on.  Tickets are drawn
// by workgroups that run, so whatever a workgroup waits for is done by a workgroup that already runs and waits, if
// at all, for a lower ticket only; the first role waits for nobody.  Hence every wait ends, whatever the
// order in which workgroups are started and whatever else runs on the GPU.  (Counters that another call
// writes over, against the rules, end them too: see handover.h.)
// GATES saves a launch over all tokens, but layer 1 then waits for a compute unit that has to load its 256 KiB of weights
// first (some 5 us); see run() for where it pays.
template <int C, bool GATES>
__global__ __launch_bounds__(4 * C) void hash_recurrence(float *pre, const float *__restrict__ c0, const float *__restrict__ w_ih1,
                                                         const float *__restrict__ b_ih1, const float *__restrict__ b_hh1,
                                                         const float *__restrict__ w_hh1,
                                                         const float *__restrict__ w_ih2, const float *__restrict__ w_hh2,
                                                         const float *__restrict__ b_ih2, const float *__restrict__ b_hh2,
                                                         int n_seq, int T, float *h1, float *h2, int *counters)
{
    __shared__ __attribute__((aligned(16))) RecurrenceLds<C> lds;
    if (threadIdx.x == 0) lds.ticket = __hip_atomic_fetch_add(counters, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int ticket = __builtin_amdgcn_readfirstlane(lds.ticket);
    const Role of = GATES ? role_of_four(ticket, n_seq) : role_of(ticket, n_seq);
    const int role = of.what, seq = of.seq;
    float *p = pre + (size_t)seq * T * 4 * C, *a = h1 + (size_t)seq * T * C, *b = h2 + (size_t)seq * T * C;
    int *layer1_done = counters + layer1_line(seq), *gates2_done = counters + gates2_line(seq), *gates1_done = counters + gates1_line(seq);
    if (GATES && role < 0) gates_ahead<C, true>(c0 + (size_t)seq * T * C, w_ih1, b_ih1, b_hh1, T, p, nullptr, gates1_done, lds);
    else if (role == 0) lstm_layer<C, GATES, true>(p, w_hh1, T, a, gates1_done, layer1_done, lds);
    else if (role == 1) gates_ahead<C, false>(a, w_ih2, b_ih2, b_hh2, T, p, layer1_done, gates2_done, lds);
    else lstm_layer<C, true, false>(p, w_hh2, T, b, gates2_done, nullptr, lds);
}

// One layer alone, a workgroup per sequence: for batches of so many sequences that three workgroups
// for each would not all run at a time, where doing the layers one after the other loses nothing.
template <int C>
__global__ __launch_bounds__(4 * C) void hash_lstm(const float *__restrict__ pre, const float *__restrict__ w_hh, int T,
                                                   float *__restrict__ out)
{
    __shared__ __attribute__((aligned(16))) RecurrenceLds<C> lds;
    lstm_layer<C, false, false>(pre + (size_t)blockIdx.x * T * 4 * C, w_hh, T, out + (size_t)blockIdx.x * T * C, nullptr,
                                nullptr, lds);
}

// ---- attention ----------------------------------------------------------------------------------
// Sum / maximum over the 32 lanes of a half wavefront.
__device__ __forceinline__ float half_sum(float v)
{
    v = row_sum(v);
    return v + __shfl_xor(v, 16, 64);
}
__device__ __forceinline__ float half_max(float v)
{
    v = row_max(v);
    return fmaxf(v, __shfl_xor(v, 16, 64));
}

// Sparse attention + residual: r[t] = c0[t] + sum_u sparsemax_u(h2[t] . h2[u]) h2[u], for `queries` (at
// most 16) consecutive tokens of one sequence per workgroup of 8 wavefronts.  Scores and weights sit in
// LDS, [queries][pitch]; both products run on the matrix units with the queries as columns.
// SparseMax: the threshold tau with sum_u max(s_u - tau, 0) = 1 is (sum of the support - 1) / size of the
// support; starting from the support of max - 1, taking the closed form on the scores above it and
// dropping what falls below it ends, after a few rounds, with the support that reproduces itself.
template <int C>
__global__ __launch_bounds__(512) void hash_attention(const float *__restrict__ h2, const float *__restrict__ c0, int T,
                                                      int queries, int blocks_per_seq, int pitch, float *__restrict__ r)
{
    extern __shared__ __attribute__((aligned(16))) float s[];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, col = lane & 15, g = lane >> 4;
    const int seq = blockIdx.x / blocks_per_seq, t0 = (blockIdx.x % blocks_per_seq) * queries;
    const int nq = min(queries, T - t0);
    const float *hs = h2 + (size_t)seq * T * C;
    const int T16 = (T + 15) & ~15;
    f32x4 q[C / 16];
#pragma unroll
    for (int k = 0; k < C / 16; ++k) q[k] = load4(hs + (size_t)(t0 + min(col, nq - 1)) * C + k * 16 + 4 * g);
    for (int u0 = wv * 16; u0 < T16; u0 += 8 * 16) {
        const float *key = hs + (size_t)min(u0 + col, T - 1) * C + 4 * g;
        f32x4 k4[C / 16];
#pragma unroll
        for (int k = 0; k < C / 16; ++k) k4[k] = load4(key + k * 16);
        loads_issued();
        f32x4 d0 = {}, d1 = {};
#pragma unroll
        for (int k = 0; k < C / 16; k += 2) {
            d0 = mfma4(k4[k], q[k], d0);
            d1 = mfma4(k4[k + 1], q[k + 1], d1);
        }
        d0 += d1;
        if (col < queries) *reinterpret_cast<f32x4 *>(s + col * pitch + u0 + 4 * g) = d0;
    }
    __syncthreads();
    for (int row = wv * 2 + (lane >> 5); row < ((nq + 1) & ~1); row += 16) {   // both halves of a wavefront take part
        float *z = s + min(row, nq - 1) * pitch;
        const int l = lane & 31;
        // the first kHeld * 32 scores of a row in registers, what is beyond stays in LDS
        constexpr int kHeld = 12;
        float held[kHeld];
        float mx = -FLT_MAX;
#pragma unroll
        for (int i = 0; i < kHeld; ++i) held[i] = i * 32 + l < T ? z[i * 32 + l] : -FLT_MAX;
#pragma unroll
        for (int i = 0; i < kHeld; ++i) mx = fmaxf(mx, held[i]);
        for (int u = kHeld * 32 + l; u < T; u += 32) mx = fmaxf(mx, z[u]);
        mx = half_max(mx);
        float tau = -1.f, size = 0.f;                          // relative to the largest score
        for (;;) {
            float sum = 0.f, cnt = 0.f;
            auto take = [&](float score) {
                const float v = score - mx;
                sum += v > tau ? v : 0.f;
                cnt += v > tau ? 1.f : 0.f;
            };
#pragma unroll
            for (int i = 0; i < kHeld; i += 4)
                if (i * 32 < T) {
#pragma unroll
                    for (int e = i; e < i + 4; ++e) take(held[e]);
                }
            for (int u = kHeld * 32 + l; u < T; u += 32) take(z[u]);
            sum = half_sum(sum);
            cnt = half_sum(cnt);
            if (!(cnt > 0.f) || (size > 0.f && cnt >= size)) break;   // the support stands: it shrinks or the loop ends
            tau = (sum - 1.f) / cnt;
            size = cnt;
        }
        if (row < nq) {
#pragma unroll
            for (int i = 0; i < kHeld; ++i)
                if (i * 32 + l < T16) z[i * 32 + l] = i * 32 + l < T ? fmaxf(held[i] - mx - tau, 0.f) : 0.f;
            for (int u = kHeld * 32 + l; u < T16; u += 32) z[u] = u < T ? fmaxf(z[u] - mx - tau, 0.f) : 0.f;
        }
    }
    __syncthreads();
    if (wv * 16 >= C) return;
    // r^T[c, query] = sum_u h2[u, c] p[query, u]: 16 columns c per wavefront
    const int c = wv * 16;
    f32x4 acc = {};
    const float *p = s + min(col, nq - 1) * pitch + 4 * g;
    const float *hv = hs + c + col;
    for (int u0 = 0; u0 < T16; u0 += 64) {                     // four blocks of 16 keys' loads in flight
        f32x4 pv[4], v[4];
        bool any = false;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            pv[b] = u0 + b * 16 < T16 ? load4(p + u0 + b * 16) : f32x4{0.f, 0.f, 0.f, 0.f};
            any |= pv[b][0] > 0.f || pv[b][1] > 0.f || pv[b][2] > 0.f || pv[b][3] > 0.f;
        }
        if (!__any(any)) continue;
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int j = 0; j < 4; ++j) v[b][j] = hv[(size_t)min(u0 + b * 16 + 4 * g + j, T - 1) * C];
        loads_issued();
        // A key of weight 0 is multiplied too.  A state is NaN or within [-1, 1]; a key with a NaN has a NaN score
        // and weight 0 for every query: any finite number in its place (the median with a NaN is the least of
        // the others) leaves it out of the sums.
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int j = 0; j < 4; ++j) v[b][j] = __builtin_amdgcn_fmed3f(v[b][j], -2.f, 2.f);
#pragma unroll
        for (int b = 0; b < 4; ++b) acc = mfma4(v[b], pv[b], acc);
    }
    if (col < nq) {
        const size_t at = ((size_t)seq * T + t0 + col) * C + c + 4 * g;
        *reinterpret_cast<f32x4 *>(r + at) = acc + load4(c0 + at);
    }
}

// ---- heads --------------------------------------------------------------------------------------
// The k most probable experts of a token: 16 lanes hold its logits, NT each (experts col, col + 16, ...).
template <int NT>
__device__ __forceinline__ void best_experts(const float *row, int l, int n, int n_tokens, int E, int top_k, int col,
                                             int32_t *__restrict__ ids, float *__restrict__ alpha)
{
    float z[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) z[i] = i * 16 + col < E ? row[i * 16 + col] : -FLT_MAX;
    float mx = -FLT_MAX, sum = 0.f;
    for (int j = 0; j < top_k; ++j) {
        // Largest remaining logit (NaN is none), ties to the lower expert id: the largest first and then whose it is, which
        // takes half of the instructions that carrying both along does (8192 tokens, 6 layers of 128 experts 21.2 -> 19.8
        // us, 2664 tokens 10.6 -> 9.9).
        float best = -FLT_MAX;
#pragma unroll
        for (int i = 0; i < NT; ++i) best = fmaxf(best, z[i]);
        best = row_max(best);
        int arg = E;
#pragma unroll
        for (int i = NT - 1; i >= 0; --i) arg = z[i] == best ? i * 16 + col : arg;
        arg = best > -FLT_MAX ? arg : E;
        arg = min(arg, dpp<kXor1>(arg));
        arg = min(arg, dpp<kXor2>(arg));
        arg = min(arg, dpp<kHalfMirror>(arg));
        arg = min(arg, dpp<kMirror>(arg));
        if (j == 0) {
            mx = best;
#pragma unroll
            for (int i = 0; i < NT; ++i) sum += __expf(z[i] - mx);         // an expert that is not there adds nothing
            sum = row_sum(sum);
        }
        if (col == 0 && n < n_tokens) {
            const size_t at = ((size_t)l * n_tokens + n) * top_k + j;
            ids[at] = arg < E ? arg : 0;
            alpha[at] = __expf(best - mx) / sum;
        }
#pragma unroll
        for (int i = 0; i < NT; ++i)
            if (i * 16 + col == arg) z[i] = -FLT_MAX;                      // taken
    }
}

// Per MoE layer the E logits of a token, their SoftMax, and the k most probable experts.  A workgroup
// takes TT*16 tokens and one layer: all operands go to LDS at once, its four wavefronts make NT tiles of
// 16 experts in turn (matrix product, experts as rows), hand the logits over in LDS, and then take a
// token per 16 lanes with NT logits in each lane's registers.
template <int C, int NT, int TT>
constexpr int heads_lds_bytes() { return C / 32 * (NT + TT) * 16 * TileRow<float>::kBytes; }

template <int C, int NT, int TT, bool DIRECT>
__global__ __launch_bounds__(256) void hash_heads(const float *__restrict__ r, const float *__restrict__ w_out,
                                                  const float *__restrict__ b_out, int E, int top_k, int n_tokens,
                                                  int32_t *__restrict__ ids, float *__restrict__ alpha)
{
    constexpr int kPitch = NT * 16 + 16, kMine = (NT + 3) / 4, kSteps32 = C / 32;
    constexpr int kW = NT * 16 * TileRow<float>::kBytes, kStage = kW + TT * 16 * TileRow<float>::kBytes;
    typedef TileLoader<float, NT * 16, 4, DIRECT> LoadW;
    typedef TileLoader<float, TT * 16, 4, DIRECT> LoadX;
    constexpr int kStepLoads = LoadW::kLoads + LoadX::kLoads;
    static_assert(TT * 16 * kPitch * 4 <= heads_lds_bytes<C, NT, TT>(), "the logits replace the operands");
    static_assert((kSteps32 - 1) * kStepLoads <= 63, "vmcnt range");
    extern __shared__ __attribute__((aligned(1024))) char tiles[];
    float *logit = reinterpret_cast<float *>(tiles);
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), col = lane & 15, g = lane >> 4;
    const int l = blockIdx.y, n0 = blockIdx.x * TT * 16;
    f32x4 bias[kMine];                                         // asked for first: behind the products they would be waited for
#pragma unroll
    for (int i = 0; i < kMine; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) bias[i][e] = b_out[l * E + min((i * 4 + wv) * 16 + 4 * g + e, E - 1)];
    loads_issued();
    {
        const LoadW load_w(w_out + (size_t)l * E * C, E, C, lane, wv);
        const LoadX load_x(r + (size_t)n0 * C, n_tokens - n0, C, lane, wv);
#pragma unroll
        for (int s = 0; s < kSteps32; ++s) {
            load_w.issue(s, tiles + s * kStage);
            load_x.issue(s, tiles + s * kStage + kW);
        }
    }
    f32x4 acc[kMine][TT] = {};
    auto multiply = [&](int s) {
        const char *tile = tiles + s * kStage;
        float b[TT][8];
#pragma unroll
        for (int m = 0; m < TT; ++m) TileRow<float>::read(tile + kW, m * 16 + col, g, b[m]);
        Parts pb[TT];
        if constexpr (TT > 1)
#pragma unroll
            for (int m = 0; m < TT; ++m) pb[m] = parts_of(b[m]);
#pragma unroll
        for (int i = 0; i < kMine; ++i) {
            if (NT < 4 && i * 4 + wv >= NT) continue;
            float a[8];
            TileRow<float>::read(tile, (i * 4 + wv) * 16 + col, g, a);
            if constexpr (TT > 1) {
                const Parts pa = parts_of(a);
#pragma unroll
                for (int m = 0; m < TT; ++m) acc[i][m] = mfma_parts(pa, pb[m], acc[i][m]);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e)
#pragma unroll
                    for (int m = 0; m < TT; ++m)
                        acc[i][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[m][e], acc[i][m], 0, 0, 0);
            }
        }
    };
    tiles_arrived<(kSteps32 - 1) * kStepLoads, DIRECT>();
    __builtin_amdgcn_s_barrier();
    multiply(0);
    tiles_arrived<(kSteps32 - 2) * kStepLoads, DIRECT>();
    __builtin_amdgcn_s_barrier();
    multiply(1);
    if (kSteps32 > 2) {
        tiles_arrived<kStepLoads, DIRECT>();
        __builtin_amdgcn_s_barrier();
        multiply(2);
        tiles_arrived<0, DIRECT>();
        __builtin_amdgcn_s_barrier();
        multiply(3);
    }
    if (TT > 1 && any_overflow(acc)) {
#pragma unroll 1
        for (int t = 0; t < kMine * TT; ++t) {
            const int i = t / TT, m = t % TT;
            if (NT < 4 && i * 4 + wv >= NT) continue;
            f32x4 again = {};
#pragma unroll 1
            for (int s = 0; s < kSteps32; ++s) {
                float a[8], b[8];
                TileRow<float>::read(tiles + s * kStage, (i * 4 + wv) * 16 + col, g, a);
                TileRow<float>::read(tiles + s * kStage + kW, m * 16 + col, g, b);
#pragma unroll
                for (int e = 0; e < 8; ++e) again = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], again, 0, 0, 0);
            }
#pragma unroll
            for (int j = 0; j < kMine * TT; ++j)
                if (j == t) acc[j / TT][j % TT] = where_overflowed(acc[j / TT][j % TT], again);
        }
    }
    lds_barrier();                                             // every operand has been read
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
        const int tile = i * 4 + wv;
        if (NT < 4 && tile >= NT) continue;
#pragma unroll
        for (int m = 0; m < TT; ++m)
            *reinterpret_cast<f32x4 *>(&logit[(m * 16 + col) * kPitch + tile * 16 + 4 * g]) = acc[i][m] + bias[i];
    }
    __syncthreads();
#pragma unroll 1
    for (int m = 0; m < TT; ++m) {
        const int tok = m * 16 + wv * 4 + g;
        best_experts<NT>(logit + tok * kPitch, l, n0 + tok, n_tokens, E, top_k, col, ids, alpha);
    }
}

// The same for many tokens and layers, all products through bf16 parts.  In hash_heads a workgroup fetches and cuts a layer's
// weights (64 KiB of 128 experts) for 32 tokens, and cutting them takes as long as multiplying: 8192 tokens, 6
// layers of 128 experts 19.8 us, of which the matrix instructions take 4.  Here WAVES wavefronts keep the layer's weights, cut
// once, in registers (NT / WAVES tiles of 16 experts each) and walk over tiles of 16 * TT tokens.  A wavefront cuts one
// 16 x 32 piece of the next tile and puts the parts into LDS in the order in which the matrix instruction takes
// them, so that nothing is cut twice; the piece behind it is on its way from memory meanwhile.  One barrier a
// tile: parts and logits have two places each.  17.1 us (5 before the first product), 12 layers of 64 experts 25.0 -> 17.6, 6 layers of
// 256 experts 45.4 -> 28.5; bits unchanged.
template <int C, int NT, int WAVES>
__global__ __launch_bounds__(WAVES * 64, 2) void hash_heads_walk(const float *__restrict__ r, const float *__restrict__ w_out,
                                                                 const float *__restrict__ b_out, int E, int top_k, int n_tokens,
                                                                 int32_t *__restrict__ ids, float *__restrict__ alpha)
{
    constexpr int kMine = NT / WAVES, TT = WAVES / 4, kSteps32 = C / 32, kPitch = NT * 16 + 16, kTokens = heads_walk_tokens(WAVES);
    static_assert(NT % WAVES == 0 && WAVES % 4 == 0 && kTokens == 16 * TT && kSteps32 <= 4, "tiles and pieces of a wavefront");
    __shared__ bf16x8 parts[2][TT][kSteps32][3][64];
    __shared__ __attribute__((aligned(16))) float logit[2][kTokens * kPitch];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), col = lane & 15, g = lane >> 4;
    const int l = blockIdx.y, tiles = (n_tokens + kTokens - 1) / kTokens, stride = gridDim.x;
    const float *w_l = w_out + (size_t)l * E * C;
    // this wavefront's piece of a tile: 16 tokens, 32 of the C values
    const int piece_t = wv >> 2, piece_s = wv & 3;
    const bool cuts = piece_s < kSteps32;
    const __amdgpu_buffer_rsrc_t r_rsrc = make_rsrc(r, (uint32_t)n_tokens * C * 4);
    f32x4 raw[2];
    auto ask = [&](int tile) {                                 // past the end: zeros
        const int at = ((tile * kTokens + piece_t * 16 + col) * C + piece_s * 32 + 8 * g) * 4;
#pragma unroll
        for (int h = 0; h < 2; ++h) raw[h] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r_rsrc, at + h * 16, 0, 0));
    };
    auto cut = [&](int buf) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = raw[e >> 2][e & 3];
        const Parts p = parts_of(v);
        parts[buf][piece_t][piece_s][0][lane] = p.hi;
        parts[buf][piece_t][piece_s][1][lane] = p.mid;
        parts[buf][piece_t][piece_s][2][lane] = p.lo;
    };
    int tile = blockIdx.x;
    if (cuts) ask(tile);
    f32x4 bias[kMine];
    Parts w[kMine][kSteps32];
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
        const int first = (i * WAVES + wv) * 16;
#pragma unroll
        for (int e = 0; e < 4; ++e) bias[i][e] = b_out[l * E + min(first + 4 * g + e, E - 1)];
        const float *row = w_l + (size_t)min(first + col, E - 1) * C + 8 * g;
#pragma unroll
        for (int s = 0; s < kSteps32; ++s) {
            float v[8];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const f32x4 q = load4_param(row + s * 32 + 4 * h);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[4 * h + e] = q[e];
            }
            w[i][s] = parts_of(v);
        }
    }
    if (cuts) {
        cut(0);
        ask(tile + stride);
    }
    lds_barrier();
    for (int buf = 0; tile < tiles; tile += stride, buf ^= 1) {
        f32x4 acc[kMine][TT] = {};
#pragma unroll
        for (int s = 0; s < kSteps32; ++s)
#pragma unroll
            for (int m = 0; m < TT; ++m) {
                const Parts x{parts[buf][m][s][0][lane], parts[buf][m][s][1][lane], parts[buf][m][s][2][lane]};
#pragma unroll
                for (int i = 0; i < kMine; ++i) acc[i][m] = mfma_parts(w[i][s], x, acc[i][m]);
            }
        if (any_overflow(acc)) {
#pragma unroll 1
            for (int t = 0; t < kMine * TT; ++t) {
                const int i = t / TT, m = t % TT;
                const float *row = w_l + (size_t)min((i * WAVES + wv) * 16 + col, E - 1) * C + 8 * g;
                const float *token = r + (size_t)min(tile * kTokens + m * 16 + col, n_tokens - 1) * C + 8 * g;
                f32x4 again = {};
#pragma unroll 1
                for (int s = 0; s < kSteps32; ++s)
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        again = __builtin_amdgcn_mfma_f32_16x16x4f32(row[s * 32 + e], token[s * 32 + e], again, 0, 0, 0);
#pragma unroll
                for (int j = 0; j < kMine * TT; ++j)
                    if (j == t) acc[j / TT][j % TT] = where_overflowed(acc[j / TT][j % TT], again);
            }
        }
#pragma unroll
        for (int i = 0; i < kMine; ++i)
#pragma unroll
            for (int m = 0; m < TT; ++m)
                *reinterpret_cast<f32x4 *>(&logit[buf][(m * 16 + col) * kPitch + (i * WAVES + wv) * 16 + 4 * g]) = acc[i][m] + bias[i];
        if (cuts) {
            cut(buf ^ 1);
            ask(tile + 2 * stride);
        }
        lds_barrier();
        const int tok = wv * 4 + g;
        best_experts<NT>(&logit[buf][tok * kPitch], l, tile * kTokens + tok, n_tokens, E, top_k, col, ids, alpha);
    }
}

// ---- one call -----------------------------------------------------------------------------------
// Sequences whose layers run side by side: three workgroups each, or four with the gate pre-activations of layer 1 among
// them, one per compute unit (a workgroup of the recurrence fills the registers of its compute unit).
constexpr int kSideBySide = 256 / 3;
// Gate pre-activations of layer 1 in the recurrence's launch, us a call, before -> with: C = 128 60 x 40 tokens 69.2 -> 67.1,
// 48 x 128 141.4 -> 137.5, 64 x 128 145.6 -> 139.6, 64 x 100 126.8 -> 121.2, 16 x 192 162.6 -> 162.2; C = 64 60 x 40 50.5 ->
// 48.0, 48 x 128 94.1 -> 91.3, 16 x 512 241.1 -> 241.6.  With few sequences or tokens the launch in front is short:
// 1 x 128 106.9 -> 110.3, 2 x 512 339.8 -> 345.0, 8 x 333 243.9 -> 244.3, 12 x 333 at C = 64 160.0 -> 160.7.
inline bool gates_in_recurrence(int n_seq, int tokens) { return n_seq >= 16 && n_seq <= 256 / 4 && tokens >= 2048; }
constexpr int kMaxScoreBytes = 144 * 1024;                     // LDS for an attention block's scores

template <int C>
int run(const HashShape &sh, const float *p, const void *x, int n_seq, int T, int32_t *ids, float *alpha, float *ws,
        hipStream_t st)
{
    const int N = n_seq * T, d = sh.d_model;
    // parameters, packed in this order
    const float *w_in = p, *b_in = w_in + (size_t)C * d;
    const float *w_ih1 = b_in + C, *w_hh1 = w_ih1 + 4 * C * C, *b_ih1 = w_hh1 + 4 * C * C, *b_hh1 = b_ih1 + 4 * C;
    const float *w_ih2 = b_hh1 + 4 * C, *w_hh2 = w_ih2 + 4 * C * C, *b_ih2 = w_hh2 + 4 * C * C, *b_hh2 = b_ih2 + 4 * C;
    const float *w_out = b_hh2 + 4 * C, *b_out = w_out + (size_t)sh.L * sh.E * C;
    // workspace
    float *c0 = ws, *pre = c0 + (size_t)N * C, *h1 = pre + (size_t)N * 4 * C, *h2 = h1 + (size_t)N * C,
          *r = h2 + (size_t)N * C;
    // Counters of the recurrence, in the part of the workspace that the attention writes later; cleared by the first launch.
    int *counters = reinterpret_cast<int *>(r);                // N*C words, of which a sequence needs 3*kLine and the ticket kLine
    static_assert(C >= 4 * kLine, "counters fit");
    const __bf16 *xb = (const __bf16 *)x;
    // Tiles: as large as leave every compute unit (nearly) one workgroup.
    const int n_counters = n_seq <= kSideBySide ? counter_words(n_seq) : 0;
    auto dense = [&](auto kernel, int tokens, int rows, auto in, const float *w, const float *ba, const float *bb, int k,
                     int units, float *out, int n_clear) {
        hipLaunchKernelGGL(kernel, dim3((N + tokens - 1) / tokens, units / rows), dim3(256), 0, st, in, w, ba, bb, k, units, N, out,
                           counters, n_clear);
    };
    // Tiles are loaded straight into LDS, 16 bytes at a time, where x and the parameters start at a 16-byte
    // boundary (rows are multiples of 16 bytes).  Elsewhere the smallest tiles go through registers.
    const bool direct = ((reinterpret_cast<uintptr_t>(p) | reinterpret_cast<uintptr_t>(x)) & 15u) == 0;
    if (!direct) dense(hash_dense<1, 1, 1, 1, 4, 2, 4, __bf16, false>, 16, 16, xb, w_in, b_in, nullptr, d, C, c0, n_counters);
    else if (N >= 6144) dense(hash_dense<1, 4, 4, 1, 1, 2, 4, __bf16, true>, 64, 64, xb, w_in, b_in, nullptr, d, C, c0, n_counters);
    else if (N >= 2048) dense(hash_dense<1, 2, 2, 2, 1, 2, 4, __bf16, true>, 64, 32, xb, w_in, b_in, nullptr, d, C, c0, n_counters);
    else dense(hash_dense<1, 1, 1, 1, 4, 2, 4, __bf16, true>, 16, 16, xb, w_in, b_in, nullptr, d, C, c0, n_counters);
    auto gates = [&](const float *in, const float *w_ih, const float *b_ih, const float *b_hh) {
        if (!direct) dense(hash_dense<1, 1, 4, 1, 1, 2, 3, float, false>, 16, 64, in, w_ih, b_ih, b_hh, C, 4 * C, pre, 0);
        else if (N >= 2048) dense(hash_dense<2, 2, 2, 2, 1, 2, 2, float, true>, 64, 64, in, w_ih, b_ih, b_hh, C, 4 * C, pre, 0);
        else dense(hash_dense<1, 1, 4, 1, 1, 2, 3, float, true>, 16, 64, in, w_ih, b_ih, b_hh, C, 4 * C, pre, 0);
    };
    auto recurrence = [&](auto kernel, int roles) {
        hipLaunchKernelGGL(kernel, dim3(roles * n_seq), dim3(4 * C), 0, st, pre, c0, w_ih1, b_ih1, b_hh1, w_hh1, w_ih2, w_hh2, b_ih2,
                           b_hh2, n_seq, T, h1, h2, counters);
    };
    const bool gates_too = gates_in_recurrence(n_seq, N);
    if (!gates_too) gates(c0, w_ih1, b_ih1, b_hh1);
    if (gates_too) {
        recurrence(hash_recurrence<C, true>, 4);
    } else if (n_seq <= kSideBySide) {
        recurrence(hash_recurrence<C, false>, 3);
    } else {
        hipLaunchKernelGGL(hash_lstm<C>, dim3(n_seq), dim3(4 * C), 0, st, pre, w_hh1, T, h1);
        gates(h1, w_ih2, b_ih2, b_hh2);
        hipLaunchKernelGGL(hash_lstm<C>, dim3(n_seq), dim3(4 * C), 0, st, pre, w_hh2, T, h2);
    }
    // 16 queries per attention block, or 8 where the scores of 16 would not fit the LDS
    const int pitch = (T + 15) / 16 * 16 + 4;
    const int queries = 16 * pitch * 4 <= kMaxScoreBytes ? 16 : 8;
    const int score_bytes = queries * pitch * 4, blocks_per_seq = (T + queries - 1) / queries;
    if (score_bytes > 64 * 1024) {
        static LdsGrant grant;
        const int rc = allow_lds(grant, reinterpret_cast<const void *>(&hash_attention<C>), kMaxScoreBytes);
        if (rc) return rc;
    }
    hipLaunchKernelGGL(hash_attention<C>, dim3(n_seq * blocks_per_seq), dim3(512), score_bytes, st, h2, c0, T, queries,
                       blocks_per_seq, pitch, r);
    int err = 0;
    auto heads = [&](auto nt, auto tt, auto dir) {
        constexpr int NT = decltype(nt)::value, TT = decltype(tt)::value, kBytes = heads_lds_bytes<C, NT, TT>();
        constexpr bool DIRECT = decltype(dir)::value;
        if (kBytes > 64 * 1024) {
            static LdsGrant grant;
            err = allow_lds(grant, reinterpret_cast<const void *>(&hash_heads<C, NT, TT, DIRECT>), kBytes);
            if (err) return;
        }
        hipLaunchKernelGGL((hash_heads<C, NT, TT, DIRECT>), dim3((N + TT * 16 - 1) / (TT * 16), sh.L), dim3(256), kBytes, st, r, w_out,
                           b_out, sh.E, sh.top_k, N, ids, alpha);
    };
    auto heads_of = [&](auto tt, auto dir) {
        if (sh.E <= 16) heads(std::integral_constant<int, 1>(), tt, dir);
        else if (sh.E <= 64) heads(std::integral_constant<int, 4>(), tt, dir);
        else if (sh.E <= 128) heads(std::integral_constant<int, 8>(), tt, dir);
        else heads(std::integral_constant<int, 16>(), tt, dir);
    };
    auto walk = [&](auto nt, auto waves) {
        constexpr int NT = decltype(nt)::value, WAVES = decltype(waves)::value;
        hipLaunchKernelGGL((hash_heads_walk<C, NT, WAVES>), dim3(heads_walk_workgroups(N, sh.L, WAVES), sh.L), dim3(WAVES * 64), 0, st, r,
                           w_out, b_out, sh.E, sh.top_k, N, ids, alpha);
    };
    const bool walks = direct && heads_walk(C, sh.E, sh.L, N);
    if (walks && sh.E <= 64) walk(std::integral_constant<int, 4>(), std::integral_constant<int, 4>());
    else if (walks && sh.E <= 128) walk(std::integral_constant<int, 8>(), std::integral_constant<int, 4>());
    else if (walks) walk(std::integral_constant<int, 16>(), std::integral_constant<int, 8>());
    else if (!direct) heads_of(std::integral_constant<int, 1>(), std::false_type());
    else if (N >= 2048) heads_of(std::integral_constant<int, 2>(), std::true_type());
    else heads_of(std::integral_constant<int, 1>(), std::true_type());
    if (err) return err;
    return (int)hipGetLastError();
}

}  // namespace

int hash_static_scratch(float **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return (int)e;
    if (dev < 0 || dev >= kMaxDevices) return (int)hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));      // the current device's copy of the array
        if (e != hipSuccess) return (int)e;
        if (!p) return (int)hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = static_cast<float *>(p);
    }
    *out = g_scratch_ptr[dev];
    return 0;
}

int launch_hash_forward(const HashShape &sh, const float *params, const void *x, int32_t n_seq, int32_t seq_len,
                        int32_t *ids, float *alpha, float *ws, hipStream_t st)
{
    if (sh.C == 64) return run<64>(sh, params, x, n_seq, seq_len, ids, alpha, ws, st);
    return run<128>(sh, params, x, n_seq, seq_len, ids, alpha, ws, st);
}

}  // namespace sida
