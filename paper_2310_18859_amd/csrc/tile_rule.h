// How the experts of a layer are cut into tiles of the grouped GEMMs, which of them are streamed, and how wide a launch's
// tiles are.  Plain integer and double arithmetic, without HIP, so that the rules can be checked without a GPU.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>

namespace sida {

constexpr int kGemmTileM = 128;   // token rows per GEMM tile of large launches
constexpr int kGemmTileSmall = 64; // ... of small launches

// Weight rows per tile of a launch over `slots` workgroup slots, where the matrix has a multiple of 256: 256 (two stripes
// per wavefront, one LDS fragment read per two MFMAs, the token rows fetched half as often) or 128, twice as many at a
// little more than half the time each.  Tiles are dealt to the workgroups in turn, so what counts is how full the rounds are that 128-row
// tiles take; and many-token experts gain more from wide tiles than experts of one tile, long rows (K > N, a second
// GEMM) more than short ones.  Time of wide over narrow of 2483 GEMMs (1127 layers of 8 to 256 experts, 300 to 32768
// tokens, Zipf 0 to 1.2, 384 x 1536 to 1024 x 4096), least, mean and most, by rounds of narrow tiles; walked launches apart
// by whether more than half of the tiles belong to experts of several (tall), and launches with streamed experts:
//               short rows                       long rows                       streamed
//               others          tall             others          tall
//   0   - 0.5                                    1.20 1.39 1.63  1.19 1.45 1.57  0.97 1.06 1.35
//   0.5 - 0.65                                   0.84 0.99 1.42  0.90 1.01 1.45  0.96 1.00 1.13
//       - 0.77  0.93 0.99 1.11  0.98 1.04 1.10   0.83 0.96 1.04  0.91 0.98 1.06  0.96 1.00 1.12
//       - 0.92  0.94 1.00 1.04  0.96 1.05 1.22   0.93 0.97 1.06  0.89 0.98 1.08  0.94 0.98 1.05
//       - 1     0.92 1.01 1.09  0.99 1.05 1.20   0.92 0.99 1.05  0.86 0.96 1.01  0.90 0.96 1.01
//       - 1.2   1.07 1.14 1.21  1.01 1.12 1.21   1.02 1.11 1.16  0.99 1.07 1.14  0.95 0.97 1.01
//       - 1.45  1.00 1.11 1.21  0.98 1.10 1.29   1.02 1.10 1.15  0.99 1.06 1.14  0.97 1.01 1.06
//       - 1.5   1.00 1.07 1.14  0.92 1.05 1.18   0.92 1.05 1.10  0.91 1.00 1.11  0.95 0.98 1.01
//       - 2     0.89 0.97 1.03  0.87 0.93 0.99   0.86 0.93 1.01  0.81 0.88 0.95  0.86 0.95 1.01
//       - 2.2   1.00 1.05 1.11  0.94 1.01 1.05   0.96 1.05 1.13  0.92 0.98 1.03  0.96 0.98 1.01
//       - 2.4   0.96 1.02 1.08  0.91 1.00 1.06   0.94 1.03 1.11  0.91 0.96 1.03  0.99 0.99 1.00
//       - 2.7   0.91 0.96 1.04  0.86 0.93 1.03   0.90 0.98 1.09  0.85 0.91 0.97  0.98 0.99 1.00
//       - 3     0.85 0.95 0.99  0.85 0.92 0.99   0.92 0.96 1.00  0.84 0.89 0.93  0.91 0.98 1.00
//   above       0.88 0.98 1.07  0.81 0.89 1.01                                   0.85 0.94 1.00
// The lines below are on average 0.6 % behind the better width of each, by whole rounds (wide from one to two and from three
// on, but for at most three quarters of the slots over mostly single tiles) 1.6 %.  With one line at 1.45 rounds and all of 0.77 to 0.92 wide, 1.0 %, small layers
// were slowed: 9 experts x 187 tokens, first GEMM 17.3 -> 20.5 us, 44 x 19 40.3 -> 43.9, 31 experts, 516 tokens of 1024 x 4096 47.6 -> 51.5.
// 0.65 to 0.77 and 0.92 to 1 are narrow throughout.
inline bool gemm_tiles_wide(int64_t m_tiles, int64_t m_tall, bool streamed, int64_t N, int64_t K, int64_t slots)
{
    if (N % 256 != 0) return false;
    const int64_t narrow = 100 * m_tiles * (N / 128);         // rounds of narrow tiles, in 100ths of `slots`
    const bool long_rows = K > N, tall = 2 * m_tall > m_tiles, part = narrow >= 77 * slots && narrow <= 92 * slots;
    if (streamed) return narrow >= 145 * slots || (long_rows && part);
    if (narrow <= 150 * slots) return long_rows && (part || (tall && narrow >= 145 * slots));
    if (narrow > 200 * slots && narrow <= 220 * slots) return long_rows && tall;
    if (narrow > 220 * slots && narrow <= 240 * slots) return 4 * m_tall > m_tiles;
    return true;
}

// How a layer's experts are cut into tiles.  A wavefront sums over K in another order where tiles are streamed, so
// `few` depends on the token counts and the experts' size alone: a layer gives the same bits in one wave as in many.
// tile_m may depend on the waves, since it changes the order of no sum.
struct TileRule {
    int32_t tile_m;                   // token rows per tile, 64 or 128
    int32_t few[2];                   // experts of at most this many tokens are streamed, in tiles of 64 rows, by either GEMM
};

// A layer whose experts of at most `few` tokens are streamed and the others walked in tiles of tile_m rows.
struct SplitWork {
    int32_t few;
    int64_t m_tiles;                  // walked tiles
    int64_t low, high;                // streamed experts of at most 32 tokens, of more
};
// What a launch takes, in rounds of 512 wide tiles: the slots' rounds of walked tiles, or all of the work if that is
// more, which streamed tiles spread over the slots that come free.  full: more than 64 tokens per expert, on average, or
// more than 32 per few-token one.  Fitted to 360 layers (8 to 256 experts, 384 x 1536
// to 1024 x 4096, 600 to 32768 tokens, Zipf 0 to 1.2), every threshold timed with either width.
inline double launch_cost(const SplitWork &l, int64_t N, bool full)
{
    const int64_t tiles = l.m_tiles * (N / 128);              // narrow ones, 0.56 of a wide one each
    const double streamed = (0.9 * (double)l.low + 2.2 * (double)l.high) * (double)N / (256. * 512.);
    const double also = streamed > 0. ? streamed + 0.15 : 0.;
    // The fit's two lines; gemm_tiles_wide() has more of them, which take 0 to 5 % off.
    const bool wide = N % 256 == 0 && (100 * tiles >= 145 * 512 || (100 * tiles >= 77 * 512 && 100 * tiles <= 92 * 512));
    if (!wide) return std::max(0.56 * (double)((tiles + 511) / 512), 0.56 * (double)tiles / 512. + also);
    const double walked = (double)tiles / 1024.;
    // Wide tiles for less than half of the slots run alone on their compute units and take little more than half of the
    // time (second GEMM of 768 x 3072, 0.77 to 0.92 rounds of narrow tiles: 50 to 63 us, a whole round 100), most where they
    // are full of tokens; the more, the more of the other slots streamed tiles take.
    const double alone = full ? 0.65 : 0.55;
    const double round = walked < 0.5 ? alone + (1. - alone) * std::min(1., streamed / (1. - walked)) : std::ceil(walked);
    return std::max(round, walked + also);
}

// Token rows per tile.  A grouped GEMM is bound by the rows its tiles pull through LDS:
// a tile of tile_m token rows and 256 weight rows costs tile_m + 256 rows per K-step whether or not
// all its token rows exist.  64-row tiles pay when most experts have at most 64 tokens, i.e. when
// halving the tile height adds few tiles: tiles(64) * 320 <= tiles(128) * 384.  (Measured on the
// Switch-base-128 shape: 64-row tiles are 8-10 % faster at 8-16 tokens per expert, even at 64, and
// 6 % slower at 128 tokens per expert.)
// Streamed (see grouped_ffn.hip) are
//  * all tiles of a layer of few tiles, where walking them leaves most compute units idle - up to 20, and up to two
//    stripes of 32 weight rows per compute unit (256 of them) in the narrower GEMM (768 x 3072, walked and streamed:
//    16 experts x 8 tokens 67 and 56 us a layer, 20 x 48 58 and 57; 32 tiles of 64 rows 56 and 67; 1024 x 4096:
//    16 x 48 77 and 71, 20 x 48 88 and 94);
//  * and of a layer of at most 10 rows per tile with hardly an expert of more than one (128 x 8: 208 and 188 us;
//    1024 x 4096: 64 x 8 180 and 172; 384 x 1536: 200 x 8 96 and 84);
//  * of a layer of many experts that all have at most 64 tokens, if those are at most 24 on average, or 32 where the
//    rounds of 512 tiles of 128 weight rows that walking them takes would be a
//    fifth empty (768 x 3072: 128 experts x 16 218 and 214 us, x 24 227 and 227, x 32 237 and 245; 48 x 28, rounds 36 %
//    empty, 106 and 94; 1024 x 4096, whole rounds: 64 x 28 192 and 198), or 16 with less than two workgroups per
//    compute unit (64 experts of 384 x 1536: x 16 39 and 39, x 24 41 and 43; 48 of 640 x 2560: 64 and 62, 67 and 69);
//    with at most one, walking leaves most of the chip idle again (48 of 256 x 1024 x 28: 22.4 and 21.7);
//  * beside larger tiles the experts of at most 20, 28, 36 or 64 tokens, by each GEMM those with which launch_cost() is least:
//    a launch of walked tiles ends when its last round does, however few tiles that has, and streamed ones fill
//    the slots that come free.
//    - Layers of at least 48 experts, at most 64 tokens on average, with a workgroup and a half of 64 weight rows per
//      compute unit among those of at most 64 tokens, which have at most 32 on average: where that is no more than
//      walking them all.  Where the narrow tiles of all experts are less than 0.65 of a round, those of at most 64 tokens: most slots are
//      idle, and streams fill them (85 second GEMMs of 384 x 1536 to 768 x 3072: with 36 tokens at the most 3.6 % more on average, up to
//      8; 49 experts, 1852 tokens of 640 x 2560 37.3 -> 39.0 us, 54, 1778 of 512 x 2048 30.2 -> 31.7).  (Those of at most 64
//      tokens beside half of the slots -> now, us, first and second GEMM: 157 experts, 640 x 2560, 7824 tokens 109 / 108 ->
//      102 / 105; 64 experts, 1111 tokens, Zipf(1.2) 52 / 56 -> 51 / 53; 67 experts, 2979 tokens 63 / 66 -> 58 / 63, the second
//      all walked, as in the layer before.)
//    - Others of at least 32 experts, of which at most half are streamed: where narrow tiles of all experts are more than one round (16
//      second GEMMs of 0.77 to 1, chosen by cost: 1.7 % more than walked on average, up to 6) and that is 8 % less than walking them all
//      (64 experts, 8192 tokens, Zipf(1.2) 87 / 86 -> 81 / 81; 128 experts, 16384 tokens, second GEMM, 2.4 rounds of narrow tiles
//      -> 0.95 of wide ones and 43 streamed experts, 153 -> 147).
//    Counting a whole round for wide tiles that are part of one chose otherwise in 1.4 % of drawn layers; 56 drawn from
//    those GEMMs take 1.9 % less this way on average, 27 of them 2 % and more, five 3 to 8 % more (second GEMMs: 55 experts,
//    1890 tokens 57.3 -> 49.8; 101 experts, 1173 tokens of 512 x 2048 43.5 -> 37.0; 58 experts, 3693 tokens 60.1 -> 65.1).
// With 128 columns the four parts of a sum are one step each, and many such tiles are better walked (x 8 tokens: 48
// experts 14 and 13 us, 200 experts 20 and 23).
// The counts stand for the whole chip, also on a stream with fewer compute units: the bits of a layer do not depend on
// the stream.
// counts: tokens of the n activated experts, in any order; in_waves: they run in more than one wave.
inline TileRule tile_rule(const int32_t *counts, int32_t n_active, int32_t d_model, int32_t d_ff, bool in_waves)
{
    int64_t t64 = 0, t128 = 0, n_few = 0, few_rows = 0, rows_all = 0;
    for (int32_t i = 0; i < n_active; ++i) {
        const int32_t n = counts[i];
        rows_all += n;
        t64 += (n + kGemmTileSmall - 1) / kGemmTileSmall;
        t128 += (n + kGemmTileM - 1) / kGemmTileM;
        if (n <= kGemmTileSmall) {
            ++n_few;
            few_rows += n;
        }
    }
    const int64_t narrow = std::min(d_model, d_ff);
    const bool worth = narrow >= 256 || n_active <= 96;
    const TileRule all{kGemmTileSmall, {INT32_MAX, INT32_MAX}};
    if (t64 <= 20 && t64 * (narrow / 32) <= 2 * 256) return all;
    if (worth && rows_all <= 10 * t64 && 8 * t64 <= 9 * n_active) return all;
    // A layer that is cut into waves launches a few experts at a time: small launches, hidden
    // behind the copies; 64-row tiles give them more (and deeper-fetching) tiles.
    const int32_t by_counts = 5 * t64 <= 6 * t128 ? kGemmTileSmall : kGemmTileM;
    const int32_t tile_m = in_waves ? kGemmTileSmall : by_counts;
    const int64_t wgs = n_few * (narrow / 64);                // of the narrower GEMM
    const bool alone = n_few == n_active;
    const auto rounds = [&](int64_t n) {                      // of 512 tiles, in shares of the tiles there are
        const int64_t t = n_few * (n / 128);
        return (double)((t + 511) / 512 * 512) / (double)t;
    };
    int64_t most = wgs >= 384 ? 32 : 0;                       // tokens of a streamed expert, on average
    if (alone) most = wgs <= 256 ? 32 : wgs < 512 ? 16 : rounds(d_model) + rounds(d_ff) > 2.5 ? 32 : 24;
    const bool stream = worth && n_active >= 48 && few_rows <= most * n_few && rows_all <= 64 * (int64_t)n_active;
    if (alone) return TileRule{tile_m, {stream ? kGemmTileSmall : 0, stream ? kGemmTileSmall : 0}};
    if (!stream && (narrow < 384 || n_active < 32)) return TileRule{tile_m, {0, 0}};
    SplitWork work[4] = {{0}, {20}, {28}, {36}};              // tiles of one wave: the choice is the layer's
    const int shift = by_counts == kGemmTileSmall ? 6 : 7;
    for (int32_t i = 0; i < n_active; ++i) {
        const int32_t n = counts[i], n_t = (n + by_counts - 1) >> shift;
        for (SplitWork &l : work) {
            if (n <= l.few) ++(n <= 32 ? l.low : l.high);
            else l.m_tiles += n_t;
        }
    }
    const auto choose = [&](int64_t N) {
        const int64_t tiles = work[0].m_tiles * (N / 128);
        if (stream && 100 * tiles < 65 * 512) return (int32_t)kGemmTileSmall;
        if (!stream && tiles <= 512) return 0;
        double least = launch_cost(work[0], N, !stream);
        int32_t few = 0;
        if (!stream) least *= 0.92;
        for (int i = 1; i < 4; ++i) {
            if (!stream && 2 * (work[i].low + work[i].high) > n_active) break;
            const double cost = launch_cost(work[i], N, !stream);
            if (stream ? cost <= least : cost < least) {
                least = cost;
                few = work[i].few;
            }
        }
        return few;
    };
    return TileRule{tile_m, {choose(d_ff), choose(d_model)}};
}

}  // namespace sida
