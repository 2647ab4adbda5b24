// Which calls of the hash function take the heads that keep a layer's weights and walk over tiles of tokens, with how many
// workgroups, and how far those ask ahead.  Plain integer code, without HIP, so that it can be checked without a GPU.
#pragma once
#include <cstdint>

namespace sida {

// Eight wavefronts take more than 128 experts, four fewer; a tile is four tokens per wavefront.
constexpr int heads_walk_waves(int E) { return E > 128 ? 8 : 4; }
constexpr int heads_walk_tokens(int waves) { return 4 * waves; }

// Workgroups that are resident at a time, and as many of them as each layer gets.
constexpr int heads_walk_slots(int waves) { return waves == 4 ? 3 * 256 : 256; }
constexpr int heads_walk_most(int L, int waves) { return L < heads_walk_slots(waves) ? heads_walk_slots(waves) / L : 1; }

// Workgroups of a layer, with the same number of tiles each but for the last.
inline int heads_walk_workgroups(int N, int L, int waves)
{
    const int tiles = (int)(((int64_t)N + heads_walk_tokens(waves) - 1) / heads_walk_tokens(waves));
    const int each = (tiles + heads_walk_most(L, waves) - 1) / heads_walk_most(L, waves);
    return (tiles + each - 1) / each;
}

// Bytes in front of which every load of the tokens' values ends: a workgroup asks for the tile after the next one.
inline int64_t heads_walk_bytes(int N, int L, int C, int waves)
{
    const int64_t tokens = heads_walk_tokens(waves);
    return (N + tokens - 1 + 2 * heads_walk_workgroups(N, L, waves) * tokens) * C * 4;
}

// Weights cut once pay with more work than that, us, per workgroup and walked: C = 128 128 experts, 6 layers x 4096
// tokens 11.6 and 12.1, x 6144 17.2 and 14.6; 12 layers of 64 x 2500 9.4 and 9.9, x 4096 13.5 and 11.5; 3 of 256 x 2500 9.7
// and 9.4.  C = 64 6 of 128 x 4096 7.3 and 8.0, x 5500 10.0 and 9.7; 3 of 256 x 2048 6.5 and 6.1.
// With C = 64, where cutting is half of the work it is with 128, hundreds of layers that leave more than a quarter of the
// slots without a workgroup do not (x 2048: 400 layers of 20, 400 workgroups, 91 and 111; 260 of 20, 520, 60 and 68; 200 of 40
// x 4096, 600, 92 and 93; 129 of 60, 645, 33.0 and 31.5; C = 128 400 of 20 183 and 148).
inline bool heads_walk(int C, int E, int L, int N)
{
    const int waves = heads_walk_waves(E);
    const int64_t rows = (int64_t)N * L;
    if (N < 2048 || E <= 16 || rows < (waves == 4 ? 32768 : 6144)) return false;
    if (C == 64 && 4 * heads_walk_most(L, waves) * L < 3 * heads_walk_slots(waves)) return false;
    return heads_walk_bytes(N, L, C, waves) <= INT32_MAX;      // offsets are 32-bit and signed
}

}  // namespace sida
