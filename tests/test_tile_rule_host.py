"""How a layer's experts are cut into tiles and which are streamed (csrc/tile_rule.h), checked without a GPU: for layers whose
time was measured, and for the layers by which the GPU tests stand on either side of the rule's lines."""
import ctypes
import os
import subprocess

import pytest

import test_gpu_few_tokens

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2310_18859_amd", "csrc")
ALL, NONE = 2**31 - 1, 0

SOURCE = r"""
#include "tile_rule.h"
using namespace sida;
extern "C" void rule(const int *counts, int n, int d, int F, int in_waves, int *out)
{
    const TileRule r = tile_rule(counts, n, d, F, in_waves != 0);
    out[0] = r.tile_m;
    out[1] = r.few[0];
    out[2] = r.few[1];
}
extern "C" double cost(long m_tiles, long low, long high, long N, bool full) { return launch_cost({0, m_tiles, low, high}, N, full); }
extern "C" bool wide(long m_tiles, long m_tall, bool streamed, long N, long K, long slots)
{
    return gemm_tiles_wide(m_tiles, m_tall, streamed, N, K, slots);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("tile_rule")
    src, so = str(d / "rule.cpp"), str(d / "rule.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-Wall", "-I" + CSRC, "-o", so, src], check=True)
    lib = ctypes.CDLL(so)
    lib.wide.restype = ctypes.c_bool
    lib.wide.argtypes = [ctypes.c_long] * 2 + [ctypes.c_bool] + [ctypes.c_long] * 3
    lib.cost.restype = ctypes.c_double
    lib.cost.argtypes = [ctypes.c_long] * 4 + [ctypes.c_bool]
    return lib


def pick(lib, counts, d, F, waves=False):
    """tile_m, and the most tokens of a streamed expert in either GEMM."""
    out = (ctypes.c_int * 3)()
    lib.rule((ctypes.c_int * len(counts))(*counts), len(counts), d, F, int(waves), out)
    return tuple(out)


def zipf(E, T, s):
    """T tokens over E experts, by expected counts."""
    p = [1. / (i + 1) ** s for i in range(E)]
    ends = [round(T * sum(p[:i + 1]) / sum(p)) for i in range(E)]
    return [n for n in (b - a for a, b in zip([0] + ends, ends)) if n]


@pytest.mark.parametrize("counts,d,F,want", [
    ([32] * 8, 768, 3072, (64, ALL, ALL)),                              # few tiles
    (zipf(128, 512, 0.), 768, 3072, (64, ALL, ALL)),                    # hardly an expert of more than one row block
    ([20] * 128, 768, 3072, (64, 64, 64)),                              # many experts of few tokens
    ([48] * 128, 768, 3072, (64, NONE, NONE)),                          # ... of more
    ([256] * 128, 768, 3072, (128, NONE, NONE)),
    ([2048] * 8, 768, 3072, (128, NONE, NONE)),
])
def test_layers_of_one_kind_of_expert(lib, counts, d, F, want):
    assert pick(lib, counts, d, F) == want


@pytest.mark.parametrize("seed", range(40))
def test_streamed_experts_do_not_depend_on_the_order_or_the_waves(lib, seed):
    """... which would change the order of sums."""
    import random
    rng = random.Random(seed)
    E, s = rng.randint(8, 256), rng.choice((0., 0.8, 1., 1.2))
    d, F = rng.choice(((384, 1536), (512, 2048), (640, 2560), (768, 3072), (1024, 4096)))
    counts = zipf(E, int(E * 2 ** rng.uniform(2, 8)), s)
    want = pick(lib, counts, d, F)
    rng.shuffle(counts)
    assert pick(lib, counts, d, F) == want
    assert pick(lib, counts, d, F, waves=True) == (64,) + want[1:]
    assert all(f in (0, 20, 28, 36, 64, ALL) for f in want[1:])


@pytest.mark.parametrize("N", [256, 768, 1024, 3072])
def test_widths(lib, N):
    """By rounds of narrow tiles: wide above 2.4 and from above 1.5 to 2; else for long rows or tall tiles, or beside streamed
    experts."""
    for slots in (512, 256, 16):
        for m in range(1, 2 * slots):
            r = m * (N // 128) / slots
            for streamed, K, tall in ((s, K, t) for s in (False, True) for K in (N // 2, N, 4 * N) for t in (0, m // 4, m // 4 + 1, m // 2, m // 2 + 1, m)):
                part, most = K > N and 0.77 <= r <= 0.92, 2 * tall > m
                if streamed:
                    want = part or r >= 1.45
                elif r <= 1.5:
                    want = part or (K > N and most and r >= 1.45)
                elif 2 < r <= 2.4:
                    want = K > N and most if r <= 2.2 else 4 * tall > m
                else:
                    want = True
                assert lib.wide(m, tall, streamed, N, K, slots) == want, (m, tall, streamed, K, slots, r)
    assert not any(lib.wide(m, 0, s, 640, 1280, 512) for m in range(2000) for s in (False, True))   # not a multiple of 256


def launch_widths(lib, counts, d, F):
    """Whether either GEMM of a layer on the whole chip runs in wide tiles."""
    tile_m, *few = pick(lib, counts, d, F)
    out = []
    for f, N, K in ((few[0], F, d), (few[1], d, F)):
        tiles = [-(-n // tile_m) for n in counts if n > f]
        out.append(lib.wide(sum(tiles), sum(t for t in tiles if t > 1), min(counts) <= f, N, K, 512))
    return tuple(out)


@pytest.mark.parametrize("counts,d", [
    ([188] * 9, 768),                                                   # 0.84 rounds of narrow tiles, tall: 17 us, wide 20
    ([217] * 18, 384),                                                  # ... 11.8 and 12.5
    (zipf(24, 2500, 0.8), 768),                                         # 1.5 rounds: 31 and 34
    ([28] * 32, 768),                                                   # ... 28.6 and 30.6
    ([19] * 44, 768),                                                   # 2.06: 40.3 and 43.9
    ([84] * 34, 1024),                                                  # 2.13: 57.9 and 61.3
    ([81] * 37, 1024),                                                  # 2.31: 60.3 and 61.8
])
def test_first_gemms_that_narrow_tiles_take_less_time_for(lib, counts, d):
    assert launch_widths(lib, counts, d, 4 * d)[0] is False


@pytest.mark.parametrize("counts,d,want", [
    ([256] * 128, 768, (True, True)),                                   # 12 and 3 rounds of narrow tiles
    ([2048] * 8, 768, (True, True)),                                    # 6 and 1.5, of long rows
    ([1280] * 18, 768, (True, True)),                                   # 8.4 and 2.1
    ([128] * 180, 768, (True, False)),                                  # ... of experts of one tile
    ([400] * 11, 768, (False, False)),                                  # 2.06, of short rows, and 0.52
])
def test_widths_of_larger_launches(lib, counts, d, want):
    assert launch_widths(lib, counts, d, 4 * d) == want


@pytest.mark.parametrize("E,T,s,d", [(66, 1664, 1., 768), (61, 1507, 1.2, 768), (67, 2979, 1.2, 768), (64, 1111, 1.2, 768),
                                     (55, 2094, 1.2, 768), (101, 1173, 1., 512)])
def test_wide_tiles_for_part_of_the_slots_are_walked(lib, E, T, s, d):
    """Second GEMMs of 0.77 to 0.92 rounds of narrow tiles, for which wide ones take as long: walking them all takes 50 to 63
    us (768 x 3072), streaming the smallest beside the others 4 to 9 us more."""
    counts = zipf(E, T, s)
    tile_m, _, second = pick(lib, counts, d, 4 * d)
    m_tiles = sum(-(-n // tile_m) for n in counts)
    assert 0.77 * 512 <= m_tiles * (d // 128) <= 0.92 * 512 and launch_widths(lib, counts, d, 4 * d)[1]
    assert second == NONE


@pytest.mark.parametrize("E,T,s,d", [(49, 1852, 1., 640), (54, 1778, 0.8, 512), (55, 749, 1.2, 512), (89, 2149, 1.2, 384)])
def test_experts_of_up_to_64_tokens_are_streamed_where_most_slots_are_idle(lib, E, T, s, d):
    """Second GEMMs of less than 0.65 rounds of narrow tiles: with at most 36 tokens streamed they take 3 to 8 % more."""
    counts = zipf(E, T, s)
    tile_m, _, second = pick(lib, counts, d, 4 * d)
    assert 100 * sum(-(-n // tile_m) for n in counts) * (d // 128) < 65 * 512 and max(counts) > 64
    assert second == 64


@pytest.mark.parametrize("E,T,s,d", [(74, 6514, 1., 512), (46, 2542, 1., 1024), (37, 3709, 1., 1024), (49, 4219, 1.2, 768)])
def test_layers_of_larger_experts_are_walked_in_one_round(lib, E, T, s, d):
    """Second GEMMs of 0.77 to 1 round of narrow tiles: with the smallest experts streamed they take 4 to 6 % more."""
    counts = zipf(E, T, s)
    tile_m, first, second = pick(lib, counts, d, 4 * d)
    assert 0.77 * 512 <= sum(-(-n // tile_m) for n in counts) * (d // 128) <= 512
    assert second == NONE


@pytest.mark.parametrize("full", [False, True])
@pytest.mark.parametrize("N", [256, 768, 1024, 3072])
def test_cost_of_a_round(lib, N, full):
    """What a launch of walked tiles is taken to cost does not jump where their width changes inside a round, and a few
    streamed experts more add their own share at the most."""
    per = N // 128
    one = [lib.cost(m, 0, 0, N, full) for m in range(1, 512 // per + 1)]
    assert all(0.55 <= c <= 0.65 for c in one)
    for m in range(1, 6 * 512 // per):
        for low in (1, 10, 40):
            cost, more = lib.cost(m, low, 0, N, full), lib.cost(m, low + 1, 0, N, full)
            assert cost <= more <= cost + 2 * 0.9 * N / (256 * 512) + 1e-9, (m, low)


@pytest.mark.parametrize("case", range(len(test_gpu_few_tokens.CASES)))
def test_layers_of_the_gpu_test_are_cut_as_it_says(lib, case):
    """... and so are the sizes on either side of the lines of 20, 28, 36 and 64 tokens streamed and walked there."""
    name, counts, d, F, want = test_gpu_few_tokens.CASES[case]
    assert pick(lib, counts, d, F)[1:] == want
    lines = [few for few in want if few and (few < 64 or name == "lines-part")]
    assert not name.startswith("lines") or all(n in counts for few in lines for n in (few, few + 1))
