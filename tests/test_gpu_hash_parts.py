"""The hash function's products of values in bf16 parts, at the edges of what takes which tiles (2048 and 6144 tokens, rows and
columns that fill no tile), against the float64 oracle - near enough that a lost third part of a value shows: the oracle with
every weight cut to its first two parts is several times as far off as the bound."""
import numpy as np
import pytest

import paper_2310_18859_amd as sm
from oracle import hash_fn
from test_gpu_hash import make_params, run_hash
from workloads import bf16_bits_to_f32, f32_to_bf16_bits

pytestmark = pytest.mark.gpu

# Observed 0.3e-6 to 0.6e-6; sums of fp32 values in another order differ by as much.  Without third parts, all weights or
# those of the embeddings or heads alone: 8e-6 to 24e-6.
BOUND = 2e-6


def upper(v):
    return (v.view(np.uint32) & np.uint32(0xffff0000)).view(np.float32)


def without_third(v):
    first = upper(v)
    return first + upper(v - first)


def oracle_alpha(params, x, cfg, ids):
    """Probabilities that the oracle gives the experts in ids [L, N, k]."""
    n, T = x.shape[:2]
    probs = np.concatenate([hash_fn.hash_forward(params, x[s], cfg.L, cfg.E, cfg.top_k)[2] for s in range(n)], axis=1)
    return np.take_along_axis(probs, ids.astype(np.int64), axis=2)


@pytest.mark.parametrize("d,C,L,E,k,n_seq,T", [
    (64, 128, 2, 16, 1, 23, 89),          # 2047 tokens: one tile per wavefront
    (72, 128, 2, 16, 1, 16, 128),         # 2048, and a row of embeddings that ends inside a step
    (768, 128, 1, 60, 2, 89, 69),         # 6141, experts that fill no tile, layers one after the other
    (136, 64, 2, 130, 1, 48, 128),        # 6144
    (1024, 64, 1, 16, 1, 49, 127),        # 6223
    (64, 128, 1, 16, 1, 64, 33),          # as many sequences as have four workgroups each, and one more
    (64, 128, 1, 16, 1, 65, 33),
    (64, 64, 1, 16, 1, 15, 137),          # as few as have three
])
def test_parts_against_oracle(d, C, L, E, k, n_seq, T):
    rng = np.random.default_rng(d + T)
    cfg = sm.SidaHashConfig(d, C, L, E, k, T)
    params = make_params(rng, d, C, L, E)
    x_bits = f32_to_bf16_bits(rng.standard_normal((n_seq * T, d)).astype(np.float32))
    x = bf16_bits_to_f32(x_bits).reshape(n_seq, T, d)
    ids, alpha = run_hash(cfg, params, x_bits, n_seq, T)
    want = oracle_alpha(params, x, cfg, ids)
    norm = np.linalg.norm(want)
    err = float(np.linalg.norm(alpha - want) / norm)
    two = {n: without_third(v) if v.ndim == 2 else v for n, v in params.items()}
    lost = float(np.linalg.norm(oracle_alpha(two, x, cfg, ids) - want) / norm)
    print(f"relative error {err:.2e}, without the third parts {lost:.2e}", flush=True)
    assert err <= BOUND and lost > 3 * BOUND
