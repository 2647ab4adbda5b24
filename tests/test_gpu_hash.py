"""GPU parity of the hash function (Section 3.4.2) against its float64 oracle: scaling factors
within a tolerance; expert ids as a valid choice (the k most probable experts by the oracle's own
probabilities, up to that tolerance at near-ties); then the predicted table drives a MoE layer."""
import numpy as np
import pytest
import torch

import oracle
import paper_2310_18859_amd as sm
from gpu_util import assert_close, bf16_tensor_to_f32, make_runner, say
from oracle import hash_fn
from workloads import Workload, bf16_bits_to_f32, f32_to_bf16_bits

pytestmark = pytest.mark.gpu

ALPHA_TOL = 2e-4        # absolute, on probabilities; fp32 network of depth ~ 2 T + 6 against float64


def make_params(rng, d, C, L, E):
    p = {}
    for name, shape in hash_fn.param_shapes(d, C, L, E):
        fan_in = shape[1] if len(shape) == 2 else 1
        scale = 1.5 / np.sqrt(fan_in) if len(shape) == 2 else 0.1
        p[name] = (rng.standard_normal(shape) * scale).astype(np.float32)
    return p


def run_hash(cfg, params, x_bits, n_seq, T):
    dev = torch.device("cuda:0")
    flat = np.concatenate([params[n].reshape(-1) for n, _ in hash_fn.param_shapes(cfg.d_model, cfg.C, cfg.L, cfg.E)])
    assert flat.size == sm.hash_param_count(cfg)
    pd = torch.from_numpy(flat).to(dev)
    xd = torch.from_numpy(x_bits).to(dev)
    N = n_seq * T
    ids = torch.full((cfg.L, N, cfg.top_k), -1, dtype=torch.int32, device=dev)
    alpha = torch.zeros((cfg.L, N, cfg.top_k), dtype=torch.float32, device=dev)
    ws = torch.zeros(sm.hash_workspace_bytes(cfg, N), dtype=torch.uint8, device=dev)
    torch.cuda.synchronize()
    sm.hash_forward(cfg, pd, xd, n_seq, T, ids, alpha, ws, None)
    torch.cuda.synchronize()
    return ids.cpu().numpy(), alpha.cpu().numpy()


@pytest.mark.parametrize("d,C,L,E,k,n_seq,T", [
    (64, 64, 2, 8, 1, 1, 1),
    (64, 64, 3, 5, 2, 2, 17),
    (256, 128, 2, 16, 3, 3, 70),
    (768, 128, 6, 128, 1, 2, 128),
    (768, 128, 6, 128, 3, 1, 200),
    # some thousand tokens, ragged; with wide embeddings (d of 2056 and 6400), and with many logits per token
    (256, 128, 2, 16, 1, 33, 125),
    (64, 64, 2, 8, 2, 9, 115),
    (2056, 64, 1, 4, 1, 33, 125),
    (6400, 64, 1, 4, 1, 9, 115),
    (64, 64, 9, 256, 2, 33, 125),
    (64, 64, 30, 256, 1, 9, 115),
])
def test_hash_forward_against_oracle(d, C, L, E, k, n_seq, T):
    say(f"hash function d={d} C={C} L={L} E={E} k={k} sequences={n_seq} x {T}")
    rng = np.random.default_rng(d + C + T)
    cfg = sm.SidaHashConfig(d, C, L, E, k, max(T, 1))
    params = make_params(rng, d, C, L, E)
    x_bits = f32_to_bf16_bits(rng.standard_normal((n_seq * T, d)).astype(np.float32))
    ids, alpha = run_hash(cfg, params, x_bits, n_seq, T)
    x = bf16_bits_to_f32(x_bits)
    worst = 0.0
    for b in range(n_seq):
        want_ids, want_alpha, probs = hash_fn.hash_forward(params, x[b * T:(b + 1) * T], L, E, k)
        got_ids, got_alpha = ids[:, b * T:(b + 1) * T], alpha[:, b * T:(b + 1) * T]
        assert got_ids.min() >= 0 and got_ids.max() < E
        worst = max(worst, float(np.abs(got_alpha - want_alpha).max()))
        for l in range(L):
            for t in range(T):
                chosen = got_ids[l, t].tolist()
                assert len(set(chosen)) == k                                   # k different experts
                # a valid choice: each chosen expert is as probable as the oracle's k-th, up to the tolerance
                assert probs[l, t, chosen].min() >= want_alpha[l, t, k - 1] - ALPHA_TOL
                np.testing.assert_allclose(got_alpha[l, t], probs[l, t, chosen], atol=ALPHA_TOL)
        exact = float((got_ids == want_ids).mean())
        assert exact > 0.97, exact                                             # near-ties are rare
    assert worst <= ALPHA_TOL, worst
    say(f"  max |alpha - oracle| {worst:.2e}")


@pytest.mark.parametrize("d,C,L,E,k,n_seq,T", [
    # around the 8 time steps that the two LSTM layers hand over at a time
    (64, 128, 1, 4, 1, 2, 7),
    (64, 64, 1, 4, 1, 1, 8),
    (64, 128, 1, 4, 1, 1, 9),
    (64, 128, 1, 4, 1, 1, 12),
    # the most sequences whose layers run side by side, and one more
    (64, 64, 1, 4, 1, 85, 11),
    (64, 64, 1, 4, 1, 86, 11),
    # layer after layer: whole chunks in a row at both widths, with a partial one at the end and without
    (64, 128, 1, 4, 1, 86, 27),
    (64, 128, 1, 4, 1, 96, 40),
    (64, 64, 1, 4, 1, 86, 29),
    (64, 64, 1, 4, 1, 96, 40),
    # d_model with a remainder of 8 / 24 / 40 over a stage of the dense stage's operands; less than one stage
    (8, 64, 1, 4, 1, 1, 3),
    (200, 128, 1, 4, 1, 1, 20),
    (1048, 128, 1, 4, 1, 1, 20),
    # dense tiles by batch size: below and from 2048 tokens, from 6144
    (72, 128, 2, 20, 2, 23, 89),
    (72, 128, 2, 20, 2, 32, 64),
    (72, 64, 2, 20, 2, 64, 96),
    # tiles of 16 experts: one, four, eight and sixteen, full and partly filled
    (64, 64, 3, 16, 3, 1, 40),
    (64, 128, 3, 17, 3, 1, 40),
    (64, 64, 2, 65, 1, 1, 40),
    (64, 128, 2, 129, 1, 1, 40),
    (64, 128, 1, 256, 8, 1, 40),
    # attention: more scores than a row's registers hold, 8 queries per workgroup, the longest sequence
    (64, 64, 1, 4, 1, 1, 385),
    (64, 64, 1, 4, 1, 1, 2301),
    (64, 128, 1, 4, 1, 1, 4096),
])
def test_hash_forward_at_the_edges_of_tiles_and_chunks(d, C, L, E, k, n_seq, T):
    test_hash_forward_against_oracle(d, C, L, E, k, n_seq, T)


def assert_agrees(got_ids, got_alpha, probs, k):
    """ids [L, t, k] and alpha [L, t, k] are a valid choice by the oracle's probabilities [L, t, E]."""
    chosen = np.take_along_axis(probs, got_ids.astype(np.int64), axis=2)
    np.testing.assert_allclose(got_alpha, chosen, atol=ALPHA_TOL)
    assert (chosen.min(axis=2) >= np.sort(probs, axis=2)[:, :, -k] - ALPHA_TOL).all()


@pytest.mark.parametrize("n_seq,T,bad", [
    (1, 40, 37), (2, 100, 99), (1, 100, 65), (1, 500, 470),
    # products in parts: gates in the recurrence, in front of it, and layer after layer; larger tiles of embeddings
    (16, 128, 77), (70, 31, 12), (90, 70, 33),
])
def test_a_token_that_is_not_a_number_leaves_earlier_tokens_as_they_are(n_seq, T, bad):
    """A NaN embedding at token t makes the LSTM states from t on NaN; their scores are NaN, their attention weights
    0: tokens before t are those of the sequence cut off at t; other sequences do not change at all."""
    say(f"hash function: NaN at token {bad} of {n_seq} x {T}")
    d, C, L, E, k = 64, 128, 2, 20, 2
    rng = np.random.default_rng(T + bad)
    cfg = sm.SidaHashConfig(d, C, L, E, k, T)
    params = make_params(rng, d, C, L, E)
    x_bits = f32_to_bf16_bits(rng.standard_normal((n_seq * T, d)).astype(np.float32))
    clean_ids, clean_alpha = run_hash(cfg, params, x_bits, n_seq, T)
    broken = x_bits.copy()
    broken[bad, 3] = 0x7FC0
    ids, alpha = run_hash(cfg, params, broken, n_seq, T)
    _, _, probs = hash_fn.hash_forward(params, bf16_bits_to_f32(x_bits[:bad]), L, E, k)
    assert_agrees(ids[:, :bad], alpha[:, :bad], probs, k)
    assert np.isnan(alpha[:, bad]).all()
    # behind it no score is left: the residual, the token's own compressed embedding, goes to the heads alone
    c0 = bf16_bits_to_f32(x_bits[bad + 1:T]).astype(np.float64) @ params["w_in"].T + params["b_in"]
    e = np.exp((c0 @ params["w_out"].T + params["b_out"]).reshape(-1, L, E).transpose(1, 0, 2))
    assert_agrees(ids[:, bad + 1:T], alpha[:, bad + 1:T], e / e.sum(axis=2, keepdims=True), k)
    assert np.array_equal(ids[:, T:], clean_ids[:, T:]) and np.array_equal(alpha[:, T:], clean_alpha[:, T:])


@pytest.mark.parametrize("x_off,p_off", [(2, 0), (8, 0), (0, 4), (14, 12)])
@pytest.mark.parametrize("d,C,L,E,k,n_seq,T", [
    (200, 128, 2, 12, 2, 2, 21),          # every number of expert tiles, both widths, ragged rows and columns
    (64, 64, 2, 33, 1, 1, 40),
    (64, 128, 2, 70, 1, 1, 9),
    (72, 64, 1, 250, 3, 1, 17),
    (64, 128, 1, 20, 1, 32, 64),          # as many tokens as take larger tiles when they are aligned
])
def test_hash_forward_off_a_16_byte_boundary(d, C, L, E, k, n_seq, T, x_off, p_off):
    """Embeddings at the address of any bf16 value, parameters at that of any float (a slice of a larger tensor)."""
    say(f"hash function d={d} C={C} E={E} {n_seq} x {T}, x {x_off} and parameters {p_off} bytes off")
    dev, N = torch.device("cuda:0"), n_seq * T
    rng = np.random.default_rng(d + E)
    cfg = sm.SidaHashConfig(d, C, L, E, k, T)
    params = make_params(rng, d, C, L, E)
    flat = np.concatenate([params[n].reshape(-1) for n, _ in hash_fn.param_shapes(d, C, L, E)])
    x_bits = f32_to_bf16_bits(rng.standard_normal((N, d)).astype(np.float32))
    pd = torch.zeros(flat.size + 8, device=dev)[p_off // 4:][:flat.size]
    pd.copy_(torch.from_numpy(flat))
    xd = torch.zeros(N * d + 8, dtype=torch.int16, device=dev)[x_off // 2:][:N * d]
    xd.copy_(torch.from_numpy(x_bits.reshape(-1).view(np.int16)))
    assert xd.data_ptr() % 16 == x_off and pd.data_ptr() % 16 == p_off
    ids = torch.full((L, N, k), -1, dtype=torch.int32, device=dev)
    alpha = torch.zeros((L, N, k), device=dev)
    ws = torch.zeros(sm.hash_workspace_bytes(cfg, N), dtype=torch.uint8, device=dev)
    torch.cuda.synchronize()
    sm.hash_forward(cfg, pd, xd, n_seq, T, ids, alpha, ws, None)
    torch.cuda.synchronize()
    ids, alpha, x = ids.cpu().numpy(), alpha.cpu().numpy(), bf16_bits_to_f32(x_bits)
    for b in range(n_seq):
        at = slice(b * T, (b + 1) * T)
        assert_agrees(ids[:, at], alpha[:, at], hash_fn.hash_forward(params, x[at], L, E, k)[2], k)


def test_predicted_table_drives_the_layer():
    """Hash-building side to inference side: the predicted ids / alpha of layer l (top-2) are planned
    and run through the MoE layer, and the result equals the oracle's layer on the same table."""
    d, C, L, E, k, T = 128, 64, 2, 6, 2, 50
    rng = np.random.default_rng(77)
    cfg = sm.SidaHashConfig(d, C, L, E, k, T)
    params = make_params(rng, d, C, L, E)
    x_bits = f32_to_bf16_bits(rng.standard_normal((T, d)).astype(np.float32))
    ids, alpha = run_hash(cfg, params, x_bits, 1, T)
    wl = Workload(500, "hash-to-layer", L, E, d, 256, T * k, None, 4, 2)
    r = make_runner(wl)
    r.ctx.set_top_k(k)
    hw = r.host_weights.numpy()
    for l in range(L):
        plan = r.ctx.moe_plan(l, np.ascontiguousarray(ids[l].reshape(-1)))
        xd, idd, ad, yd = r.to_device(x_bits, ids[l].reshape(-1), alpha[l].reshape(-1))
        r.ctx.moe_layer_forward(plan, xd, idd, ad, yd, r.workspace, r.compute, r.copy)
        r.sync()
        ref = oracle.moe_forward_topk(x_bits, ids[l], alpha[l], [hw[l * E + e] for e in range(E)], d, 256)
        assert_close(bf16_tensor_to_f32(yd), ref, f"layer {l}")
    r.close()


def test_hash_argument_errors():
    dev = torch.device("cuda:0")
    t = torch.zeros(1 << 16, dtype=torch.uint8, device=dev)
    for bad in (sm.SidaHashConfig(64, 96, 1, 4, 1, 8), sm.SidaHashConfig(64, 64, 1, 300, 1, 8),
                sm.SidaHashConfig(64, 64, 1, 4, 5, 8)):
        assert sm.hash_param_count(bad) == 0
        with pytest.raises(sm.SidaError):
            sm.hash_forward(bad, t, t, 1, 4, t, t, t, None)
    assert sm.hash_param_count(sm.SidaHashConfig(68, 64, 1, 4, 1, 8)) == 0          # d_model not a multiple of 8
    ok = sm.SidaHashConfig(64, 64, 1, 4, 1, 8)
    with pytest.raises(sm.SidaError):                     # sequence longer than configured
        sm.hash_forward(ok, t, t, 1, 9, t, t, t, None)
    small = torch.zeros(256, dtype=torch.uint8, device=dev)
    with pytest.raises(sm.SidaError) as e:                # workspace too small
        sm.hash_forward(ok, t, t, 2, 8, t, t, small, None)
    assert e.value.code == -2
