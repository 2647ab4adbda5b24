"""Performance cases: what a user of this package has it do, through its public entry points.

A serving process holds one model and takes batch after batch.  Three kinds of work:

  moe     a batch through L consecutive MoE layers with every expert resident in the slot pool:
          plan on the host, then sort, grouped expert FFN and gate-weighted combine per layer
          (``MoERunner.plan_all`` and ``MoERunner.run``)
  stream  the same with a pool smaller than the model, so that experts come from pinned host memory
          on every pass
  serve   a burst of small batches through the hash-table queue (``push_table``, ``serve_next``) with
          part of the experts resident and a replacement policy
  hash    the predictor that fills the hash table (``hash_forward``)

The model (weights, expert popularity) depends on the case alone and is loaded once, as in a server;
activations, expert ids and gate values come from the seed.  Shapes are those of ``workloads`` and
``bench.py``; activations N(0, 1), expert weights N(0, 0.02), gates U(0.1, 1), ids Zipf distributed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2310_18859_amd.binding import SidaHashConfig, hash_forward, hash_param_count, hash_workspace_bytes
from paper_2310_18859_amd.runner import MoERunner

BASE, LARGE = (768, 3072), (1024, 4096)          # (d_model, d_ff) of Switch-base and Switch-large
BURST = 8                                        # batches that a serve pass pushes and serves

# Most work of a drawn case: that of the Switch-base-128 layers listed below.
MAX_FLOPS = 6 * 16384 * 4.0 * 768 * 3072
MAX_WEIGHTS = 6 * 128 * 4 * 768 * 3072


def _moe(name, L, E, dims, T, k=1, zipf=1.0):
    return {"name": name, "kind": "moe", "L": L, "E": E, "d": dims[0], "F": dims[1], "T": T, "k": k, "zipf": zipf}


def _hash(name, n_seq, seq_len, C=128, d=768, L=6, E=128, k=1):
    return {"name": name, "kind": "hash", "n_seq": n_seq, "seq_len": seq_len, "C": C, "d": d, "L": L, "E": E, "k": k}


def listed():
    return [
        # The table of one 128-token sentence: the latency ahead of every first token of a request.
        _hash("hash-1x128", 1, 128),
        # A few paragraphs of a reading-comprehension set (200 to 500 tokens), three experts per token.
        _hash("hash-8x333-top3", 8, 333, k=3),
        # A full batch of sentences.
        _hash("hash-64x128", 64, 128),
        # One layer of eight experts and 256 tokens: the smallest layer call, all launch latency.
        _moe("layer-8-T256", 1, 8, BASE, 256, zipf=0.0),
        # One or two sentences per batch with everything resident: a few tokens for each activated expert.
        _moe("base-128-T128", 6, 128, BASE, 128),
        # An odd, middling batch, many experts with one partly filled tile.
        _moe("base-64-T1111", 6, 64, BASE, 1111, zipf=1.2),
        # 64 sequences of 128 tokens, strongly skewed.
        _moe("base-64-T8192", 6, 64, BASE, 8192, zipf=1.2),
        # The benchmark's shape with every expert resident.
        _moe("base-128-T16384", 6, 128, BASE, 16384),
        # The larger model's layers with the largest batch: matrix-product bound.
        _moe("large-128-T32768", 2, 128, LARGE, 32768, zipf=1.2),
        # Three experts per token: separate combine, 5461 tokens.
        _moe("base-128-top3", 6, 128, BASE, 16383, k=3),
        # The benchmark's default: a pool of 32 experts, everything else streams from host memory.
        {"name": "stream-base-128", "kind": "stream", "L": 6, "E": 128, "d": 768, "F": 3072, "T": 16384, "k": 1,
         "zipf": 1.0, "S": 32, "W": 16},
        # Algorithm 1 on single sentences with half of the experts resident and the queue as the known future.
        {"name": "serve-half-pool", "kind": "serve", "L": 6, "E": 128, "d": 768, "F": 3072, "T": 128, "k": 1,
         "zipf": 1.0, "S": 384, "W": 128, "policy": "belady", "lookahead": 8},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choices(("moe", "hash", "stream", "serve"), (6, 3, 1, 1))[0]
    if kind == "hash":
        seq_len = _log_int(rng, 16, 512)
        return {"kind": "hash", "n_seq": _log_int(rng, 1, min(96, 8192 // seq_len)), "seq_len": seq_len,
                "C": rng.choice((64, 128, 128)), "d": rng.choice((512, 768, 768, 1024)), "L": rng.choice((3, 6, 6, 12)),
                "E": rng.choice((8, 64, 128, 256)), "k": rng.choice((1, 1, 2, 3))}
    d, F = rng.choice((BASE, BASE, BASE, LARGE, LARGE, (512, 2048), (640, 2560), (384, 1536)))
    bytes_per_expert = 4 * d * F
    zipf = rng.choice((0.0, 0.8, 1.0, 1.2))
    if kind == "serve":
        E = _log_int(rng, 32, 128)
        L = max(1, min(6, MAX_WEIGHTS // (E * bytes_per_expert)))
        S = int(L * E * rng.uniform(0.3, 0.9))
        return {"kind": "serve", "L": L, "E": E, "d": d, "F": F, "T": _log_int(rng, 24, 256), "k": 1, "zipf": zipf,
                "S": max(S, E), "W": min(E, max(S, E)), "policy": rng.choice(("fifo", "lru", "belady")), "lookahead": 8}
    if kind == "stream":
        E = _log_int(rng, 16, 128)
        L = rng.randint(1, max(1, min(6, MAX_WEIGHTS // (E * bytes_per_expert))))
        S = max(4, int(E * rng.uniform(0.2, 0.6)))
        return {"kind": "stream", "L": L, "E": E, "d": d, "F": F, "T": _log_int(rng, 256, 16384), "k": 1, "zipf": zipf,
                "S": S, "W": max(1, S // 2)}
    E = _log_int(rng, 8, 256)
    k = rng.choice((1, 1, 1, 2, 3))
    T = max(k, _log_int(rng, 16, 32768) // k * k)
    most = min(6, MAX_WEIGHTS // (E * bytes_per_expert), int(MAX_FLOPS // (4.0 * d * F * T)))
    return {"kind": "moe", "L": rng.randint(1, max(1, most)), "E": E, "d": d, "F": F, "T": T, "k": k, "zipf": zipf}


# ---- the model a server keeps -------------------------------------------------------------------
class _Model:
    """Runner, expert weights in pinned host memory and the experts' popularity; every expert loaded
    where the pool holds them all."""

    def __init__(self, case):
        L, E, d, F = case["L"], case["E"], case["d"], case["F"]
        resident = case["kind"] == "moe"
        S, W = (L * E, E) if resident else (case["S"], case["W"])
        r = self.runner = MoERunner(L, E, d, F, S, W, case["T"])
        g = torch.Generator(device="cuda").manual_seed(L * 1_000_003 + E * 1009 + d)
        r.alloc_host_weights()
        w = r.host_weights.view(torch.bfloat16)
        for key in range(0, L * E, 16):          # in pieces: the model may be several GB
            part = w[key:key + 16]
            part.copy_(torch.randn(part.shape, generator=g, device="cuda", dtype=torch.bfloat16) * 0.02)
        p = np.arange(1, E + 1, dtype=np.float64) ** -float(case["zipf"])
        self.cdf = torch.from_numpy(np.cumsum(p / p.sum())).cuda()
        self.rank_to_expert = [torch.randperm(E, generator=g, device="cuda") for _ in range(L)]
        r.ctx.set_top_k(case["k"])
        if case["kind"] == "serve":
            r.ctx.set_policy(case["policy"], case["lookahead"])
        torch.cuda.synchronize()
        if resident:
            self._load_all(case)

    def _load_all(self, case):
        r, k = self.runner, case["k"]
        per = case["T"] // k * k
        for e0 in range(0, case["E"], per):
            ids = np.arange(e0, e0 + per, dtype=np.int32) % case["E"]
            x = torch.zeros((per // k, case["d"]), dtype=torch.bfloat16, device="cuda")
            a = torch.zeros(per, device="cuda")
            i = torch.from_numpy(ids).cuda()
            y = torch.empty_like(x)
            torch.cuda.synchronize()
            n = case["L"]
            r.run(r.plan_all([ids] * n), [x] * n, [i] * n, [a] * n, [y] * n)
            r.sync()

    def ids(self, layer, T, g):
        u = torch.rand(T, generator=g, device="cuda", dtype=torch.float64)
        rank = torch.searchsorted(self.cdf, u).clamp_(max=len(self.rank_to_expert[layer]) - 1)
        return self.rank_to_expert[layer][rank].to(torch.int32)


_loaded: list = [None, None]                     # (key, _Model) of the model in memory: one at a time


def _model(case):
    key = tuple(sorted((k, v) for k, v in case.items() if k != "name"))
    if _loaded[0] != key:
        if _loaded[1] is not None:
            _loaded[1].runner.close()
        _loaded[:] = [None, None]
        torch.cuda.empty_cache()
        _loaded[:] = [key, _Model(case)]
    return _loaded[1]


# ---- one batch ----------------------------------------------------------------------------------
def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 17)
    if case["kind"] == "hash":
        return _prepare_hash(case, g)
    m = _model(case)
    L, T, k, d = case["L"], case["T"], case["k"], case["d"]
    batches = BURST if case["kind"] == "serve" else 1
    state = {"case": case, "runner": m.runner, "batches": []}
    for _ in range(batches):
        ids = [m.ids(l, T, g) for l in range(L)]
        y = torch.empty((L, T // k, d), dtype=torch.bfloat16, device="cuda")
        state["batches"].append({
            "x": [torch.randn((T // k, d), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(L)],
            "ids": ids,
            "alpha": [torch.rand(T, generator=g, device="cuda") * 0.9 + 0.1 for _ in range(L)],
            "y": y, "y_layers": [y[l] for l in range(L)],
            "table": np.ascontiguousarray(torch.stack(ids).cpu().numpy()),   # the hash table, host side
        })
    torch.cuda.synchronize()
    return state


def _prepare_hash(case, g):
    cfg = SidaHashConfig(case["d"], case["C"], case["L"], case["E"], case["k"], case["seq_len"])
    C, LE = case["C"], case["L"] * case["E"]

    def uniform(bound, *shape):
        return (torch.rand(shape, generator=g, device="cuda") * 2 - 1) * bound

    # layers scaled as they are initialised for training (uniform in +-1/sqrt(fan in)); the heads eight
    # times as large, so that their probabilities are as peaked as a trained predictor's
    parts = [uniform(case["d"] ** -0.5, C * case["d"] + C)]
    parts += [uniform(C ** -0.5, 8 * C * C + 8 * C) for _ in range(2)]
    parts += [uniform(8 * C ** -0.5, LE * C), uniform(C ** -0.5, LE)]
    params = torch.cat(parts)
    assert params.numel() == hash_param_count(cfg)
    n = case["n_seq"] * case["seq_len"]
    return {
        "case": case, "cfg": cfg, "params": params,
        "x": torch.randn((n, case["d"]), generator=g, device="cuda", dtype=torch.bfloat16),
        "ids": torch.empty((case["L"], n, case["k"]), dtype=torch.int32, device="cuda"),
        "alpha": torch.empty((case["L"], n, case["k"]), dtype=torch.float32, device="cuda"),
        "ws": torch.empty(hash_workspace_bytes(cfg, n), dtype=torch.uint8, device="cuda"),
    }


def run(state):
    case = state["case"]
    if case["kind"] == "hash":
        hash_forward(state["cfg"], state["params"], state["x"], case["n_seq"], case["seq_len"], state["ids"],
                     state["alpha"], state["ws"], torch.cuda.current_stream())
        return {"ids": state["ids"], "alpha": state["alpha"]}
    r, batches = state["runner"], state["batches"]
    if case["kind"] == "serve":
        for tag, b in enumerate(batches):        # the hash-building side is ahead
            r.push_table(tag, b["table"])

        def lookup(tag):
            b = batches[tag]
            return b["x"], b["ids"], b["alpha"], b["y_layers"]

        for _ in batches:
            r.serve_next(lookup)
        return [b["y"] for b in batches]
    b = batches[0]
    plans = r.plan_all(b["table"])
    r.run(plans, b["x"], b["ids"], b["alpha"], b["y_layers"])
    return b["y"]


# ---- what a pass cannot do without --------------------------------------------------------------
def _active(case):
    """Expected experts with tokens in one layer of one batch."""
    p = np.arange(1, case["E"] + 1, dtype=np.float64) ** -float(case["zipf"])
    return float((1.0 - (1.0 - p / p.sum()) ** case["T"]).sum())


def work(case):
    if case["kind"] == "hash":
        n, C, d, LE = case["n_seq"] * case["seq_len"], case["C"], case["d"], case["L"] * case["E"]
        params = C * d + C + 2 * (8 * C * C + 8 * C) + LE * C + LE
        return {"bytes": 4.0 * params + n * (2.0 * d + 8.0 * case["L"] * case["k"]),
                "flops": n * (2.0 * C * d + 32.0 * C * C + 4.0 * C * case["seq_len"] + 2.0 * C * LE)}
    n = (BURST if case["kind"] == "serve" else 1) * case["L"]
    T, d, F = case["T"], case["d"], case["F"]
    # per layer: activated experts once, a row in and a row out per token, id and gate per (token, expert)
    return {"bytes": n * (_active(case) * 4.0 * d * F + T // case["k"] * 4.0 * d + 8.0 * T),
            "flops": n * 4.0 * d * F * T}


def tolerance(case):
    if case["kind"] == "hash":
        # fp32 sums through a recurrence and a SoftMax; an id may change where two logits nearly tie
        return {"rel": 2e-5, "max": 2e-3, "differ": 1e-3}
    # bf16 inputs, hidden values and results, fp32 sums
    return {"rel": 1e-2, "max": 0.1}
