"""The calls whose speed counts: softmax, softmax + top-k, and the projection
ahead of them, from single-decode-step sizes to a whole training batch.

A case is a dict of plain values:

* ``op``: ``softmax`` (``softmax_fwd``), ``topk`` (``softmax_topk``), ``both``
  (one after the other on the same batch, the benchmark's step), ``values``
  (``topk``: the elements themselves), ``proj`` (logits = h . w^T) or
  ``proj_topk`` (the projection with softmax + top-k, logits never written);
* ``N`` rows of ``V`` elements of ``dtype``; ``H`` hidden size of a projection;
* ``K`` of a top-k; ``mode`` of a softmax;
* ``sigma`` of the logits, ``shift`` / ``ties``: 1% of the rows shifted by
  +1000 (overflow safety), or with the row maximum at four places.

Sizes are those of ``paper_1805_02867_amd.synth.WORKLOADS``, of the benchmark's
sweeps and of its projection comparison.  Output buffers are allocated once, as
the benchmark and a serving loop do.
"""
from __future__ import annotations

import math

import torch

import paper_1805_02867_amd as osm
from paper_1805_02867_amd import synth

# What a drawn case may cost at most: the largest batch and projection listed.
MAX_ELEMS = 4096 * 128256
MAX_FLOPS = 2.0 * 4000 * 4096 * 32000


def _rows(name, op, N, V, dtype, sigma, K=0, mode="online", shift=False, ties=False):
    return dict(name=name, op=op, N=N, V=V, dtype=dtype, sigma=sigma, K=K, mode=mode,
                shift=shift, ties=ties)


def _proj(name, op, N, H, V, K=0):
    return dict(name=name, op=op, N=N, H=H, V=V, K=K)


def listed():
    return [
        # The smallest call: a classifier head's 16 rows of 1000 scores, probabilities
        # and the five best of each.  Launch latency and the host path.
        _rows("both_16x1000_f32", "both", 16, 1000, "f32", 1.0, K=5),
        # The benchmark's step: softmax, then the five best, over a training batch of
        # 4000 rows with a 32000-word vocabulary.
        _rows("both_4000x32000_f32", "both", 4000, 32000, "f32", 2.0, K=5, shift=True),
        # Middle-sized rows of an odd length: no row but each fourth starts on a
        # 16-byte boundary.
        _rows("softmax_4000x3001_f32", "softmax", 4000, 3001, "f32", 2.0),
        # A few rows of a very large vocabulary: each row is spread over the chip.
        _rows("softmax_10x1000000_f32", "softmax", 10, 1_000_000, "f32", 3.0),
        # Output distribution of a language model's training step, 4096 tokens.
        _rows("softmax_4096x128256_bf16", "softmax", 4096, 128256, "bf16", 4.0),
        # Candidates out of short rows: a router or a 1000-class head over a batch.
        _rows("topk_4000x1000_f32_k5", "topk", 4000, 1000, "f32", 2.0, K=5, ties=True),
        # Beam candidates from few, very long rows.
        _rows("topk_10x1000000_f32_k5", "topk", 10, 1_000_000, "f32", 3.0, K=5),
        # One decode step of 64 sequences: top-50 sampling over the vocabulary.
        _rows("topk_64x128256_bf16_k50", "topk", 64, 128256, "bf16", 4.0, K=50),
        # Top-50 distillation targets of a whole training batch.
        _rows("topk_32768x128256_bf16_k50", "topk", 32768, 128256, "bf16", 4.0, K=50),
        # The vocabulary projection of one decode step of 64 sequences, straight to the
        # five best (streams the weights).
        _proj("proj_topk_64x4096x128256_k5", "proj_topk", 64, 4096, 128256, K=5),
        # Logits of a prefill chunk of 512 tokens, written out.
        _proj("proj_512x4096x128256", "proj", 512, 4096, 128256),
        # Scoring a batch of 4000 positions, straight to the five best.
        _proj("proj_topk_4000x4096x32000_k5", "proj_topk", 4000, 4096, 32000, K=5),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(["softmax", "softmax", "topk", "topk", "both", "values", "proj", "proj_topk"])
    if op.startswith("proj"):
        H = 8 * _log_int(rng, 32, 512)               # 256 .. 4096, whole 16-byte chunks
        V = _log_int(rng, 1000, 128256)
        N = _log_int(rng, 1, max(1, min(4000, int(MAX_FLOPS / (2.0 * H * V)))))
        return dict(op=op, N=N, H=H, V=V, K=rng.randint(1, 16) if op == "proj_topk" else 0)
    V = _log_int(rng, 35, 1_000_000)
    N = _log_int(rng, 1, max(1, min(32768, MAX_ELEMS // V)))
    dtype = rng.choice(["f32", "bf16"])
    mode = "online"
    if op in ("softmax", "both"):
        mode = rng.choice(["online", "online", "online", "safe", "naive", "resident"])
        held = osm.RESIDENT_MAX_VEC * (8 if dtype == "bf16" else 4)
        if mode == "resident" and V > held:
            mode = "online"
    K = 0 if op == "softmax" else min(V, rng.choice([1, 5, 5, 10, 20, 50, rng.randint(1, 64)]))
    return dict(op=op, N=N, V=V, dtype=dtype, sigma=rng.choice([1.0, 2.0, 3.0, 4.0]), K=K,
                mode=mode, shift=mode != "naive" and rng.random() < 0.3,
                ties=rng.random() < 0.3)


def _proj_inputs(case, seed):
    """Hidden vectors and weights that give logits of about N(0, 1)."""
    N, H, V = case["N"], case["H"], case["V"]
    g = torch.Generator(device="cuda").manual_seed(seed)
    h = torch.randn(N, H, device="cuda", generator=g).to(torch.bfloat16)
    w = (torch.randn(V, H, device="cuda", generator=g) / H ** 0.5).to(torch.bfloat16)
    return h, w


def _logits(case, seed):
    return synth.logits(case["N"], case["V"], sigma=case["sigma"], seed=seed, dtype=case["dtype"],
                        device="cuda", shift_frac=0.01 if case["shift"] else 0.0,
                        tie_frac=0.01 if case["ties"] else 0.0,
                        tie_copies=min(3, case["V"] - 1))


def prepare(case, seed):
    op, N, V, K = case["op"], case["N"], case["V"], case["K"]
    s = dict(op=op, K=K)
    if op.startswith("proj"):
        s["h"], s["w"] = _proj_inputs(case, seed)
    else:
        s["x"] = _logits(case, seed)
        s["mode"] = case["mode"]
    if op in ("softmax", "both"):
        s["y"] = torch.empty_like(s["x"])
    if op == "proj":
        s["y"] = torch.empty((N, V), dtype=torch.float32, device="cuda")
    if K:
        s["vals"] = torch.empty((N, K), dtype=torch.float32, device="cuda")
        s["idx"] = torch.empty((N, K), dtype=torch.int32, device="cuda")
    return s


def run(s):
    op = s["op"]
    if op == "softmax":
        return osm.softmax_fwd(s["x"], s["y"], mode=s["mode"])
    if op == "topk":
        return osm.softmax_topk(s["x"], s["K"], s["vals"], s["idx"])
    if op == "both":
        y = osm.softmax_fwd(s["x"], s["y"], mode=s["mode"])
        vals, idx = osm.softmax_topk(s["x"], s["K"], s["vals"], s["idx"])
        return y, vals, idx
    if op == "values":
        return osm.topk(s["x"], s["K"], s["vals"], s["idx"])
    if op == "proj":
        return osm.proj(s["h"], s["w"], s["y"])
    return osm.proj_softmax_topk(s["h"], s["w"], s["K"], s["vals"], s["idx"])


def work(case):
    """Each input read once and each output written once; a multiply and an add
    per product of a projection.  (Two calls on one batch each read it.)"""
    op, N, V, K = case["op"], case["N"], case["V"], case["K"]
    if op.startswith("proj"):
        H = case["H"]
        out = 4 * N * V if op == "proj" else 8 * N * K
        return {"bytes": 2 * (N + V) * H + out, "flops": 2 * N * H * V}
    es = 2 if case["dtype"] == "bf16" else 4
    reads = 2 if op == "both" else 1
    writes = 1 if op in ("softmax", "both") else 0
    return {"bytes": es * N * V * (reads + writes) + 8 * N * K, "flops": 0}


def tolerance(case):
    op = case["op"]
    if op == "values":
        return "exact"                       # copies of inputs, and their places
    if op == "proj":
        # binary32 sums of H products in another order
        return {"rel": 2e-6, "max": 2e-5}
    if op == "proj_topk":
        # the same sums; two logits closer than their rounding may change places
        return {"rel": 6e-6, "max": 6e-5, "differ": 2e-3}
    if op == "topk" or case["dtype"] == "f32":
        # exponentials and sums in binary32; the selection itself is exact
        return {"rel": 2e-6, "max": 2e-5}
    # bfloat16 outputs: a sum in another order moves a few values across a
    # rounding boundary, by 2^-8 of the value
    return {"rel": 2e-4, "max": 1e-2}


def _row_blocks(case):
    N, V = case["N"], case["V"]
    step = max(1, (1 << 28) // V)            # 2 GB of binary64 at a time
    return [(a, min(N, a + step)) for a in range(0, N, step)]


def _topk64(x, K):
    """(probabilities, None): the K largest of softmax(x) per row.  Equal
    logits give equal probabilities, so no rule for ties is needed."""
    top = torch.topk(x, K, dim=1).values
    return torch.exp(top - torch.logsumexp(x, dim=1, keepdim=True))


def exact(case, seed):
    op, K = case["op"], case["K"]
    if op.startswith("proj"):
        if 2.0 * case["N"] * case["H"] * case["V"] > 0.6e15:
            return None                      # over 20 seconds in 64 bits
        h, w = _proj_inputs(case, seed)
        h = h.double()
        N, V = case["N"], case["V"]
        logits = torch.empty((N, V), dtype=torch.float64, device="cuda")
        for a in range(0, V, 16384):
            torch.matmul(h, w[a:a + 16384].double().t(), out=logits[:, a:a + 16384])
        return logits if op == "proj" else (_topk64(logits, K), None)
    x = _logits(case, seed)
    if op == "values":
        return torch.topk(x.double(), K, dim=1).values, None
    y, vals = [], []
    for a, b in _row_blocks(case):
        x64 = x[a:b].double()
        if op in ("softmax", "both"):
            y.append(torch.softmax(x64, dim=1))
        if op in ("topk", "both"):
            vals.append(_topk64(x64, K))
    if op == "softmax":
        return torch.cat(y)
    if op == "topk":
        return torch.cat(vals), None
    return torch.cat(y), torch.cat(vals), None
