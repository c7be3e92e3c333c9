"""The work that programs built on this classifier-head library have it do, as cases to be measured.

A case is a dict of plain values.  Kinds:

  step      one training step of a head (`Head.step`): logits, input gradient and fused weight update
            over all label chunks of one batch;
  topk      top-k scoring of a batch against all labels of a head (`Head.topk`);
  eval      the same followed by the P@k numerators of the batch (`elmo_precision_hits`);
  serve     top-k without a head or a workspace (`elmo_topk_static`), as a serving loop calls it;
  adamw     one Kahan-AdamW step on BF16 parameters (`elmo_kahan_adamw`);
  quantize  FP32 -> E4M3 / BF16 conversion of a slice of weights (`elmo_quantize`).

Sizes are those of `synth.CONFIGS` and of bench.py's sweep, and generic ones between them.  Weights, inputs
and labels follow synth.py: W ~ N(0, 0.02), unit-length rows of X, Zipf label ids, a handful of positives per
sample.  A head that is scored (topk, eval, serve) has seen training: the rows of the queries' own labels
point towards the queries.
"""
from __future__ import annotations

import numpy as np
import torch

from paper_2510_11168_amd import binding as b
from paper_2510_11168_amd import synth

DEV = "cuda:0"
FMT = {"bf16": b.ELMO_BF16, "e4m3": b.ELMO_FP8_E4M3}


def _step(name, L, d, B, chunk, fmt, sr, kahan, zipf, counts, **more):
    case = dict(name=name, kind="step", L=L, d=d, B=B, chunk=chunk, fmt=fmt, sr=sr, kahan=kahan, kahan_rows=0, zipf=zipf,
                counts=counts, dx=True, loss=False, weight_decay=0.0, dropout=0.0)
    case.update(more)
    return case


def listed():
    return [
        # The smallest head of the configurations: a few launches' worth of work, latency counts.
        _step("step_tiny", 8192, 256, 64, 2048, "bf16", True, False, 1.1, "fixed5"),
        # A mid-size extreme-classification head, BF16 weights with compensation and nearest rounding.
        _step("step_mid", 131072, 768, 256, 32768, "bf16", False, True, 1.0, "lognormal5"),
        # A large head in pure BF16 with stochastic rounding, ragged in its last chunk.
        _step("step_large", 670091, 768, 512, 65536, "bf16", True, False, 1.0, "poisson4.5"),
        # The headline: three million labels in E4M3 with BF16 compensation.
        _step("step_xl", 3000000, 768, 1024, 131072, "e4m3", True, True, 1.05, "poisson7"),
        # The same head at a batch where the stream of weights and compensation is the work.
        _step("step_xl_b128", 3000000, 768, 128, 262144, "e4m3", True, True, 1.05, "poisson7"),
        # The same head at the largest batch of the sweep, where the matrix products are the work.
        _step("step_xl_b4096", 3000000, 768, 4096, 65536, "e4m3", True, True, 1.05, "poisson7"),
        # Nothing a multiple of a tile, and every option of the step at once: compensation for the head labels
        # only, weight decay, classifier dropout, the loss read out.
        _step("step_ragged", 100003, 640, 200, 30000, "e4m3", True, True, 1.05, "poisson7", kahan_rows=19968, loss=True,
              weight_decay=0.01, dropout=0.25),
        # Bulk scoring of a test set against three million labels.
        dict(name="topk_xl", kind="topk", L=3000000, d=768, B=1024, k=100, fmt="e4m3", zipf=1.05, counts="poisson7"),
        # A validation batch: top-k and its P@k numerators.
        dict(name="eval_mid", kind="eval", L=131072, d=768, B=256, k=100, fmt="bf16", zipf=1.0, counts="lognormal5"),
        # One query against a large head, as an online service asks.
        dict(name="serve_one", kind="serve", L=670091, d=768, B=1, k=10, fmt="bf16", zipf=1.0, counts="poisson4.5"),
        # The optimiser step of the encoder in front of the head, 110 M parameters.
        dict(name="adamw_110m", kind="adamw", n=110000000, state="bf16", weight_decay=0.01),
        # A slice of freshly initialised weights into the storage format.
        dict(name="quantize_slice", kind="quantize", n=65536 * 768, fmt="e4m3", sr=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["step"] * 7 + ["topk", "topk", "eval", "serve", "serve", "adamw", "quantize"])
    fmt = rng.choice(["bf16", "e4m3"])
    if kind == "adamw":
        return dict(kind=kind, n=_log_int(rng, 10000, 110000000), state=rng.choice(["bf16", "fp32"]), weight_decay=rng.choice([0.0, 0.01]))
    if kind == "quantize":
        return dict(kind=kind, n=_log_int(rng, 10000, 65536 * 768), fmt=fmt, sr=rng.random() < 0.5)
    L = _log_int(rng, 8192, 3000000 if fmt == "e4m3" else 1500000)
    d = rng.choice([768, 768, 768, 256, 384, 512, 640, 1024])
    zipf, counts = rng.choice([1.0, 1.05, 1.1]), rng.choice(["fixed5", "lognormal5", "poisson4.5", "poisson7"])
    if d == 1024:
        L = min(L, 2000000)
    if kind == "step":
        B = min(_log_int(rng, 16, 4096), int(4096 * 768 / d))
        chunk = 2048 if L < 16384 else rng.choice([c for c in (16384, 30000, 32768, 65536, 131072, 262144) if c < 2 * L])
        kahan = rng.random() < 0.5
        rows = L // 5 // 128 * 128 if kahan and rng.random() < 0.25 else 0
        return dict(kind=kind, L=L, d=d, B=B, chunk=chunk, fmt=fmt, sr=rng.random() < 0.75 or not kahan, kahan=kahan, kahan_rows=rows, zipf=zipf,
                    counts=counts, dx=rng.random() < 0.9, loss=rng.random() < 0.25, weight_decay=rng.choice([0.0, 0.0, 0.0, 0.01]),
                    dropout=rng.choice([0.0, 0.0, 0.0, 0.0, 0.25]))
    B = _log_int(rng, 1, 128 if kind == "serve" else 2048)
    return dict(kind=kind, L=L, d=d, B=B, k=rng.choice([1, 3, 5, 10, 50, 100]), fmt=fmt, zipf=zipf, counts=counts)


def _batch(case, rng):
    """One batch on the device, X as BF16 bits, and its positives as CSR."""
    X = torch.from_numpy(synth.make_x(rng, case["B"], case["d"]).view(np.int16)).to(DEV)
    indptr, indices = synth.ZipfLabels(case["L"], case["zipf"]).draw_csr(rng, case["B"], case["counts"])
    return X, indptr, indices


def _init_weights(W, fmt, gen, std=0.02, slab=1 << 26):
    """W [L, d] (storage bits) <- N(0, std) rounded by the library, slice by slice."""
    L, d = W.shape
    for l0 in range(0, L, slab // d):
        w = W[l0:l0 + slab // d]
        f = torch.randn(w.numel(), device=DEV, generator=gen) * std
        b.elmo_quantize(f, f.numel(), fmt, 0, 0, 0, 0, w)


def _teach(W, fmt, X, indptr, indices, gen, pull=0.5):
    """The rows of the batch's own labels point towards the mean of their inputs, as training leaves them."""
    order = np.argsort(indices, kind="stable")
    labels, first = np.unique(indices[order], return_index=True)
    rows = np.repeat(np.arange(len(indptr) - 1), np.diff(indptr))[order]
    mean = np.add.reduceat(X.view(torch.bfloat16).double().cpu().numpy()[rows], first, axis=0)
    mean = torch.from_numpy(pull * mean / np.linalg.norm(mean, axis=1, keepdims=True)).float().to(DEV)
    f = mean + torch.randn(mean.shape, device=DEV, generator=gen) * 0.02
    bits = torch.empty(f.shape, dtype=W.dtype, device=DEV)
    b.elmo_quantize(f, f.numel(), fmt, 0, 0, 0, 0, bits)
    W[torch.from_numpy(labels.astype(np.int64)).to(DEV)] = bits


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    rng = np.random.default_rng(seed)
    kind = case["kind"]
    s = {"case": case, "step": 0}
    if kind == "adamw":
        n, state = case["n"], torch.bfloat16 if case["state"] == "bf16" else torch.float32
        draw_n = lambda scale, dtype: (torch.randn(n, device=DEV, generator=gen) * scale).to(dtype)  # noqa: E731
        s["p"], s["g"] = draw_n(0.02, torch.bfloat16), draw_n(1e-3, torch.bfloat16)
        s["c"] = torch.zeros(n, dtype=torch.bfloat16, device=DEV)
        s["m"], s["v"] = draw_n(1e-4, state), draw_n(1e-3, torch.float32).square_().to(state)
        return s
    if kind == "quantize":
        s["src"] = torch.randn(case["n"], device=DEV, generator=gen) * 0.02
        s["dst"] = torch.empty(case["n"], dtype=torch.uint8 if case["fmt"] == "e4m3" else torch.int16, device=DEV)
        return s
    L, d, B, fmt = case["L"], case["d"], case["B"], FMT[case["fmt"]]
    X, indptr, indices = _batch(case, rng)
    s.update(X=X, indptr=torch.from_numpy(indptr).to(DEV), indices=torch.from_numpy(indices).to(DEV))
    if kind == "step":
        flags = (b.ELMO_SR if case["sr"] else 0) | (b.ELMO_KAHAN if case["kahan"] else 0)
        s["head"] = b.Head(L, d, fmt, case["chunk"], flags, B, 64 * B, device=DEV, kahan_rows=case["kahan_rows"],
                           weight_decay=case["weight_decay"], dropout_p=case["dropout"])
        _init_weights(s["head"].weights(), fmt, gen)
        s["dX"] = torch.zeros((B, d), dtype=torch.bfloat16, device=DEV) if case["dx"] else None
        s["loss"] = torch.zeros(1, dtype=torch.float32, device=DEV) if case["loss"] else None
        return s
    k = case["k"]
    if kind == "serve":
        s["W"] = torch.empty((L, d), dtype=torch.uint8 if case["fmt"] == "e4m3" else torch.int16, device=DEV)
        W = s["W"]
    else:
        s["head"] = b.Head(L, d, fmt, 131072, 0, B, 64 * B, device=DEV)
        W = s["head"].weights()
    _init_weights(W, fmt, gen)
    _teach(W, fmt, X, indptr, indices, gen)
    s["idx"] = torch.zeros((B, k), dtype=torch.int32, device=DEV)
    s["score"] = torch.zeros((B, k), dtype=torch.float32, device=DEV)
    s["hits"] = torch.zeros(k, dtype=torch.int64, device=DEV)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "step":
        head = s["head"]
        head.step(s["X"], s["indptr"], s["indices"], 0.05, 0, s["step"], s["dX"], s["loss"])
        s["step"] += 1
        return {"W": head.weights(), "comp": head.compensation(), "dX": s["dX"], "loss": s["loss"]}
    if kind == "topk":
        s["head"].topk(s["X"], case["k"], s["idx"], s["score"])
        return s["idx"], s["score"]
    if kind == "eval":
        s["head"].topk(s["X"], case["k"], s["idx"], s["score"])
        b.elmo_precision_hits(s["idx"], case["B"], case["k"], s["indptr"], s["indices"], s["hits"])
        return s["idx"], s["score"], s["hits"]
    if kind == "serve":
        b.elmo_topk_static(s["W"], case["L"], case["d"], FMT[case["fmt"]], s["X"], case["B"], case["k"], s["idx"], s["score"])
        return s["idx"], s["score"]
    if kind == "adamw":
        s["step"] += 1
        b.elmo_kahan_adamw(s["p"], s["c"], s["m"], s["v"], s["g"], case["n"], b.ELMO_BF16 if case["state"] == "bf16" else b.ELMO_FP32,
                           1e-4, 0.9, 0.999, 1e-8, case["weight_decay"], s["step"])
        return s["p"], s["c"], s["m"], s["v"]
    b.elmo_quantize(s["src"], case["n"], FMT[case["fmt"]], int(case["sr"]), 0, 0, 0, s["dst"])
    return s["dst"]


def work(case):
    kind = case["kind"]
    if kind == "adamw":
        # p, c, m, v read and written, g read
        return {"bytes": case["n"] * (10 + (8 if case["state"] == "bf16" else 16)), "flops": 24.0 * case["n"]}
    if kind == "quantize":
        return {"bytes": case["n"] * (4 + (1 if case["fmt"] == "e4m3" else 2)), "flops": 0}
    L, d, B, s_w = case["L"], case["d"], case["B"], 1 if case["fmt"] == "e4m3" else 2
    if kind == "step":
        rows = (case["kahan_rows"] or L) if case["kahan"] else 0
        products = 3 if case["dx"] else 2
        return {"bytes": L * d * 2 * s_w + rows * d * 4 + B * d * 2 * (products - 1) + 32 * B, "flops": 2.0 * products * B * L * d}
    return {"bytes": L * d * s_w + B * d * 2 + B * case["k"] * 8, "flops": 2.0 * B * L * d}


def tolerance(case):
    kind = case["kind"]
    if kind in ("adamw", "quantize"):
        return "exact"        # every operation is rounded once, by rule
    if kind == "step":
        # dX in BF16: against the FP64 oracle the two roundings differ for a few values in a thousand (1.3e-4 in norm), by one
        # BF16 spacing each (up to 2^-7 of the value).  Weights and compensation are compared bit by bit.  A weight lands on the
        # other side of a rounding boundary where FP32 sums in another order do: up to 4.7e-4 of the BF16 weights against the
        # FP64 oracle, 3e-6 of the E4M3 ones.  The compensation carries the last bits of those sums: 0.3 - 0.8 % of its patterns
        # differ over E4M3 weights and 2.6 - 4.2 % over BF16 ones.
        return {"rel": 6e-4, "max": 3e-2, "differ": 1e-2 if case["kahan"] else 2e-3}
    # FP32 sums of exact products, within 2e-7 of FP64; ids may swap where two scores tie to that precision
    return {"rel": 1e-6, "max": 1e-5, "differ": 1e-3}
