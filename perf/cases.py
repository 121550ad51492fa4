"""The work that users of libtng have it do, as measurable cases: encode + decode of worker gradients, and whole
iterations (tng_step) of every problem kind, from launch-bound sizes to the largest workloads of bench.py.

A case is a dict of plain values.  kind:
  "codec"       tng_normalize_encode + tng_decode_aggregate over gradients that are in device memory
  "external"    tng_step on gradients that the caller computed (TNG_PROB_EXTERNAL)
  "dense"       tng_step, dense logistic regression
  "csr"         tng_step, sparse logistic regression
  "rosenbrock"  tng_step, chain Rosenbrock function with Gaussian gradient noise

Every pass is one iteration with its own iteration number, as in a training loop: the iterate, the reference and the
draws differ from pass to pass.
"""
import math

import torch

from paper_1901_08227_amd import binding as B
from paper_1901_08227_amd import synth

DEVICE = "cuda:0"
NORMS = {"none": B.NORM_NONE, "sub": B.NORM_SUB, "quot": B.NORM_QUOT, "comb": B.NORM_COMB, "mean": B.NORM_MEAN}
SCALES = {"max": B.SCALE_MAX, "l2": B.SCALE_L2}
PROBLEMS = {"codec": B.PROB_EXTERNAL, "external": B.PROB_EXTERNAL, "dense": B.PROB_LOGREG_DENSE,
            "csr": B.PROB_LOGREG_CSR, "rosenbrock": B.PROB_ROSENBROCK}


def listed():
    return [
        # the smallest training run of the benchmark: every iteration is a few launches over 1 MB of rows
        dict(name="dense_tiny", kind="dense", d=1000, M=4, rows=2000, batch=64, bits=2, norm="sub", period=1, l2=0.0),
        # an ordinary dense model whose dimension is a multiple of nothing, regularised, 4-bit codes
        dict(name="dense_ragged", kind="dense", d=10007, M=8, rows=2048, batch=128, bits=4, norm="sub", period=1, l2=1e-4),
        # the wide dense workload: 16 workers, quotient normalisation, 1 GiB of minibatch rows per iteration
        dict(name="dense_wide", kind="dense", d=1 << 16, M=16, rows=2048, batch=256, bits=2, norm="quot", period=16,
             l2=0.0),
        # sparse features, the scaled shape of the parity tests
        dict(name="csr_small", kind="csr", d=1 << 16, M=8, rows=2048, batch=512, nnz=66, bits=4, norm="sub", period=1,
             pairs=True, index=True),
        # the sparse workload: d = 2^24, 64 workers, 0.1 % density (2048 of its 16384 rows per worker resident)
        dict(name="csr_large", kind="csr", d=1 << 24, M=64, rows=2048, batch=512, nnz=16777, bits=4, norm="sub", period=1,
             pairs=True, index=True),
        # the non-convex workload, noise made on the device, reference refreshed every 16 iterations
        dict(name="rosenbrock", kind="rosenbrock", d=1 << 20, M=8, noise="device", bits=2, norm="sub", period=16),
        # gradients that come from the caller's own model, of a middling size
        dict(name="external_mid", kind="external", d=4000000, M=8, bits=2, norm="sub", scale="max", policy="last", period=1,
             window=1),
        # a small layer's gradients: launches and latency
        dict(name="codec_small", kind="codec", d=25000, M=4, bits=4, norm="sub", scale="max"),
        # the scale of the QSGD family, 16 workers
        dict(name="codec_l2", kind="codec", d=1 << 24, M=16, bits=2, norm="sub", scale="l2"),
        # long rows of odd length, a worker count that no power of two divides
        dict(name="codec_ragged", kind="codec", d=(1 << 25) + 3, M=5, bits=2, norm="sub", scale="max"),
        # the headline microbenchmark
        dict(name="codec_ternary", kind="codec", d=1 << 27, M=8, bits=2, norm="sub", scale="max"),
        # the same gradients with the wider codes and the other normalisation
        dict(name="codec_4bit_quot", kind="codec", d=1 << 27, M=8, bits=4, norm="quot", scale="max"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _dimension(rng, lo, hi, unit):
    """Any length, or (half of the time) a multiple of `unit` where the length allows it."""
    d = _log_int(rng, lo, hi)
    return max(unit, d // unit * unit) if d >= unit and rng.random() < 0.5 else d


def _codec_options(rng):
    return dict(bits=rng.choice([2, 2, 4]), norm=rng.choice(["sub"] * 5 + ["quot"] * 2 + ["none", "mean", "comb"]),
                scale=rng.choice(["max"] * 4 + ["l2"]))


def draw(rng):
    kind = rng.choice(["codec", "codec", "external", "dense", "dense", "csr", "rosenbrock"])
    if kind == "codec":
        d = _dimension(rng, 1 << 10, 1 << 27, 1024)
        M = max(1, min(_log_int(rng, 1, 64), (1 << 30) // d))
        return dict(kind=kind, d=d, M=M, **_codec_options(rng))
    if kind == "external":
        d = _dimension(rng, 1 << 10, 1 << 25, 1024)
        M = max(1, min(_log_int(rng, 1, 32), (1 << 28) // d))
        return dict(kind=kind, d=d, M=M, **_codec_options(rng), policy=rng.choice(["last", "last", "window"]),
                    period=rng.choice([1, 16]), window=rng.choice([2, 4]))
    if kind == "dense":
        d = _dimension(rng, 64, 1 << 16, 256)
        M = _log_int(rng, 1, 32)
        batch = max(8, min(_log_int(rng, 8, 512), (1 << 28) // (M * d)))
        return dict(kind=kind, d=d, M=M, rows=min(2048, (1 << 31) // (M * d)), batch=batch, bits=rng.choice([2, 4]),
                    norm=rng.choice(["sub", "sub", "quot", "none"]), period=rng.choice([1, 16]), l2=rng.choice([0.0, 1e-4]))
    if kind == "csr":
        d = _dimension(rng, 1 << 12, 1 << 24, 1 << 14)
        nnz = max(4, round(1e-3 * d))
        M = _log_int(rng, 2, 64)
        return dict(kind=kind, d=d, M=M, rows=1024, batch=_log_int(rng, 32, 512), nnz=nnz, bits=rng.choice([2, 4]),
                    norm=rng.choice(["sub", "sub", "none"]), period=rng.choice([1, 16]), pairs=rng.random() < 0.75,
                    index=rng.random() < 0.75)
    return dict(kind=kind, d=_dimension(rng, 1 << 10, 1 << 22, 1024), M=_log_int(rng, 1, 16),
                noise=rng.choice(["device", "tensor"]), bits=rng.choice([2, 4]), norm=rng.choice(["sub", "sub", "none"]),
                period=rng.choice([1, 16]))


def _full_gradient(X, y, w, l2):
    """What the convex experiments start the reference from: the gradient over all rows."""
    g = torch.zeros_like(w)
    for m in range(X.shape[0]):
        g += X[m].t() @ (torch.sigmoid(X[m] @ w) - y[m]) / (X.shape[0] * X.shape[1])
    return g + l2 * w


def prepare(case, seed):
    kind, d, M, bits = case["kind"], case["d"], case["M"], case["bits"]
    norm, scale = NORMS[case["norm"]], SCALES[case.get("scale", "max")]
    window = case.get("policy") == "window"
    lr = 1e-5 if kind == "rosenbrock" else 0.1
    ctx = B.Context(d=d, M=M, bits=bits, norm=norm, scale=scale, seed=seed, lr=lr, l2=case.get("l2", 0.0),
                    batch=case.get("batch", 0), problem=PROBLEMS[kind], ref_period=case.get("period", 1),
                    ref_policy=B.REF_WINDOW_AVG if window else B.REF_LAST_AVG, ref_window=case.get("window", 1), device=DEVICE)
    st = dict(kind=kind, ctx=ctx, it=0, codes=torch.empty((M, ctx.words), dtype=torch.int32, device=DEVICE),
              scales=torch.empty(M, device=DEVICE), vbar=torch.empty(d, device=DEVICE))
    if kind in ("codec", "external"):
        st["g"], st["gref"] = synth.codec_inputs(M, d, seed, rel_variance=0.1, device=DEVICE)
    else:
        st["g"] = torch.empty((M, d), device=DEVICE)
        st["gref"] = torch.zeros(d, device=DEVICE)
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed + 1)
    if norm == B.NORM_COMB:
        ctx.set_second_reference(torch.randn(d, generator=gen, device=DEVICE))
    if norm == B.NORM_MEAN:
        st["means"] = torch.empty(M, device=DEVICE)
        ctx.set_worker_means(st["means"])
    if window:
        st["history"] = torch.zeros((case["window"], d), device=DEVICE)
        ctx.set_reference_history(st["history"])
    if kind == "external":
        st["w"] = torch.randn(d, generator=gen, device=DEVICE)
    elif kind == "dense":
        X, y, w_star = synth.logreg_dense(M, case["rows"], d, seed, device=DEVICE)
        ctx.set_logreg_dense([X[m] for m in range(M)], [y[m] for m in range(M)])
        st["w"] = 0.5 * w_star
        st["gref"] = _full_gradient(X, y, st["w"], case["l2"])
    elif kind == "csr":
        shards = []
        for m in range(M):  # one worker at a time: the generator's temporaries are three times a shard
            (shard,), w_star = synth.logreg_csr(1, case["rows"], d, case["nnz"], seed * 1009 + m, device=DEVICE)
            if m == 0:
                st["w"] = 0.5 * w_star
            shards.append((shard[0], B.csr_pairs(shard[1], shard[2]), shard[3]) if case["pairs"] else shard)
        if case["pairs"]:
            ctx.set_logreg_csr_pairs([s[0] for s in shards], [s[1] for s in shards], [s[2] for s in shards])
        else:
            ctx.set_logreg_csr([s[0] for s in shards], [s[1] for s in shards], [s[2] for s in shards],
                               [s[3] for s in shards])
        if case["index"]:
            ctx.build_csr_index()
    elif kind == "rosenbrock":
        st["w"] = synth.rosenbrock_start(d, seed, device=DEVICE)
        if case["noise"] == "device":
            ctx.set_noise_variance(0.01)
        else:
            ctx.set_noise(synth.gradient_noise(M, d, seed, 0, variance=0.01, device=DEVICE))
    return st


def run(st):
    ctx, it = st["ctx"], st["it"]
    st["it"] = it + 1
    out = {"codes": st["codes"], "scales": st["scales"], "vbar": st["vbar"]}
    if st["kind"] == "codec":
        ctx.normalize_encode(it, st["g"], st["gref"], st["codes"], st["scales"])
        ctx.decode_aggregate(st["codes"], st["scales"], st["gref"], st["vbar"])
    else:
        ctx.step(it, st["w"], st["gref"], st["g"], st["codes"], st["scales"], st["vbar"])
        out["w"], out["gref"] = st["w"], st["gref"]
        if st["kind"] != "external":
            out["g"] = st["g"]
        if "history" in st:
            out["history"] = st["history"]
    if "means" in st:
        out["means"] = st["means"]
    return out


def work(case):
    kind, d, M = case["kind"], case["d"], case["M"]
    words = -(-d * case["bits"] // 32)
    refs = {"none": 0, "mean": 0, "comb": 2}.get(case["norm"], 1)
    nbytes = 4 * M * d + 4 * d * refs + 4 * M * words + 4 * M + 4 * d      # g, references, codes, scales, average
    flops = 5 * M * d                                                     # normalise, compare, scale, round, average
    if kind != "codec":
        period = case["period"]
        nbytes += 8 * d                                                   # the iterate, read and written
        if case.get("policy") == "window":
            nbytes += 4 * d + 4 * d * (case["window"] + 1) // period
        else:
            nbytes += 4 * d // period
        flops += 2 * d
    if kind in ("dense", "csr"):
        # rows are drawn with replacement: the distinct ones of a minibatch
        rows = case["rows"] * (1 - (1 - 1 / case["rows"]) ** case["batch"])
        stored = d if kind == "dense" else case["nnz"]
        nbytes += int(M * rows * (stored * (4 if kind == "dense" else 8) + 4))
        flops += 4 * M * case["batch"] * stored
    if kind == "rosenbrock":
        nbytes += 4 * M * d if case["noise"] == "tensor" else 0
        flops += 14 * d + M * d
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    kind = case["kind"]
    if kind in ("codec", "external") or (kind == "rosenbrock" and case["noise"] == "tensor"):
        return "exact"  # one rounding per operation, sums in a stated order: one correct result, bit for bit
    if kind == "rosenbrock":
        return {"rel": 1e-6, "max": 1e-5, "differ": 1e-6}
    # Gradients of another summation order differ in their last bits (measured: up to 5e-7, single elements 3e-6).
    n = case["M"] * case["d"]
    if n < 1 << 14:
        return {"rel": 2e-6, "max": 2e-5}
    # Of 10^9 draws about 150 then fall on the other side of their rounding decision, and each moves one element of the
    # average by a whole step of the code: 3e-4 of the average in the largest case, where that was measured, and more
    # the fewer elements the average has (one element: a step of R / 7 / 8 against about 2^8 R / 60 at d = 2^16).
    return {"rel": 1.3e-3 if n >= 1 << 28 else 4e-3 if n >= 1 << 18 else 1e-2, "max": 0.9,
            "differ": min(0.01, (2 + 6e-7 * n) / (n * case["bits"] / 32))}
