"""Elements of a gradient that are infinite or no number: every path gives them the same codes (two bits: level 0; four: the top
level, negative only below 0), rows without a number code to 0, and what an iteration averages is what its codes decode to."""
import numpy as np
import pytest
import torch

from oracle import tng_oracle as O
from gpu_util import DEV, buffers, make_ctx, u32
from paper_1901_08227_amd import binding as B

pytestmark = pytest.mark.gpu


def plant(g, kinds):
    """Row m gets kind m: odd ends, a middle and every 97th element; kind "all": a row without a number."""
    for m, kind in enumerate(kinds):
        if kind == "all":
            g[m] = -np.nan
        elif kind is not None:
            g[m, 5::97] = kind
            g[m, -1] = g[m, g.shape[1] // 2] = kind


def expected(g, gref, seed, it, bits):
    S, codes, scales = np.float32(2 ** (bits - 1) - 1), [], []
    with np.errstate(all="ignore"):
        for m in range(len(g)):
            v = g[m] - gref
            R = np.fmax.reduce(np.abs(v), initial=np.float32(0.0))
            R = R if R >= O.FLT_MIN else np.float32(0.0)
            u = O.uniform_from_word(O.quant_draw_words(seed, it, m, len(v)))
            if R == 0.0:
                level = np.zeros(len(v), np.uint32)
            else:
                p = np.abs(v) * (np.float32(1.0) / R)
                if bits == 2:
                    level = (u < p).astype(np.uint32)
                else:
                    x = np.fmin(p, np.float32(1.0)) * S
                    lo = np.floor(x)
                    level = lo.astype(np.uint32) + (u < x - lo)
            codes.append(O.pack(level, (v < 0) & (level != 0), bits))
            scales.append(R)
    return np.stack(codes), np.array(scales, np.float32)


NAN, NNAN, INF = np.float32(np.nan), np.float32(-np.nan), np.float32(np.inf)
KINDS = [NAN, NNAN, INF, -INF, "all", None]


# one launch, rows longer than it takes (two passes), one workgroup, tails of an iteration with one and with many wavefronts for the
# workers, and one with more workers than they take
@pytest.mark.parametrize("d,M", [(1000, 6), (1003, 6), (4097, 7), (30001, 6), (1 << 18, 8), ((1 << 18) + 5, 6), (1 << 21, 6),
                                 ((1 << 21) + 1027, 7), (5000, 64), (5000, 66)])
@pytest.mark.parametrize("bits", [2, 4])
def test_not_finite(d, M, bits):
    print(f"not finite d={d} M={M} bits={bits}", flush=True)
    rng = np.random.default_rng(d)
    g = rng.standard_normal((M, d), dtype=np.float32)
    gref = (0.5 * rng.standard_normal(d)).astype(np.float32)
    plant(g, KINDS)
    want, scales = expected(g, gref, 3, 4, bits)
    ctx = make_ctx(d, M, bits, B.NORM_SUB, seed=3, lr=0.1, ref_policy=B.REF_ZERO)
    buf, dev = buffers(ctx), torch.from_numpy(gref).to(DEV)
    ctx.normalize_encode(4, torch.from_numpy(g).to(DEV), dev, buf["codes"], buf["scales"])
    assert np.array_equal(buf["scales"].cpu().numpy(), scales)
    bad = np.nonzero(u32(buf["codes"]) != want)
    assert len(bad[0]) == 0, f"encode: {len(bad[0])} words, first {bad[0][0]}, {bad[1][0]}"
    average = torch.empty(d, device=DEV)
    ctx.decode_aggregate(buf["codes"], buf["scales"], dev, average)
    buf["g"].copy_(torch.from_numpy(g))
    buf["codes"].fill_(-1)
    ctx.step(4, torch.zeros(d, device=DEV), dev.clone(), buf["g"], buf["codes"], buf["scales"], buf["vbar"])
    assert np.array_equal(buf["scales"].cpu().numpy(), scales)
    bad = np.nonzero(u32(buf["codes"]) != want)
    assert len(bad[0]) == 0, f"step: {len(bad[0])} words, first {bad[0][0]}, {bad[1][0]}"
    assert np.array_equal(buf["vbar"].cpu().numpy(), average.cpu().numpy(), equal_nan=True)
    ctx.close()


# The candidate slots (two bits, 2^26 elements and more).  In the tiles of the sample (every 128th of 1024 elements) a number that is none
# leaves the row to the ordinary path and an infinite one makes the bound infinite; elsewhere they meet slots that have a bound.  Rows that
# all have slots go through the scale pass's loop without branches, next to others through the one with them.
OUT, SAMPLED = (1024 * 5 + 3, 1024 * 5 + 700, 1024 * 300 + 64, -1), (0, 1024 * 128 + 511, 1024 * 256 + 1023)


@pytest.mark.parametrize("M,d,plants", [
    (8, 1 << 23, [(NAN, None), (NNAN, None), (INF, None), (-INF, None), (None, INF), (NAN, -INF), (INF, INF), (None, None)]),
    (8, (1 << 23) + 1027, [(None, NAN), (INF, NNAN), ("all", None), (NAN, None), (INF, None), (None, -INF), (NAN, INF), (None, None)]),
    (5, 13108 * 1024, [(NAN, None), (INF, None), (NNAN, INF), (None, -INF), (None, None)]),
    (1, (1 << 26) + 1024, [(NAN, None)]), (1, (1 << 26) + 1024, [(-INF, None)])])
def test_not_finite_in_slots(M, d, plants):
    print(f"not finite in slots d={d} M={M}", flush=True)
    rng = np.random.default_rng(M)
    gref = rng.standard_normal(d, dtype=np.float32)
    g = np.stack([gref + np.float32(0.3) * rng.standard_normal(d, dtype=np.float32) * np.abs(gref) for _ in range(M)])
    for m, (out, sampled) in enumerate(plants):
        if isinstance(out, str):
            g[m] = NAN
            continue
        for value, at in ((out, OUT), (sampled, SAMPLED)):
            if value is not None:
                g[m, list(at)] = value
    want, scales = expected(g, gref, 3, 4, 2)
    assert all(np.isinf(s) == (INF in np.abs([p for p in kinds if not isinstance(p, str) and p is not None])) for s, kinds in zip(scales, plants))
    ctx = make_ctx(d, M, 2, B.NORM_SUB, seed=3)
    buf = buffers(ctx)
    ctx.normalize_encode(4, torch.from_numpy(g).to(DEV), torch.from_numpy(gref).to(DEV), buf["codes"], buf["scales"])
    assert np.array_equal(buf["scales"].cpu().numpy(), scales)
    bad = np.nonzero(u32(buf["codes"]) != want)
    assert len(bad[0]) == 0, f"{len(bad[0])} words, first {bad[0][0]}, {bad[1][0]}"
    ctx.close()


# Eight columns that are infinite in every row make NaN of the gradient there (0 times infinity where the residual is 0) and leave
# the rest of it alone: the scale is the largest of the rest, which lies next to them, in each kernel that leaves maxima.
@pytest.mark.parametrize("d,M,batch", [(1000, 4, 64), (1003, 3, 20), (5003, 3, 40), (5000, 3, 8), (9001, 2, 6), (20002, 16, 40),
                                       (65536, 2, 300), (65540, 2, 9)])
def test_maxima_of_gradients_with_nan(d, M, batch):
    rng = np.random.default_rng(d)
    n, a, b = 16, d // 2 // 8 * 8, d // 2 // 8 * 8 + 8
    X, w = rng.standard_normal((n, d), dtype=np.float32), np.full(d, 1e-3, np.float32)
    X[:, a:b], X[:, a - 1], X[:, b] = np.inf, 40.0, -30.0
    y = np.arange(n, dtype=np.float32) % 2  # z = infinity: residuals 1 and 0
    ctx = make_ctx(d, M, 4, B.NORM_SUB, seed=1, lr=0.0, batch=batch, problem=B.PROB_LOGREG_DENSE, ref_policy=B.REF_ZERO)
    ctx.set_logreg_dense([torch.from_numpy(X).to(DEV)] * M, [torch.from_numpy(y).to(DEV)] * M)
    buf = buffers(ctx)
    ctx.step(1, torch.from_numpy(w).to(DEV), torch.zeros(d, device=DEV), buf["g"], buf["codes"], buf["scales"], buf["vbar"])
    g = buf["g"].cpu().numpy()
    assert np.isnan(g[:, a:b]).all() and np.isfinite(np.delete(g, np.s_[a:b], axis=1)).all()
    assert np.array_equal(buf["scales"].cpu().numpy(), np.fmax.reduce(np.abs(g), axis=1))
    ctx.close()
