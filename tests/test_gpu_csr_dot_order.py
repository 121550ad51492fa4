"""Dot products of sparse rows by the column tiles: 32 running sums per row and tile (or pair of tiles), added in pairs, whatever the
segment's length and wherever it starts.  One row of one worker is drawn and its dot product is near -30, so that the gradient, the
residual times the row's values, shows the last bit of z: the residual is then exp(z) but for 1e-13, and one bit of z is 1.9e-6
of it, against 2^-24 of each of a handful of operations on the way."""
import numpy as np
import pytest
import torch

from oracle import tng_oracle as O
from gpu_util import DEV, make_ctx, set_csr
from paper_1901_08227_amd import binding as B

pytestmark = pytest.mark.gpu
TILE = 1 << 14


def fma(a, b, c):
    """One rounding (of the sum in binary64: twice in one of 2^29 cases)."""
    return (a.astype(np.float64) * b + c).astype(np.float32)


def dot(col, val, w, width):
    """z as the kernels add it: tiles of width columns, their sums by four quarters of the tiles, four sums each."""
    parts = []
    for c0 in range(0, len(w), width):
        a, b = np.searchsorted(col, [c0, c0 + width])
        n = -(-(b - a) // 32) * 32
        v, x = np.zeros(n, np.float32), np.zeros(n, np.float32)
        v[:b - a], x[:b - a] = val[a:b], w[col[a:b]]
        acc = np.zeros(32, np.float32)
        for k in range(0, n, 32):
            acc = fma(v[k:k + 32], x[k:k + 32], acc)
        while len(acc) > 1:
            acc = acc[:len(acc) // 2] + acc[len(acc) // 2:]
        parts.append(acc[0])
    per, quarters = -(-len(parts) // 4), []
    for q in range(4):
        mine = parts[q * per:(q + 1) * per]
        a = [np.float32(0.0)] * 4
        whole = len(mine) // 4 * 4
        for k in range(whole):
            a[k % 4] = a[k % 4] + mine[k]
        for p in mine[whole:]:
            a[0] = a[0] + p
        quarters.append((a[0] + a[1]) + (a[2] + a[3]))
    return ((quarters[0] + quarters[1]) + quarters[2]) + quarters[3]


@pytest.mark.parametrize("d,M,width", [(1 << 19, 5, 2 * TILE), ((1 << 19) - 21, 5, 2 * TILE), (TILE, 130, TILE)])
@pytest.mark.parametrize("pairs", [True, False])
def test_order_of_the_sums(d, M, width, pairs):
    n, seed, it = 4, 11, 3
    rng = np.random.default_rng(d)
    shards, host = [], []
    w = rng.uniform(0.5, 1.5, d).astype(np.float32)
    for m in range(M):  # dense rows, a handful of entries, odd and even numbers of them
        rows = []
        for i in range(n):
            share = (1.0, 0.5, 0.01, 0.003, 0.001)[(m + i) % 5]
            keep = np.nonzero(rng.random(d) < share)[0] if share < 1 else np.arange(d - (m // 5 + i) % 2)
            rows.append(keep.astype(np.int32) if len(keep) else np.array([d // 2], np.int32))
        ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
        val = [-rng.uniform(0.1, 1.9, len(r)) for r in rows]
        val = [(30.0 * v / -(v @ w[r])).astype(np.float32) for v, r in zip(val, rows)]
        host.append((rows, val))
        shards.append(tuple(torch.from_numpy(a).to(DEV) for a in (ptr, np.concatenate(rows), np.concatenate(val),
                                                                   np.zeros(n, np.float32))))
    ctx = make_ctx(d, M, 2, B.NORM_SUB, seed=seed, batch=1, problem=B.PROB_LOGREG_CSR)
    set_csr(ctx, shards, pairs)
    g = torch.empty((M, d), device=DEV)
    ctx.local_grad(it, torch.from_numpy(w).to(DEV), g)
    torch.cuda.synchronize()
    ctx.close()
    for m in range(min(M, 20)):
        i = int(O.minibatch_indices(seed, it, m, 1, n)[0])
        cols, vals = host[m][0][i], host[m][1][i]
        z = dot(cols, vals, w, width)
        got = g[m].cpu().numpy()[cols].astype(np.float64) / vals
        off = np.abs(got / np.exp(np.float64(z)) - 1.0).max()
        assert off <= 8 * 2.0 ** -24, f"worker {m}, {len(cols)} entries: {off}"


# Columns that no row stores may hold anything: lanes without an entry of their own must not bring them into a sum.
@pytest.mark.parametrize("d,M", [(1 << 17, 17), ((1 << 17) + 5, 17), (TILE, 130), (300, 7000), (1 << 16, 3)])
@pytest.mark.parametrize("pairs", [True, False])
def test_columns_without_entries_are_not_read_into_the_sums(d, M, pairs):
    n, batch, rng = 6, 9, np.random.default_rng(d)
    rows = [np.sort(rng.choice(np.arange(1, min(d, TILE)), k, replace=False)) for k in (1, 2, 17, 33, 64, 199)]
    rows = [np.concatenate([r + t for t in range(0, d, TILE) if t + r[-1] < d]).astype(np.int32) for r in rows]
    ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
    shard = tuple(torch.from_numpy(a).to(DEV) for a in (ptr, np.concatenate(rows), rng.standard_normal(ptr[-1]).astype(np.float32),
                                                        np.zeros(n, np.float32)))
    ctx = make_ctx(d, M, 2, B.NORM_SUB, seed=7, batch=batch, problem=B.PROB_LOGREG_CSR)
    set_csr(ctx, [shard] * M, pairs)
    w = 0.1 * torch.randn(d, device=DEV)
    g = []
    for filling in (1.0, float("inf"), float("nan")):
        w[::TILE] = filling
        g.append(torch.empty((M, d), device=DEV))
        ctx.local_grad(1, w, g[-1])
    ctx.close()
    assert torch.isfinite(g[0]).all() and torch.equal(g[0], g[1]) and torch.equal(g[0], g[2])
