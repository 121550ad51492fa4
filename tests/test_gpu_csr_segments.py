"""Sparse logistic gradient with row segments of every length at the edges of what the lanes of a group hold (16 entries a
load, two and three loads, the loop behind them), odd lengths (read with the entry before them) and the first entries of
the arrays (which have none before them), by the column tiles and by the few-columns kernels, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import tng_oracle as O
from gpu_util import DEV, buffers, grad_close, logistic_condition_csr, make_ctx, set_csr
from paper_1901_08227_amd import binding as B

pytestmark = pytest.mark.gpu
TILE = 1 << 14
LENGTHS = [1, 0, 2, 3, 15, 16, 17, 31, 32, 33, 34, 47, 48, 49, 63, 64, 65, 97, 200, 5]


def shard(n, d, first, seed):
    """n rows; segment t of row i has LENGTHS[(i + 3 t + first) mod ...] entries; first < 0: one entry in all, column 7."""
    rng = np.random.default_rng(seed)
    rows = []
    for i in range(n):
        if first < 0:
            rows.append(np.array([7] if i == n - 1 else [], dtype=np.int32))
            continue
        parts = []
        for t in range(-(-d // TILE)):
            width = min(TILE, d - t * TILE)
            k = min(width, LENGTHS[(i + 3 * t + first) % len(LENGTHS)])
            parts.append(t * TILE + np.sort(rng.choice(width, k, replace=False)).astype(np.int32))
        rows.append(np.concatenate(parts))
    ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
    col = np.concatenate(rows).astype(np.int32)
    val = rng.standard_normal(len(col)).astype(np.float32)
    y = rng.integers(0, 2, n).astype(np.float32)
    return tuple(torch.from_numpy(a).to(DEV) for a in (ptr, col, val, y))


@pytest.mark.parametrize("M,d,pairs,l2", [(17, 1 << 17, True, 0.0), (17, 1 << 17, False, 0.0), (17, (1 << 17) + 5, True, 1e-3),
                                          (1, 130 * TILE, True, 0.0), (3, 1 << 16, True, 0.0), (3, 70003, False, 0.0)])
@pytest.mark.parametrize("norm", [B.NORM_SUB, B.NORM_COMB])
def test_segment_lengths(M, d, pairs, l2, norm):
    n, batch, seed = 20, 48, 3
    shards = [shard(n, d, m % 20 if m != 2 else -1, seed + m) for m in range(M)]
    ctx = make_ctx(d, M, 4, norm, seed=seed, lr=0.1, l2=l2, batch=batch, problem=B.PROB_LOGREG_CSR)
    set_csr(ctx, shards, pairs)
    gen = torch.Generator(device=DEV).manual_seed(seed)
    w = 0.1 * torch.randn(d, device=DEV, generator=gen)
    g = torch.empty((M, d), device=DEV)
    w0 = w.cpu().numpy()
    ctx.set_second_reference(torch.ones(d, device=DEV))
    ctx.step(2, w, torch.zeros(d, device=DEV), g, torch.empty((M, -(-d // 8)), dtype=torch.int32, device=DEV),
             torch.empty(M, device=DEV), torch.empty(d, device=DEV))
    torch.cuda.synchronize()
    for m in range(M):
        host = tuple(t.cpu().numpy() for t in shards[m])
        ids = O.minibatch_indices(seed, 2, m, batch, n)
        ref = O.grad_logreg_csr(*host, w0, ids, d, l2)
        assert grad_close(g[m].cpu().numpy(), ref, logistic_condition_csr(*host, w0, ids, d, l2)), f"worker {m}"
    ctx.close()


# A workgroup of the pipeline over tiles stores a tile's maximum while its wavefronts are already at the next one's: the scale is
# the one of the gradient that was written, wherever the row's largest entry lies (first, last and any tile between, any wavefront's columns).
@pytest.mark.parametrize("M,norm", [(1, B.NORM_NONE), (1, B.NORM_SUB), (1, B.NORM_QUOT), (2, B.NORM_COMB)])
def test_scales_of_the_pipeline_over_tiles(M, norm):
    ntiles, n, batch, seed = 130, 12, 3, 5
    d, rng = ntiles * TILE, np.random.default_rng(5)
    col = np.concatenate([np.concatenate([t * TILE + np.sort(rng.choice(TILE, 30, replace=False)) for t in range(ntiles)])
                          for _ in range(n)]).astype(np.int32)
    val = rng.uniform(0.5, 1.0, len(col)).astype(np.float32)
    for i in range(n):
        val[i * 30 * ntiles + (0, 30 * ntiles - 1, *rng.integers(0, 30 * ntiles, n - 2))[i]] = 50.0
    row = tuple(torch.from_numpy(a).to(DEV) for a in (np.arange(n + 1, dtype=np.int64) * 30 * ntiles, col, val, np.zeros(n, np.float32)))
    ctx = make_ctx(d, M, 4, norm, seed=seed, lr=0.0, batch=batch, problem=B.PROB_LOGREG_CSR)
    set_csr(ctx, [row] * M, True)
    gref, gref2 = torch.full((d,), 1e-3, device=DEV), torch.ones(d, device=DEV)
    ctx.set_second_reference(gref2)
    buf = buffers(ctx)
    for it in range(12):
        ref = gref.clone()
        ctx.step(it, torch.zeros(d, device=DEV), ref, buf["g"], buf["codes"], buf["scales"], buf["vbar"])
        g = buf["g"].cpu().numpy()
        want = [O.scale_of(O.normalize(g[m], gref.cpu().numpy(), norm, float(ctx.cfg.quot_eps), gref2.cpu().numpy()), O.SCALE_MAX)
                for m in range(M)]
        assert np.array_equal(buf["scales"].cpu().numpy(), np.array(want, np.float32)), f"iteration {it}"
    ctx.close()
