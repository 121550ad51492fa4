"""Sparse logistic gradient by column tiles, minibatches around the ends of the pieces of 128 and 256 rows in which the two passes take them
(one to four pieces a trip, up to four trips of one worker), segments of every length, rows of any length and whole tiles; and
workgroups that turn the ring of three staged rounds more than once: nine workers of a tile in the gradient pass, four in the dot
products.  Against the oracle; scales from the gradient that was written."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest
import torch

from gpu_util import DEV, buffers, grad_close, logistic_condition_csr, make_ctx, set_csr
from oracle import tng_oracle as O
from paper_1901_08227_amd import binding as B
from test_gpu_csr_segments import TILE, shard

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 2, 127, 128, 129, 255, 256, 257, 383, 384, 385, 511, 512, 513, 640, 768, 769, 1700])
@pytest.mark.parametrize("M,d,pairs,norm", [(17, 8 * TILE, True, B.NORM_SUB), (33, 5 * TILE - 7, False, B.NORM_NONE)])
def test_minibatches_around_the_ends_of_a_piece(batch, M, d, pairs, norm):
    n, seed = 40, 7
    shards = [shard(n, d, m % 20 if m != 2 else -1, seed + m) for m in range(M)]
    ctx = make_ctx(d, M, 4, norm, seed=seed, lr=0.0, batch=batch, problem=B.PROB_LOGREG_CSR)
    set_csr(ctx, shards, pairs)
    ctx.build_csr_index()
    w = 0.1 * torch.randn(d, device=DEV, generator=torch.Generator(device=DEV).manual_seed(seed))
    buf, w0 = buffers(ctx), w.cpu().numpy()
    ctx.step(3, w, torch.zeros(d, device=DEV), buf["g"], buf["codes"], buf["scales"], buf["vbar"])
    torch.cuda.synchronize()
    g = buf["g"].cpu().numpy()
    for m in range(M):
        host = tuple(t.cpu().numpy() for t in shards[m])
        ids = O.minibatch_indices(seed, 3, m, batch, n)
        ref = O.grad_logreg_csr(*host, w0, ids, d)
        assert grad_close(g[m], ref, logistic_condition_csr(*host, w0, ids, d)), f"worker {m}"
        assert buf["scales"][m].item() == O.scale_of(g[m], O.SCALE_MAX), f"scale of worker {m}"
    ctx.close()


@pytest.mark.parametrize("d,batch,pairs,norm", [(1 << 24, 200, True, B.NORM_SUB), ((1 << 24) - 9, 100, False, B.NORM_NONE),
                                                ((1 << 24) - 9, 200, True, B.NORM_QUOT), ((1 << 24) - 9, 400, False, B.NORM_SUB),
                                                (1 << 24, 300, False, B.NORM_NONE), ((1 << 24) - 9, 384, True, B.NORM_SUB)])
def test_rounds_of_a_workgroup(d, batch, pairs, norm):
    M, n, seed = 9, 24, 11
    rng, rows = np.random.default_rng(d + batch), []
    for m in range(M):
        cols = [np.unique(np.append(rng.integers(0, d, k), (0, d - 1)[:k])) for k in (0, 1, 2, 300, 5000, 40000, *rng.integers(0, 3000, n - 6))]
        ptr = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int64)
        rows.append((ptr, np.concatenate(cols).astype(np.int32), rng.standard_normal(ptr[-1]).astype(np.float32), rng.integers(0, 2, n).astype(np.float32)))
    ctx = make_ctx(d, M, 4, norm, seed=seed, lr=0.0, batch=batch, problem=B.PROB_LOGREG_CSR)
    set_csr(ctx, [tuple(torch.from_numpy(a).to(DEV) for a in r) for r in rows], pairs)
    ctx.build_csr_index()
    gen = torch.Generator(device=DEV).manual_seed(seed)
    w, gref = 0.1 * torch.randn(d, device=DEV, generator=gen), 1e-3 * torch.randn(d, device=DEV, generator=gen)
    buf, w0, r0 = buffers(ctx), w.cpu().numpy(), gref.cpu().numpy()
    ctx.step(3, w, gref, buf["g"], buf["codes"], buf["scales"], buf["vbar"])
    torch.cuda.synchronize()
    g, scales = buf["g"].cpu().numpy(), buf["scales"].cpu().numpy()

    def right(m):
        ids = O.minibatch_indices(seed, 3, m, batch, n)
        return (grad_close(g[m], O.grad_logreg_csr(*rows[m], w0, ids, d), logistic_condition_csr(*rows[m], w0, ids, d))
                and scales[m] == O.scale_of(O.normalize(g[m], r0, norm, float(ctx.cfg.quot_eps)), O.SCALE_MAX))

    with ThreadPoolExecutor(max_workers=5) as pool:
        assert [m for m, ok in enumerate(pool.map(right, range(M))) if not ok] == []
    ctx.close()
