"""Sparse logistic gradient by column tiles, minibatches around the ends of the pieces of 128 rows in which the two passes take them (one,
two or four pieces a trip, several trips), segments of every length, rows of any length and whole tiles, one worker per
workgroup and several, against the oracle; scales from the gradient that was written."""
import numpy as np
import pytest
import torch

from gpu_util import DEV, buffers, grad_close, logistic_condition_csr, make_ctx, set_csr
from oracle import tng_oracle as O
from paper_1901_08227_amd import binding as B
from test_gpu_csr_segments import TILE, shard

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 2, 127, 128, 129, 255, 256, 257, 385, 511, 512, 513, 640])
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
