"""The ordered row sums (mean reference, l2 scale) where their finishing kernel takes its groups of 256 chunks in several
batches: rows of 2^24 elements (16 groups, one round of loads) and of 2^26 (64 groups, one batch), and a chunk to either
side, against the oracle bit for bit."""
import numpy as np
import pytest
import torch

from gpu_util import DEV, buffers, make_ctx, say
from oracle import tng_oracle as O
from paper_1901_08227_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,d", [(2, (1 << 24) - 4096), (2, (1 << 24) + 1), (1, 1 << 26), (1, (1 << 26) + 5),
                                 (1, 5 * (1 << 25) - 3)])
def test_edges_of_the_batches(M, d):
    say(f"row sums d={d} M={M}")
    g = torch.randn((M, d), device=DEV, generator=torch.Generator(device=DEV).manual_seed(d % 1000))
    ctx = make_ctx(d, M, 2, B.NORM_MEAN, seed=3, scale=B.SCALE_L2)
    buf = buffers(ctx)
    means = torch.full((M,), float("nan"), device=DEV)
    ctx.set_worker_means(means)
    ctx.normalize_encode(1, g, g[0], buf["codes"], buf["scales"])
    torch.cuda.synchronize()
    ctx.close()
    for m in range(M):
        row = g[m].cpu().numpy()
        mu = O.worker_mean(row)
        assert means[m].item() == mu
        assert buf["scales"][m].item() == O.scale_of(O.normalize(row, None, B.NORM_MEAN, mu=mu), B.SCALE_L2)
