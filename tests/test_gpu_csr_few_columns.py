"""Sparse logistic gradient on either side of the rule for few columns (2^21 columns of all workers): the row and
sub-tile kernels at the edges of their column blocks, and the column-tile kernels with few workers, ragged lengths,
an l2 term, long minibatches and two references, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import tng_oracle as O
from gpu_util import DEV, buffers, grad_close, logistic_condition_csr, make_ctx, oracle_cfg, set_csr, u32
from paper_1901_08227_amd import binding as B
from test_gpu_step import _ragged_csr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,M,batch,norm,l2,index,pairs", [
    (1, 2, 3, B.NORM_SUB, 0.0, True, True), (257, 3, 70, B.NORM_QUOT, 0.0, False, True),
    (1025, 64, 5, B.NORM_NONE, 0.0, True, False), (4097, 9, 64, B.NORM_COMB, 1e-3, False, False),
    ((1 << 16) - 3, 8, 520, B.NORM_SUB, 1e-3, True, True), (1 << 18, 8, 40, B.NORM_MEAN, 0.0, True, True),
    # one column more than the rule takes, and the pipelines over tiles (M = 1, two references) and workers
    ((1 << 18) + 1, 8, 40, B.NORM_SUB, 1e-3, False, True), (130 << 14, 1, 40, B.NORM_SUB, 0.0, True, True),
    (22 << 14, 7, 130, B.NORM_COMB, 0.0, True, False), (22 << 14, 7, 130, B.NORM_QUOT, 0.0, False, True),
    (22 << 14, 7, 600, B.NORM_NONE, 0.0, True, True), (200, 10500, 2, B.NORM_SUB, 0.0, False, True)])
def test_gradient_and_step(d, M, batch, norm, l2, index, pairs):
    n, seed = 30 if M < 100 else 2, 31
    longest = min(d, 3000)
    lens = lambda m, i: min(longest, [0, 1, 70, 3000, 40, 1500][(i + m) % 6])
    shards = _ragged_csr(min(M, 7), n, d, lens, seed)
    shards = [shards[m % len(shards)] for m in range(M)]
    ctx = make_ctx(d, M, 4, norm, seed=seed, lr=0.1, l2=l2, batch=batch, problem=B.PROB_LOGREG_CSR)
    set_csr(ctx, shards, pairs)
    if index:
        ctx.build_csr_index()
    gen = torch.Generator(device=DEV).manual_seed(seed)
    w = 0.1 * torch.randn(d, device=DEV, generator=gen)
    gref = 1e-3 * torch.randn(d, device=DEV, generator=gen)
    gref2 = torch.rand(d, device=DEV, generator=gen) + 0.5
    if norm == B.NORM_COMB:
        ctx.set_second_reference(gref2)
    if norm == B.NORM_MEAN:
        means = torch.zeros(M, device=DEV)
        ctx.set_worker_means(means)
    buf = buffers(ctx)
    w0, r0 = w.cpu().numpy(), gref.cpu().numpy()
    ctx.step(5, w, gref, buf["g"], buf["codes"], buf["scales"], buf["vbar"])
    torch.cuda.synchronize()
    gh = buf["g"].cpu().numpy()
    host = {id(s): tuple(t.cpu().numpy() for t in s) for s in shards}
    for m in range(M) if M < 100 else (0, 1, 6, M - 1):
        ids, h = O.minibatch_indices(seed, 5, m, batch, n), host[id(shards[m])]
        ref = O.grad_logreg_csr(*h, w0, ids, d, l2)
        assert grad_close(gh[m], ref, logistic_condition_csr(*h, w0, ids, d, l2)), f"worker {m}"
    want = O.step(oracle_cfg(ctx), 5, w0, r0, gh, gref2.cpu().numpy())
    got = (w.cpu().numpy(), gref.cpu().numpy(), u32(buf["codes"]), buf["scales"].cpu().numpy(), buf["vbar"].cpu().numpy())
    for name, a, b in zip(("iterate", "reference", "codes", "scales", "average"), got, want):
        assert np.array_equal(a, b), name
    ctx.close()
