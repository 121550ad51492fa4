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
    (22 << 14, 7, 600, B.NORM_NONE, 0.0, True, True), (200, 10500, 2, B.NORM_SUB, 0.0, False, True),
    # 512 minibatch rows in all (sixteen wavefronts each), and more rows or fewer columns than that takes
    (1 << 16, 8, 64, B.NORM_SUB, 0.0, True, True), (70001, 8, 64, B.NORM_SUB, 0.0, False, False),
    (70001, 9, 57, B.NORM_SUB, 0.0, False, True), (65535, 8, 64, B.NORM_SUB, 0.0, True, False)])
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


@pytest.mark.parametrize("M,batch", [(2, 3), (4, 160)])  # sixteen wavefronts per row, one
def test_chains_of_long_rows(M, batch):
    """One row per worker, every column stored, all products the same: the roundings of a running sum then all go one
    way.  The chains are of 512 additions, whatever the length of the row (512 and 2^19 / 2^15 roundings of at most 2^-24
    of the sum, 32 for the sums over lanes and wavefronts and the products; sigma changes by a quarter of that; 8
    roundings from the residual to the gradient)."""
    d, c = 1 << 19, np.float32(1.313 / (1 << 19))
    row = (torch.tensor([0, d], dtype=torch.int64, device=DEV), torch.arange(d, dtype=torch.int32, device=DEV),
           torch.ones(d, device=DEV), torch.ones(1, device=DEV))
    ctx = make_ctx(d, M, 2, B.NORM_SUB, seed=1, batch=batch, problem=B.PROB_LOGREG_CSR)
    set_csr(ctx, [row] * M, True)
    g = torch.empty((M, d), device=DEV)
    ctx.local_grad(0, torch.full((d,), float(c), device=DEV), g)
    torch.cuda.synchronize()
    ctx.close()
    z = float(c) * d
    want = 1.0 / (1.0 + np.exp(-z)) - 1.0
    bound = (0.25 * z * (512 + d / 2 ** 15 + 32) + 8 * abs(want)) * 2.0 ** -24
    worst = np.abs(g.cpu().numpy().astype(np.float64) - want).max()
    assert worst <= bound, f"{worst} > {bound}"


# The pipeline over workers where d is no multiple of a tile: rows of g at every 4-byte phase (odd lengths and numbers of workers), a
# last tile of one, two, three and many columns, groups of workers that do not come out even, each kind of normalisation it takes.
@pytest.mark.parametrize("d,M,batch,norm,index,pairs", [
    ((1 << 18) + 1, 9, 40, B.NORM_SUB, True, True), ((1 << 18) + 2, 9, 33, B.NORM_QUOT, False, True),
    ((13 << 14) + 3, 11, 512, B.NORM_NONE, True, False), ((1 << 17) + 5, 17, 70, B.NORM_SUB, True, False),
    ((1 << 17) + 4, 17, 5, B.NORM_QUOT, True, True), ((1 << 18) - 1, 9, 40, B.NORM_NONE, False, True),
    ((1 << 20) + 1, 3, 20, B.NORM_SUB, True, True), ((1 << 15) + 3, 70, 30, B.NORM_QUOT, False, False),
    (16385, 129, 3, B.NORM_SUB, True, True)])
def test_workers_in_turn_on_ragged_tiles(d, M, batch, norm, index, pairs):
    test_gradient_and_step(d, M, batch, norm, 0.0, index, pairs)
