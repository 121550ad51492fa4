"""Tiny dense logistic problems (all gradients in one workgroup): lengths that end inside a float4, the most workers and
columns that the two launches take and one more, minibatches around their rows per trip, against the oracle; and the
gradient of tng_local_grad against the one that tng_step makes."""
import pytest
import torch

from gpu_util import DEV, buffers, make_ctx
from paper_1901_08227_amd import binding as B, synth
from test_gpu_step import _dense_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,M,batch", [(4, 1, 1), (5, 2, 3), (7, 70, 4), (16, 256, 5), (255, 16, 130), (1000, 4, 64), (1023, 4, 517),
                                       (1024, 4, 8), (1024, 5, 8), (1025, 3, 9), (3, 2, 6)])
def test_edges(d, M, batch):
    for bits, norm in ((2, B.NORM_SUB), (4, B.NORM_QUOT)):
        _dense_case(M, 40, d, batch, bits, norm, 2, seed=d + M, l2=1e-3)


@pytest.mark.parametrize("d,norm", [(1000, B.NORM_SUB), (333, B.NORM_NONE), (1022, B.NORM_COMB), (77, B.NORM_MEAN)])
def test_local_gradient_is_the_one_of_the_step(d, norm):
    M, n, batch = 4, 52, 37  # (52 rows: every shard starts on 16 bytes)
    X, y, _ = synth.logreg_dense(M, n, d, seed=d, device=DEV)
    ctx = make_ctx(d, M, 2, norm, seed=d, lr=0.1, l2=1e-3, batch=batch, ref_period=1, problem=B.PROB_LOGREG_DENSE)
    ctx.set_logreg_dense([X[m] for m in range(M)], [y[m] for m in range(M)])
    second = torch.rand(d, device=DEV) + 0.5
    if norm == B.NORM_COMB:
        ctx.set_second_reference(second)
    means = torch.zeros(M, device=DEV)
    if norm == B.NORM_MEAN:
        ctx.set_worker_means(means)
    buf, apart = buffers(ctx), buffers(ctx)
    w = torch.linspace(-0.1, 0.1, d, device=DEV)
    gref = torch.linspace(0.01, -0.01, d, device=DEV)
    ref = gref.clone()
    ctx.local_grad(5, w, apart["g"])
    ctx.normalize_encode(5, apart["g"], ref, apart["codes"], apart["scales"])
    ctx.decode_aggregate(apart["codes"], apart["scales"], ref, apart["vbar"])
    ctx.step(5, w, gref, buf["g"], buf["codes"], buf["scales"], buf["vbar"])
    torch.cuda.synchronize()
    for name in ("g", "codes", "scales", "vbar"):
        assert torch.equal(buf[name], apart[name]), name
    assert torch.equal(gref, buf["vbar"])
    ctx.close()
