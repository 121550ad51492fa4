"""The ragged last wavefront tile (1024 coordinates) of a row in the scale, quantise and decode kernels: it has
workgroups of its own, a worker per wavefront, next to whole tiles that take 1 to 16 workers per workgroup."""
import pytest
import torch

from gpu_util import DEV, buffers, make_ctx
from paper_1901_08227_amd import binding as B
from test_gpu_codec import NORMS, _check_encode_decode, _inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("norm", NORMS)
@pytest.mark.parametrize("d", [2, 1021, 1023, 1025, 4095, 4097, 5122])
def test_edges_of_the_last_tile(d, norm):
    for M, bits in [(1, 2), (9, 4)]:
        g, gref, gref2 = _inputs(M, d, seed=d + M)
        ctx = make_ctx(d, M, bits, norm, seed=d + 3)
        _check_encode_decode(ctx, 3, g, gref, gref2, "last tile")
        ctx.close()


@pytest.mark.parametrize("M,log2d", [(2, 23), (5, 22), (8, 23), (16, 23)])  # 2, 4 (a short group), 8 and 16 workers per workgroup
def test_ragged_tail_behind_grouped_workers(M, log2d):
    d = (1 << log2d) + 1024 + 3
    for bits, norm in [(2, B.NORM_SUB), (4, B.NORM_QUOT)]:
        g, gref, gref2 = _inputs(M, d, seed=M)
        ctx = make_ctx(d, M, bits, norm, seed=M)
        _check_encode_decode(ctx, 1, g, gref, gref2, "grouped workers")
        ctx.close()


# The scale pass of one group of workers: 1024 workgroups from 4096 * 1024 coordinates on, which walk the tiles (the last trip short, a
# ragged tile behind it); the largest element in the last whole tile and in the ragged one.
@pytest.mark.parametrize("d,M,at", [((1 << 22) + 4096, 1, (1 << 22) + 4095), ((1 << 23) + 3 * 4096 + 1029, 1, (1 << 23) + 3 * 4096 + 1028),
                                    ((1 << 23) + 1024 + 3, 2, (1 << 23) + 1023)])
def test_scale_pass_that_walks_the_tiles(d, M, at):
    gen = torch.Generator(device=DEV).manual_seed(d)
    g = torch.randn((M, d), generator=gen, device=DEV).clamp_(-4, 4)
    gref = torch.zeros(d, device=DEV)
    g[M - 1, at] = -7.5
    ctx = make_ctx(d, M, 4, B.NORM_SUB, seed=3)
    buf = buffers(ctx)
    ctx.normalize_encode(1, g, gref, buf["codes"], buf["scales"])
    assert torch.equal(buf["scales"], g.abs().amax(dim=1)) and float(buf["scales"][M - 1]) == 7.5
    ctx.close()


# Encode of short rows of many workers: every tile keeps a workgroup of its own (the scale pass is held to fewer only ahead of the
# one-launch tail), seen by the rows of partial maxima at the head of a workspace that holds no problem data.
@pytest.mark.parametrize("d,M", [(163840, 64), (98304, 128), (190000, 32), (266243, 16)])
def test_scale_pass_ahead_of_the_quantiser(d, M):
    gen = torch.Generator(device=DEV).manual_seed(d)
    g, gref = torch.randn((M, d), generator=gen, device=DEV), torch.zeros(d, device=DEV)
    g[M - 1, d - 1] = -9.0
    ctx = make_ctx(d, M, 2, B.NORM_SUB, seed=3)
    _check_encode_decode(ctx, 1, g, gref, gref, "many workers")
    rows = ctx.workspace[:4 * 4096 * M].view(torch.float32).view(4096, M)
    assert int((rows.amax(dim=1) > 0).sum()) >= d // 4096
    ctx.close()
