"""The ternary coder that reads the gradients once, on rows that are not whole tiles of 1024 coordinates: the ragged
last tile in workgroups of its own next to 1 to 16 workers per workgroup, with the slots in use, with single rows too
dense for them, and with the call left to the ordinary quantiser, against the oracle."""
import numpy as np
import pytest
import torch

from gpu_util import DEV, buffers, make_ctx, oracle_cfg, say, u32
from oracle import tng_oracle as O
from paper_1901_08227_amd import binding as B
from test_gpu_candidates import _encode_one, _inputs

pytestmark = pytest.mark.gpu


def check(M, d, norm, g, gref, it, scale=B.SCALE_MAX):
    say(f"candidates d={d} M={M} norm={norm} scale={scale}")
    ctx = make_ctx(d, M, 2, norm, seed=d, scale=scale)
    buf = buffers(ctx)
    ctx.normalize_encode(it, g, gref, buf["codes"], buf["scales"])
    ctx.decode_aggregate(buf["codes"], buf["scales"], gref, buf["vbar"])
    torch.cuda.synchronize()
    cfg = oracle_cfg(ctx)
    ctx.close()
    rh, codes, scales = gref.cpu().numpy(), u32(buf["codes"]), buf["scales"].cpu().numpy()
    for m in range(M):
        want, R = _encode_one(cfg, it, m, g[m].cpu().numpy(), rh, rh)
        assert scales[m] == R and np.array_equal(codes[m], want), f"worker {m}: scale {scales[m]} of {R}"
    assert np.array_equal(buf["vbar"].cpu().numpy(), O.decode_aggregate(cfg, codes, scales, rh, d, rh, None))


@pytest.mark.parametrize("M,d,norm", [(1, (1 << 26) + 1, B.NORM_SUB), (2, (1 << 25) + 1023, B.NORM_SUB),
                                      (3, (1 << 25) + 514, B.NORM_SUB), (5, (1 << 24) + 4099, B.NORM_SUB),
                                      (9, (1 << 23) + 4, B.NORM_SUB), (17, (1 << 22) + 255, B.NORM_SUB)])
def test_ragged_rows(M, d, norm):
    g, gref, _ = _inputs(M, d, seed=M)
    g[M - 1, d - 1] += 3.0 * (g[M - 1] - gref).abs().max()  # the last worker's scale is set in the ragged tile
    check(M, d, norm, g, gref, 4)


@pytest.mark.parametrize("dense", [(2,), tuple(range(33))])
def test_dense_rows(dense):
    M, d = 33, (1 << 21) + 333
    g, gref, _ = _inputs(M, d, seed=5)
    for m in dense:
        g[m] = gref + torch.randn(d, device=DEV, generator=torch.Generator(device=DEV).manual_seed(m))
    check(M, d, B.NORM_SUB, g, gref, 4)


@pytest.mark.parametrize("M,d,norm", [(4, 1 << 24, B.NORM_SUB), (5, (1 << 24) + 4096 * 3, B.NORM_NONE), (9, 1 << 23, B.NORM_SUB),
                                      (20, (1 << 22) + 1027, B.NORM_SUB), (8, (1 << 23) + 4092, B.NORM_NONE)])
def test_l2_scale(M, d, norm):
    g, gref, _ = _inputs(M, d, seed=M)
    gen = torch.Generator(device=DEV).manual_seed(M)
    v = g - gref
    v[0, 1024 * 77:1024 * 79] *= 1e6  # nearly the whole norm in two tiles that the sample does not visit: they overflow
    v[1] = 0.0
    v[2] = (torch.rand(d, generator=gen, device=DEV) - 0.5) * 1e-38  # a norm near the smallest normal number
    v[3, 5000:] = 0.0  # a row of few elements that the sample sees: too dense where it is not zero
    check(M, d, norm, (v + gref if norm == B.NORM_SUB else v).contiguous(), gref, 2, B.SCALE_L2)


def test_l2_scale_outside_the_sample():
    # rows that are zero wherever the sample looks: no bound, every non-zero element is a candidate and most tiles overflow
    M, d = 8, 1 << 23
    v = torch.randn((M, d), device=DEV, generator=torch.Generator(device=DEV).manual_seed(1))
    v.view(M, -1, 1024)[:, ::128] = 0.0
    check(M, d, B.NORM_NONE, v, v[0].clone(), 2, B.SCALE_L2)


@pytest.mark.parametrize("d", [(1 << 24) + 4096 + 3 * 1024, (1 << 24) + 1024 + 7])
def test_l2_slots_filled_to_their_edges(d):
    # chunks that hold exactly k candidates (the rows are zero where the sample looks, so every other element is one): the
    # quantise pass takes the first 32 at once, and all of them in a loop where there are more; whole tiles behind the last whole
    # chunk have no slots
    M = 5
    gen = torch.Generator(device=DEV).manual_seed(9)
    v = torch.zeros((M, d), device=DEV)
    for m in range(M):
        for i, k in enumerate((1, 2, 31, 32, 33, 64, 127, 128, 129)):
            at = torch.randperm(4096, generator=gen, device=DEV)[:k] + 4096 * (1 + 32 * i + 5 * m)
            v[m, at] = torch.randn(k, generator=gen, device=DEV)
        v[m, -3500:] = 2 * torch.randn(3500, generator=gen, device=DEV)
    for m in range(M):
        whole = v[m, :d // 1024 * 1024].view(-1, 1024)
        whole[::128] = 0.0
    check(M, d, B.NORM_SUB, v, torch.zeros(d, device=DEV), 7, B.SCALE_L2)


def test_l2_slots_filled_tile_by_tile():
    # candidates per tile of a chunk: up to 48 wait in the staging area for the tiles behind, a tile finds room for 128, a slot holds
    # 448 with odd numbers rounded up to pairs; one too many of any and the chunk is coded from g
    M, d = 5, 1 << 24
    gen = torch.Generator(device=DEV).manual_seed(10)
    v = torch.zeros((M, d), device=DEV)
    fills = ((48, 128, 0, 0), (48, 129, 0, 0), (49, 128, 1, 0), (0, 0, 0, 128), (0, 0, 0, 176), (0, 0, 0, 177), (112, 112, 112, 112),
             (112, 112, 112, 113), (111, 111, 111, 111), (111, 111, 111, 113), (1, 1, 1, 1), (49, 49, 49, 49), (47, 2, 0, 31), (17, 17, 1, 0))
    for m in range(M):
        for i, fill in enumerate(fills):
            for t, k in enumerate(fill):
                at = torch.randperm(1024, generator=gen, device=DEV)[:k] + 4096 * (1 + 32 * i + 5 * m) + 1024 * t
                v[m, at] = torch.randn(k, generator=gen, device=DEV)
    check(M, d, B.NORM_SUB, v, torch.zeros(d, device=DEV), 8, B.SCALE_L2)


def test_l2_scale_of_rows_that_are_not_zero_in_runs():
    # three tiles in a hundred hold everything: some fifty candidates in each, hundreds where two or more share a chunk
    M, d = 16, 1 << 22
    gen = torch.Generator(device=DEV).manual_seed(5)
    v = torch.randn((M, d), generator=gen, device=DEV)
    v.view(M, -1, 1024).mul_((torch.rand((M, d // 1024, 1), generator=gen, device=DEV) < 0.03).float())
    check(M, d, B.NORM_SUB, v, torch.zeros(d, device=DEV), 9, B.SCALE_L2)


# Rows that are zero where the sample looks: every other element is a candidate.  share of the groups of four tiles hold `tiles` tiles
# with `each` candidates (and the rest nothing); the slots are used unless more than one per fifty tiles overflow.
@pytest.mark.parametrize("scale,share,tiles,each,used", [
    (B.SCALE_L2, 0.04, 1, 1024, 1), (B.SCALE_L2, 0.075, 1, 1024, 1), (B.SCALE_L2, 0.09, 1, 1024, 0), (B.SCALE_L2, 0.3, 4, 112, 1),
    (B.SCALE_L2, 0.3, 4, 113, 0), (B.SCALE_MAX, 0.04, 1, 1024, 1), (B.SCALE_MAX, 0.04, 3, 1024, 0), (B.SCALE_MAX, 0.3, 4, 127, 1)])
def test_which_rows_the_slots_are_used_for(scale, share, tiles, each, used):
    M, d = 16, 1 << 22
    gen = torch.Generator(device=DEV).manual_seed(17)
    v = torch.zeros((M, d // 4096, 4, 1024), device=DEV)
    groups = torch.arange(d // 4096, device=DEV)
    groups = groups[groups % 32 != 0]
    for m in range(M):
        some = groups[torch.randperm(len(groups), generator=gen, device=DEV)[:int(share * (d // 4096))]]
        v[m, some, :tiles, :each] = torch.randn((len(some), tiles, each), generator=gen, device=DEV)
    v = v.view(M, d)
    check(M, d, B.NORM_SUB, v, torch.zeros(d, device=DEV), 3, scale)
    ctx = make_ctx(d, M, 2, B.NORM_SUB, seed=d, scale=scale)
    buf = buffers(ctx)
    ctx.normalize_encode(3, v, torch.zeros(d, device=DEV), buf["codes"], buf["scales"])
    four_bits = B.TngConfig.from_buffer_copy(ctx.cfg)
    four_bits.bits = 4
    at = B.tng_workspace_bytes(four_bits)  # without slots: where they begin, the vote in front
    assert int(ctx.workspace[at:at + 4].view(torch.int32)[0]) == used
    ctx.close()


@pytest.mark.parametrize("scale", [B.SCALE_MAX, B.SCALE_L2])
def test_rows_below_the_smallest_normal_number(scale):
    # Rows that are zero where the sample looks (no bound: every non-zero element is a candidate) and hold a hundred values of 0x7FF
    # or 0x1FFF units of 2^-149 per tile (a few dozen per chunk with the l2 scale) under a scale of 2^-124: of 2^24 draws 512 or
    # 2048 code non-zero only by the bits that an entry has no room for, so hundreds of elements of a row tell.
    M, d, per = 4, 1 << 24, 100 if scale == B.SCALE_MAX else 25
    gen = torch.Generator(device=DEV).manual_seed(13)
    bits = torch.zeros((M, d // 1024, 1024), dtype=torch.int32, device=DEV)
    for m in range(M):
        at = torch.rand((d // 1024, 1024), generator=gen, device=DEV).topk(per, dim=1).indices
        sign = torch.randint(0, 2, at.shape, generator=gen, device=DEV, dtype=torch.int32) << 31
        bits[m].scatter_(1, at, sign | (0x7FF, 0x1FFF, 0x5FF, 0x1801)[m])
    bits[:, ::128] = 0
    bits[:, 5, 77] = (127 - 124) << 23
    v = bits.view(M, d).view(torch.float32)
    check(M, d, B.NORM_SUB, v, torch.zeros(d, device=DEV), 3, scale)


@pytest.mark.parametrize("M,d,norm", [(10, 1 << 23, B.NORM_SUB), (9, 1 << 23, B.NORM_SUB), (20, (1 << 22) + 1029, B.NORM_SUB), (10, 1 << 23, B.NORM_NONE)])
def test_groups_of_five_workers(M, d, norm):
    g, gref, _ = _inputs(M, d, seed=M)
    check(M, d, norm, g, gref, 4)
