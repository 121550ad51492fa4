"""Quantise, decode and update in one launch (tng_step): either kernel at the edges of its tiles (256 coordinates per
wavefront or workgroup), of its groups of workers (4 and 8) and of the rule that chooses, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import tng_oracle as O
from gpu_util import DEV, buffers, make_ctx, oracle_cfg, oracle_step_threaded, u32
from paper_1901_08227_amd import binding as B
from test_gpu_codec import _inputs

pytestmark = pytest.mark.gpu

ALL = [(n, B.SCALE_MAX) for n in (B.NORM_NONE, B.NORM_SUB, B.NORM_QUOT, B.NORM_COMB, B.NORM_MEAN)] + [(B.NORM_SUB, B.SCALE_L2)]


@pytest.mark.parametrize("d,M", [(1, 1), (2, 3), (255, 64), (256, 17), (1023, 5), (1028, 16), (5001, 33), (70001, 64),
                                 (1 << 18, 8), ((1 << 18) + 1, 8), ((1 << 18) + 254, 9), ((1 << 18) + 1024, 16),
                                 ((1 << 18) + 257, 17), ((1 << 19) + 3, 7), (4099, 65)])
def test_step_equals_the_oracle(d, M):
    for i, (norm, scale) in enumerate(ALL):
        bits = 2 + 2 * ((i + d) % 2)
        g, gref, gref2 = _inputs(M, d, seed=d + i)
        g, gref, gref2 = g.to(DEV), gref.to(DEV).clone(), gref2.to(DEV)
        if M > 2:
            g[2] = gref  # a worker with nothing to send (Eq. 1): its scale is 0
        ctx = make_ctx(d, M, bits, norm, seed=d, lr=0.05, ref_period=1, scale=scale, problem=B.PROB_EXTERNAL)
        if norm == B.NORM_COMB:
            ctx.set_second_reference(gref2)
        if norm == B.NORM_MEAN:
            means = torch.zeros(M, device=DEV)
            ctx.set_worker_means(means)
        buf = buffers(ctx)
        w = torch.linspace(-1.0, 1.0, d, device=DEV)
        want = O.step(oracle_cfg(ctx), 3, w.cpu().numpy(), gref.cpu().numpy(), g.cpu().numpy(), gref2.cpu().numpy())
        ctx.step(3, w, gref, g, buf["codes"], buf["scales"], buf["vbar"])
        torch.cuda.synchronize()
        got = (w.cpu().numpy(), gref.cpu().numpy(), u32(buf["codes"]), buf["scales"].cpu().numpy(), buf["vbar"].cpu().numpy())
        for name, a, b in zip(("iterate", "reference", "codes", "scales", "average"), got, want):
            assert np.array_equal(a, b), f"d={d} M={M} norm={norm} scale={scale} bits={bits}: {name}"
        ctx.close()


# Partial maxima (about d / 4096 rows of M) on both sides of where they are fetched as float4 (1024, workers a power of two)
# and of where a launch of their own reduces them (8192 up to d = 2^20, then 2048).
@pytest.mark.parametrize("d,M", [(1 << 18, 16), ((1 << 18) + 1024, 16), (70001, 64), (1 << 20, 4), ((1 << 20) + 5, 4), ((1 << 17) + 1, 64),
                                 (1 << 20, 13), ((1 << 20) + 1, 13), (1 << 20, 32), (400003, 12), (1 << 22, 2), ((1 << 21) + 4, 4)])
def test_step_scales_from_many_partial_maxima(d, M):
    rng = torch.Generator().manual_seed(d + M)
    g = torch.randn(M, d, generator=rng) * 0.01
    at = torch.randint(0, d, (M,), generator=rng)
    at[0], at[M - 1] = d - 1, 0
    g[torch.arange(M), at] = torch.linspace(-3.0, 4.0, M) + 0.125  # a worker's largest element: one partial maximum has it
    gref = torch.randn(d, generator=rng) * 0.01
    print(f"partial maxima d={d} M={M}", flush=True)
    ctx = make_ctx(d, M, 2, B.NORM_SUB, seed=d, lr=0.05, ref_period=1, problem=B.PROB_EXTERNAL)
    buf = buffers(ctx)
    w, gr, gd = torch.linspace(-1.0, 1.0, d, device=DEV), gref.to(DEV), g.to(DEV)
    want = oracle_step_threaded(oracle_cfg(ctx), 3, w.cpu().numpy(), gref.numpy(), g.numpy())
    ctx.step(3, w, gr, gd, buf["codes"], buf["scales"], buf["vbar"])
    torch.cuda.synchronize()
    got = (w.cpu().numpy(), gr.cpu().numpy(), u32(buf["codes"]), buf["scales"].cpu().numpy(), buf["vbar"].cpu().numpy())
    for name, a, b in zip(("iterate", "reference", "codes", "scales", "average"), got, want):
        assert np.array_equal(a, b), f"d={d} M={M}: {name}"
    ctx.close()


# The scale pass held to 2048 partial maxima (workers a power of two, beyond d = 2^20): a workgroup walks one to four tiles,
# the last of them short, and the ragged tile has a row of its own; M = 7 keeps the launch that reduces them.
@pytest.mark.parametrize("d,M", [((1 << 20) + 1028, 8), (1500003, 8), (1 << 22, 8), (1500004, 7)])
def test_step_scales_from_a_scale_pass_of_few_workgroups(d, M):
    test_step_scales_from_many_partial_maxima(d, M)


# ... and to half as many workgroups as tiles up to 1.6 tiles for each of those 2048 / M, of two tiles each (the last one short).
@pytest.mark.parametrize("d", [(1 << 20) + 4096, 1100000, 1250003, 1671168, 1671169])
def test_step_scales_from_a_scale_pass_of_half_the_tiles(d):
    test_step_scales_from_many_partial_maxima(d, 8)


# 2048 to 8192 partial maxima of a power of two workers, eight float4 a thread of which the last ones repeat: whole workgroups only,
# and a last one that is not (it reduces the same maxima by the other path).
@pytest.mark.parametrize("d", [(1 << 19) + 4096, 700416, 700003, (1 << 20) - 4])
def test_step_scales_from_partial_maxima_requested_ahead_of_the_rows(d):
    test_step_scales_from_many_partial_maxima(d, 16)
