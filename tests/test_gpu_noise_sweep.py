"""The arithmetic of the generated Gaussian noise over practically all arguments: 2^28 pairs of draws, so that each of the 2^24
values of the radius's word and of the angle's word comes 16 times on average, the ends and the edges of the quadrants
among them, against binary64."""
import math

import pytest
import torch

from gpu_util import DEV, make_ctx, say
from paper_1901_08227_amd import binding as B

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


def test_every_argument_against_binary64():
    """At x = 1 the gradient of the chain is 0, so with variance 1 what comes out is the noise itself.  Its radius is within
    2.14 units of 2^-24 of its size, sine and cosine within 0.75 units, their product is rounded once (one unit of its size
    at most); 0.01 units of the radius stand for products of these."""
    d, chunk = 1 << 28, 1 << 24
    ctx = make_ctx(d, 1, 2, B.NORM_NONE, seed=77, problem=B.PROB_ROSENBROCK)
    ctx.set_noise_variance(1.0)
    x, g = torch.ones(d, device=DEV), torch.empty((1, d), device=DEV)
    words = torch.empty(chunk, dtype=torch.int32, device=DEV)
    radius_seen = torch.zeros(1 << 24, dtype=torch.bool, device=DEV)
    angle_seen = torch.zeros(1 << 24, dtype=torch.bool, device=DEV)
    worst = torch.zeros((), dtype=torch.float64, device=DEV)
    for it in (0, 1):
        ctx.local_grad(it, x, g)
        for first in range(0, d, chunk):
            ctx.rng_draws(it, 0, 2, first, chunk, words)
            k = ((words.to(torch.int64) & 0xFFFFFFFF) >> 8).view(-1, 2)
            radius_seen[k[:, 0]] = True
            angle_seen[k[:, 1]] = True
            r = torch.sqrt(-2.0 * torch.log((k[:, 0] + 1).to(torch.float64) * U))
            turn = k[:, 1].to(torch.float64) * (2.0 * math.pi * U)
            pair = g[0, first:first + chunk].view(-1, 2).to(torch.float64)
            for got, part in ((pair[:, 0], torch.cos(turn)), (pair[:, 1], torch.sin(turn))):
                want = r * part
                bound = U * (3.14 * want.abs() + 0.76 * r)
                over = torch.where(bound > 0, (got - want).abs() / bound, got.abs() * math.inf)
                worst = torch.maximum(worst, torch.nan_to_num(over, nan=0.0).max())
                assert bool(torch.isfinite(got).all())
        say(f"noise sweep: iteration {it}, worst error {worst.item():.3f} of its bound")
    ctx.close()
    assert worst.item() <= 1.0
    assert radius_seen.sum() > 0.9999 * (1 << 24) and angle_seen.sum() > 0.9999 * (1 << 24)
    top = (1 << 24) - 1
    assert radius_seen[0] and radius_seen[top]  # the largest radius, and u1 = 1: radius 0
    for quadrant in range(4):  # t = -1/2 and the last t below 1/2; the middle of the quadrant
        edge = quadrant * (1 << 22)
        for at in (edge, (edge + (1 << 21)) & top, (edge + (1 << 21) - 1) & top):
            assert angle_seen[at]
