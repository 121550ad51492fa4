"""Decode and average of packed words of any pattern -- the one that no encoder writes, a sign without a level, decodes to 0 -- under
scales of every kind: ordinary, zero, negative, subnormal, and among eight workers one that is infinite, where two bits leave the
signed units for the table of values; one to seventeen workers, short and long rows of any length, bit for bit against the oracle."""
import numpy as np
import pytest
import torch

from gpu_util import DEV, make_ctx, oracle_cfg
from oracle import tng_oracle as O
from paper_1901_08227_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 7, 8, 9, 17])
@pytest.mark.parametrize("d", [1, 1023, 4097, (1 << 20) + 5, 1 << 21])
@pytest.mark.parametrize("bits,norm", [(2, B.NORM_SUB), (2, B.NORM_QUOT), (2, B.NORM_MEAN), (4, B.NORM_SUB)])
def test_words_of_any_pattern(M, d, bits, norm):
    rng = np.random.default_rng(d + M)
    ctx = make_ctx(d, M, bits, norm, seed=3)
    codes = rng.integers(0, 2 ** 32, (M, ctx.words), dtype=np.uint64).astype(np.uint32)
    gref = rng.standard_normal(d).astype(np.float32)
    means = rng.standard_normal(M).astype(np.float32)
    cfg = oracle_cfg(ctx)
    if norm == B.NORM_MEAN:
        held = torch.from_numpy(means).to(DEV)
        ctx.set_worker_means(held)
    for kind in ("ordinary", "odd", "infinite")[:3 if bits == 2 else 2]:
        scales = np.exp(rng.standard_normal(M)).astype(np.float32)
        if kind == "odd":
            scales[:] = np.array([0.0, 1e-40, -2.5, 3e38, 1.0], dtype=np.float32)[np.arange(M) % 5]
        elif kind == "infinite":
            scales[M // 2] = np.inf
        vbar = torch.empty(d, device=DEV)
        ctx.decode_aggregate(torch.from_numpy(codes.view(np.int32)).to(DEV), torch.from_numpy(scales).to(DEV), torch.from_numpy(gref).to(DEV), vbar)
        with np.errstate(invalid="ignore", over="ignore"):
            want = O.decode_aggregate(cfg, codes, scales, gref, d, None, means)
            if kind == "infinite":  # level 0 is 0 under any scale (the oracle's product with it is no number)
                finite = scales.copy()
                finite[M // 2] = 0.0
                level, _ = O.unpack(codes[M // 2], d, bits)
                zeros = O.decode_aggregate(cfg, codes, finite, gref, d, None, means)
                want = np.where(level == 0, zeros, want)
        assert np.array_equal(vbar.cpu().numpy(), want, equal_nan=True), kind
    ctx.close()
