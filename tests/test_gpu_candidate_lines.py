"""The slots' first lines and what lies behind them, for one to nine workers (the quantise pass takes eight rows at a time: eight tiles of
one worker, two to four tiles of four or two, a tile of eight): tiles that hold exactly as many candidates as the line, the slot and less or
more than that have room for, of rows with a bound (two entries to a word) and of rows without one, in the last tiles of rows whose number
of tiles is no multiple of what a wavefront or a workgroup takes.  "bound": every row has a bound, so that whole groups of workers go
through the scale pass's loop without branches; "mixed": rows without one and rows too dense for slots next to them.  Against the oracle."""
import numpy as np
import pytest
import torch

from gpu_util import DEV
from oracle import tng_oracle as O
from paper_1901_08227_amd import binding as B
from test_candidate_bound import c1_of
from test_gpu_candidates_ragged import check

pytestmark = pytest.mark.gpu

# a line holds 31 entries of a word or 62 of half a word, a slot 127 or 126
COUNTS = (0, 1, 2, 30, 31, 32, 33, 61, 62, 63, 64, 65, 94, 95, 96, 125, 126, 127, 128, 129, 1024)
IT = 6


def candidates(seed, m, tile, v, r_hat):
    """How many elements of the tile are candidates, from their draws (the sum in binary64: its rounding matters to draws near it only)."""
    draws = O.quant_draw_words(seed, IT, m, 1024, first=1024 * tile).astype(np.float32).astype(np.float64)
    bar = 2.0 ** 40 * (v != 0) if r_hat == 0 else np.abs(v).astype(np.float64) * float(c1_of(np.float32(r_hat)))
    return int(np.sum(draws < bar + 258.0))


@pytest.mark.parametrize("M,tiles,rows", [(1, 65536 + 13, "mixed"), (2, 32768 + 7, "bound"), (3, 21846 + 4, "mixed"), (4, 16384 + 3, "mixed"),
                                          (5, 13108 + 2, "mixed"), (8, 8192 + 5, "mixed"), (9, 7282 + 1, "mixed"), (1, 65536 + 9, "bound"),
                                          (4, 16384 + 1, "bound"), (5, 13108 + 5, "bound"), (8, 8192 + 3, "bound"), (9, 7282 + 3, "bound")])
def test_counts_around_the_ends_of_a_line(M, tiles, rows):
    d = 1024 * tiles
    gen = torch.Generator(device=DEV).manual_seed(M)
    v = torch.zeros((M, tiles, 1024), device=DEV)
    gref = (torch.randn(d, generator=gen, device=DEV) * (2.0 ** -20)).view(tiles, 1024)
    last = [t for t in range(tiles - 1, 0, -1) if t % 128 != 0][:len(COUNTS)]
    for m in range(M):
        form = (m + M) % 3 if rows == "mixed" else m % 2 * 2  # 0: a bound, 1: no bound, 2: a bound and a scale far beyond it
        if form != 1:
            v[m, ::128, 0] = 1.0  # every tile of the sample: its largest element bounds the row's
        if rows == "mixed" and m == 4:
            v[m] = torch.randn((tiles, 1024), generator=gen, device=DEV)  # too dense
            continue
        for i, k in enumerate(COUNTS):
            for t in (last[i], 1 + 5 * i + 31 * m):
                t += 1 if t % 128 == 0 else 0
                at = torch.randperm(1024, generator=gen, device=DEV)[:k]
                size = torch.rand(k, generator=gen, device=DEV) * 1.75 + 1.25  # above the bound: candidates whatever their draws
                v[m, t] = 0.0
                v[m, t, at] = size * (torch.randint(0, 2, (k,), generator=gen, device=DEV).float() * 2 - 1)
        if form == 2:
            v[m, 77, 5] = 9.0
        g = v[m] + gref
        for i, k in enumerate(COUNTS):
            held = (g[last[i]] - gref[last[i]]).cpu().numpy()
            assert candidates(d, m, last[i], held, 0.0 if form == 1 else (g[::128] - gref[::128]).max().item()) == k
    v = v.view(M, d)
    gref = gref.view(d)
    check(M, d, B.NORM_SUB, (v + gref).contiguous(), gref, IT)
