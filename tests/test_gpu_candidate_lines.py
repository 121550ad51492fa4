"""The slots' first lines and what lies behind them, for one to nine workers (the quantise pass takes eight tiles of workers at a time: of
one worker, of two, four, five or eight): tiles that hold counts around what the line has room for, of rows with a bound (two entries to a
word) and of rows without one, in the last tiles of rows whose number of tiles is no multiple of what a wavefront or a workgroup takes,
next to rows too dense for slots, against the oracle."""
import pytest
import torch

from gpu_util import DEV
from paper_1901_08227_amd import binding as B
from test_gpu_candidates_ragged import check

pytestmark = pytest.mark.gpu

COUNTS = (0, 1, 2, 30, 31, 32, 33, 61, 62, 63, 64, 65, 94, 95, 96, 125, 126, 127, 128, 129, 1024)


@pytest.mark.parametrize("M,tiles", [(1, 65536 + 13), (2, 32768 + 7), (3, 21846 + 4), (4, 16384 + 3), (5, 13108 + 2), (8, 8192 + 5), (9, 7282 + 1)])
def test_counts_around_the_ends_of_a_line(M, tiles):
    d = 1024 * tiles
    gen = torch.Generator(device=DEV).manual_seed(M)
    v = torch.zeros((M, tiles, 1024), device=DEV)
    for m in range(M):
        form = (m + M) % 3  # 0: a bound and elements of every size below it, 1: no bound, 2: a bound and a scale far beyond it
        if form != 1:
            v[m, ::128, 0] = 1.0  # every tile of the sample: its largest element bounds the row's
        if m == 4:
            v[m] = torch.randn((tiles, 1024), generator=gen, device=DEV)  # too dense
            continue
        for i, k in enumerate(COUNTS):
            for t in (tiles - 1 - i - i // 100, 1 + 5 * i + 31 * m):
                t += 1 if t % 128 == 0 else 0
                at = torch.randperm(1024, generator=gen, device=DEV)[:k]
                size = torch.rand(k, generator=gen, device=DEV) * 0.5 + 0.5 if form == 0 else torch.randn(k, generator=gen, device=DEV)
                v[m, t] = 0.0
                v[m, t, at] = size * (torch.randint(0, 2, (k,), generator=gen, device=DEV).float() * 2 - 1)
        if form == 2:
            v[m, 77, 5] = 9.0
    v = v.view(M, d)
    gref = torch.randn(d, generator=gen, device=DEV) * (2.0 ** -20)
    check(M, d, B.NORM_SUB, (v + gref).contiguous(), gref, 6)
