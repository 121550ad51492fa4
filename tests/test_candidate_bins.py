"""The entries of the ternary coder's slots for rows whose sample bounds their scale (R^ <= R), half a word each: x = u R^ / |v| in
one of 126 bins, against the bins of rho = R^ / R from either side.  Below the lower one the level [u < fl(|v| fl(1 / R))] must be 1, above the
upper one 0, for every scale from R^ on and with the reciprocal one unit off either way; what is left for the value itself
are one or two bins.  Bin 0 (u = 0, or no number) decides nothing."""
import numpy as np
import pytest

from test_candidate_bound import c1_of

F32 = np.float32


def bin_of(x):
    with np.errstate(invalid="ignore", over="ignore"):  # (through binary64: which side of a whole number one rounding more leaves it on does not matter)
        y = np.fmin(np.fmax((x.astype(np.float64) * 44 + 1).astype(F32), (x.astype(np.float64) * 208 - 81).astype(F32)), F32(126.0))
    return np.where(x > 0, np.where(x > 0, y, 0).astype(np.uint32), np.uint32(0))


def entry_bin(absv, word, r_hat, rcp_ulps):
    a = (absv.view(np.uint32) & np.uint32(0x7FFFFC00)).view(F32)
    with np.errstate(divide="ignore", over="ignore", invalid="ignore"):
        rc = (F32(1.0) / (a * c1_of(r_hat)).astype(F32)).astype(F32)
        for _ in range(abs(rcp_ulps)):
            rc = np.nextafter(rc, F32(np.inf) if rcp_ulps > 0 else F32(0.0)).astype(F32)
        return bin_of(((word & np.uint32(0xFFFFFF00)).astype(F32) * rc).astype(F32))


def limits(r_hat, R):
    with np.errstate(divide="ignore", over="ignore", invalid="ignore"):
        rho = (r_hat / R).astype(F32)
        below, above = bin_of((rho * F32(1.0 - 2.0 ** -18)).astype(F32)), bin_of((rho * F32(1.0 + 2.0 ** -12)).astype(F32))
    return below, np.where(rho >= 0, above, np.uint32(126))


def level(word, absv, R):
    with np.errstate(divide="ignore", over="ignore", invalid="ignore"):
        return (word >> np.uint32(8)).astype(np.float64) * 2.0 ** -24 < (absv * (F32(1.0) / R).astype(F32)).astype(F32).astype(np.float64)


@pytest.mark.parametrize("r_hat", [2.0 ** -90, 1e-3, 1.0, 3e7, 2.0 ** 126])
@pytest.mark.parametrize("values", ["below the bound", "tiny", "subnormal", "beyond"])
def test_bins_decide_from_the_safe_side(r_hat, values):
    rng = np.random.default_rng(31)
    n = 200_000
    r_hat = np.full(n, r_hat, dtype=F32)
    if values == "subnormal":
        absv = rng.integers(0, 1 << 23, n).astype(np.uint32).view(F32)
    elif values == "tiny":
        absv = (r_hat * 10.0 ** rng.uniform(-12, -3, n)).astype(F32)
    elif values == "beyond":  # larger than anything in the sample
        absv = np.minimum(r_hat * 10.0 ** rng.uniform(0, 3, n), 3e38).astype(F32)
    else:
        absv = (r_hat * rng.uniform(0, 1, n)).astype(F32)
    k = (rng.integers(0, 2 ** 24, n) >> rng.integers(0, 24, n)).astype(np.uint32)  # draws of every size, u = 0 among them
    word = (k << np.uint32(8)) | rng.integers(0, 256, n).astype(np.uint32)
    # scales from R^ on: on both sides of |v| / u and anywhere
    with np.errstate(divide="ignore", over="ignore", invalid="ignore"):
        at = absv.astype(np.float64) * 2.0 ** 24 / np.maximum(k, 1)
        R = np.where(rng.random(n) < 0.7, at * (1.0 + rng.choice([-1.0, 1.0], n) * 2.0 ** rng.uniform(-24, -2, n)),
                     r_hat * 10.0 ** rng.uniform(0, 3, n)).astype(F32)
    R = np.where(np.isfinite(R), np.maximum(np.maximum(R, r_hat), absv), F32(np.inf)).astype(F32)
    lv = level(word, absv, R)
    below, above = limits(r_hat, R)
    for ulps in (-1, 0, 1):
        b = entry_bin(absv, word, r_hat, ulps)
        assert b.max() <= 126  # (127 is the mark of no entry)
        one, zero = (b >= 1) & (b < below), b > above
        assert np.all(lv[one]), "decided 1 where the level is 0"
        assert not np.any(lv[zero]), "decided 0 where the level is 1"
        assert np.all(b[k == 0] == 0)


def test_few_elements_are_left_for_their_value():
    rng = np.random.default_rng(37)
    n = 400_000
    r_hat, x = np.ones(n, dtype=F32), rng.uniform(0, 1, n)
    absv = rng.uniform(0.2, 1.0, n).astype(F32)
    word = np.minimum(x * absv.astype(np.float64) * 2.0 ** 32, 2.0 ** 32 - 1).astype(np.uint32)
    # a bin is 1 / 208 of x above 1 / 2 and 1 / 44 below; two of them where rho lies on their border, and the cuts' 2^-12
    for rho, most in ((0.95, 1.2 / 208), (0.75, 2.2 / 208), (0.55, 1.2 / 208), (0.3, 1.2 / 44), (0.01, 1.2 / 44)):
        below, above = limits(r_hat, np.full(n, 1.0 / rho, dtype=F32))
        b = entry_bin(absv, word, r_hat, 0)
        assert np.mean((b <= above) & ~((b >= 1) & (b < below))) < most
