"""The covariance of a witness pair, extended from length to length with means
kept by the recurrence, against a direct product with the same means: its error
grows with the offset of the series over the windows' deviations.  The guard
that k_advance leaves between such a correlation and the threshold must cover
it.  The recurrences are those of the kernel, in FP64; the guard's constants
are read from its source."""

import math
import os
import re

import numpy as np
import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2304_01660_amd", "csrc", "kernels.hip")


def _constant(name, default):
    m = re.search(r"constexpr double %s = ([^;]*);" % name, open(SRC).read())
    return float.fromhex(m.group(1)) if m and "x" in m.group(1) else float(m.group(1)) if m else default


def _chains(kind, offset, minL, maxL, pairs, seed):
    """|rho by the chain - rho by a direct product|, and the pairs' contrasts
    |mu| / sigma, at the last length."""
    rng = np.random.default_rng([seed, minL, maxL])
    n = 40000
    x = np.cumsum(rng.standard_normal(n)) if kind == "rw" else rng.standard_normal(n)
    T = x + offset
    i, j = rng.integers(0, n - maxL, pairs), rng.integers(0, n - maxL, pairs)

    def start(p):
        w = T[p[:, None] + np.arange(minL)]
        mu = np.add.accumulate(w, axis=1)[:, -1] / minL
        return mu, ((w - mu[:, None]) ** 2).sum(1) / minL, w - mu[:, None]

    mi, vi, wi = start(i)
    mj, vj, wj = start(j)
    C = (wi * wj).sum(1)
    for m in range(minL + 1, maxL + 1):
        f = (m - 1.0) / m
        ti, tj = T[i + m - 1], T[j + m - 1]
        C = C + f * (ti - mi) * (tj - mj)
        di, dj = mi - ti, mj - tj
        mi, vi = ((m - 1.0) * mi + ti) / m, f * (vi + di * di / m)
        mj, vj = ((m - 1.0) * mj + tj) / m, f * (vj + dj * dj / m)
    k = np.arange(maxL)
    direct = ((T[i[:, None] + k] - mi[:, None]) * (T[j[:, None] + k] - mj[:, None])).sum(1)
    si, sj = np.sqrt(vi), np.sqrt(vj)
    return np.abs(C - direct) / (maxL * si * sj), np.abs(mi) / si + np.abs(mj) / sj


@pytest.mark.parametrize("kind", ["rw", "noise"])
@pytest.mark.parametrize("offset", [0.0, 1e3, 1e6, 1e8, 1e10])
@pytest.mark.parametrize("minL, maxL", [(8, 40), (64, 192), (128, 256), (16, 400)])
def test_the_guard_covers_the_chained_covariance(kind, offset, minL, maxL):
    err, contrast = _chains(kind, offset, minL, maxL, 4000, 7)
    base, drift = _constant("WIT_GUARD", 0.0), _constant("WIT_DRIFT", 0.0)
    guard = np.maximum(base, drift * maxL * 2.0 ** -53 * (contrast + 2.0 * math.sqrt(maxL)))
    assert np.all(err < guard), (err.max(), guard[err.argmax()])
    # ... and stays the constant one for series near zero
    if offset == 0.0:
        assert guard.max() == base
