"""The mixed form's pair loop where its rounds change: two staged sources a round
with the next ones read ahead, so odd and even numbers of steps, a single one,
stages of 256 filled exactly, by one less and by one more, and chunks whose lanes
hold one to four targets.  One leaf (depth 0) or four that all touch (depth 1):
no far field, every pair is an FP32 one.

Reference: the oracle's plain sum, particle by particle, within what FP32 pairs
may be off.  In leaf widths, with r a pair's distance, F its term |d| (1 -
exp(-c r^2)) / r^2, c = w^2 / (2 sigma^2) and e = 2^-24:
* a coordinate carries the rounding of source and target positions (e / 4 each),
  of the source's shift to the target leaf and of the difference (e each):
  2.5 e per axis, and the term's derivative is at most c;
* the exponential is off by one ulp (2 e) next to 1, so 1 - exp(..) is off by
  absolute 2 e beside its own rounding, and 4 e / r in the term covers it;
* the other operations and a sum of n terms round by (n + 16) e F.
A pair left out or taken twice is off by F itself, more than the whole bound.
"""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _built():
    oracle.build()


@pytest.mark.parametrize("L", [0, 1])
@pytest.mark.parametrize("n", [2, 3, 5, 16, 17, 33, 48, 49, 64, 65, 127, 130, 192, 255, 256, 257, 300, 513, 700, 1030])
def test_pair_rounds(n, L):
    x, y, g = workloads.uniform_square(n, 70 + n)
    w = 0.5 ** L
    sigma = 0.4 * w
    u, v, plan = run(x, y, g, sigma, 8, L, precision="mixed", fine=0)
    plan.close()
    us, vs = oracle.direct_split(x, y, g, sigma, L)
    e, c = 2.0 ** -24, w * w / (2.0 * sigma * sigma)
    r = np.hypot(x[:, None] - x[None], y[:, None] - y[None]) / w
    np.fill_diagonal(r, np.inf)                     # a particle's own term is 0 in either form
    term = -np.expm1(-c * r * r) / r
    bound = (np.abs(g)[None] * (2.5 * np.sqrt(2.0) * c * e + e * ((n + 16) * term + 4.0 / r))).sum(1) / (2.0 * np.pi * w)
    err = np.hypot(u - us, v - vs)
    assert np.all(err <= bound), float(np.max(err / bound))
