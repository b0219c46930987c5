"""The FP64 M2L by the symmetry classes of the square: every local coefficient
of every level against the oracle's, order by order (an error in a high order
does not reach the velocities), at each compiled expansion size and the padded
ones next to it, on launches of one workgroup and of many, and with the list in
one part and split.

Tolerance: the largest difference of an order on a level, relative to that
order's largest coefficient there, below 1e-11, the bound that the coefficient
test of the default form uses.  A coefficient sums 27 p terms whose sizes are
at most sqrt(n per box) < 40 times the result's (charges of random sign), so
rounding alone stays near 27 p 40 2^-53 < 4e-12.
"""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import gpu_coeffs_to_oracle, level_offset

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _built():
    oracle.build()


@pytest.mark.parametrize("p", [1, 3, 8, 9, 12, 16, 17, 18, 20, 23, 24, 25, 32])
@pytest.mark.parametrize("L", [2, 4, 6])
def test_local_coefficients_by_order(p, L):
    import torch
    import paper_0905_2637_amd as fm
    n = min(20000, 40 << (2 * L))
    x, y, g = workloads.uniform_square(n, 140 + p)
    sigma = 0.4 / (1 << L)
    *_, le, _ = oracle.fmm(x, y, g, sigma, p, L, dump=True)
    plan = fm.Plan(n, sigma, p, L)
    xd, yd, gd = (torch.as_tensor(a, device="cuda") for a in (x, y, g))
    for split in (0, 8):
        plan.set_tuning(4, split, 0)
        plan.evaluate(xd, yd, gd, check=True)
        torch.cuda.synchronize()
        got = gpu_coeffs_to_oracle(plan.dump(fm.DUMP_LE), L, 1.0, "le")
        for l in range(2, L + 1):
            sl = slice(level_offset(l), level_offset(l + 1))
            err = np.max(np.abs(got[sl] - le[sl]), axis=0) / np.max(np.abs(le[sl]), axis=0)
            assert np.max(err) < 1e-11, (split, l, int(np.argmax(err)), float(np.max(err)))
    plan.close()
