"""The tree of small plans (one counting pass over the whole leaf key) against
the oracle's keys, stable permutation and leaf ranges, bit for bit, and against
the digit passes that larger plans take (same particles, a capacity past the
small path's): one tile and many, counts at the tile's edges, one to twelve key
bits and the first past them, all particles in one leaf, equal positions,
particles outside the square and NaN, the mixed form's FP32 records (through
the velocities, which must agree bit for bit).
"""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

SMALL = 64 * 4096        # largest capacity of the small path


@pytest.fixture(scope="module", autouse=True)
def _built():
    oracle.build()


def _run(x, y, g, L, n_max, precision):
    import torch
    import paper_0905_2637_amd as fm
    plan = fm.Plan(n_max, 0.004, 8, L, precision=precision, fp32_fine_levels=min(2, max(0, L - 1)))
    dev = [torch.as_tensor(a, device="cuda") for a in (x, y, g)]
    u, v = plan.evaluate(*dev, check=False)
    torch.cuda.synchronize()
    out = [plan.dump(k) for k in (fm.DUMP_KEYS, fm.DUMP_PERM, fm.DUMP_LEAF_START)] + [u.cpu().numpy(), v.cpu().numpy()]
    bad = plan.out_of_domain()
    plan.close()
    return out, bad


@pytest.mark.parametrize("n,L,kind,precision", [
    (1, 1, "uniform", "fp64"),
    (63, 2, "uniform", "mixed"),
    (4095, 3, "uniform", "fp64"),
    (4096, 4, "uniform", "mixed"),
    (4096, 6, "one leaf", "fp64"),
    (4097, 6, "uniform", "fp64"),
    (8193, 5, "outside", "fp64"),
    (30000, 6, "clusters", "mixed"),
    (50001, 4, "one leaf", "fp64"),
    (SMALL, 6, "uniform", "fp64"),
    (20000, 7, "uniform", "fp64"),          # 14 key bits: the digit passes
])
def test_small_sort(n, L, kind, precision):
    if kind == "clusters":
        x, y, g, _, _ = workloads.gaussian_mixture(n, 4, 80)
    else:
        x, y, g = workloads.uniform_square(n, 80 + n % 97)
    if kind == "one leaf":
        x, y = 0.3 + 1e-4 * x, 0.7 + 1e-4 * y
        x[1::3], y[1::3] = x[0], y[0]
    if kind == "outside":
        x[5], y[4096], x[8192] = -0.5, 1.5, np.nan
    small, bad = _run(x, y, g, L, n, precision)
    large, bad2 = _run(x, y, g, L, SMALL + 1, precision)
    key, perm, ls, nbad = oracle.tree(x, y, L)
    assert bad == bad2 == nbad
    assert np.array_equal(small[0], key) and np.array_equal(small[1], perm) and np.array_equal(small[2], ls)
    for a, b in zip(small, large):
        assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f")
