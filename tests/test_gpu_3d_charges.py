"""3D form: a charge that is infinite or NaN.  It acts on the others, not on its
own particle nor on one at the same place: pairs at zero distance are left out
whatever the charge.  One and four wavefronts per leaf, targets and sources in
several chunks and stages, several such charges in a stage.

Reference, depth <= 1: the oracle's plain sum, infinities and NaN equal, a finite
potential within the 1e-13 of the other plain-sum test (of its terms' sizes).  With a far field: the same call
with those charges zero; what they do not act on is equal bit for bit, and every
other particle of the leaves around has an infinite or NaN potential.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _built():
    oracle.build()


def _run(x, y, z, q, p, L):
    import torch
    import paper_0905_2637_amd as fm
    plan = fm.Plan3D(len(x), p, L)
    out = plan.evaluate(*(torch.as_tensor(a, device="cuda") for a in (x, y, z, q)))
    torch.cuda.synchronize()
    plan.close()
    return [o.cpu().numpy() for o in out]


@pytest.mark.parametrize("n,L,bad", [
    (300, 0, [np.inf]),
    (300, 1, [-np.inf]),
    (1100, 1, [np.nan]),
    (700, 0, [np.inf, np.inf, -np.inf]),
])
def test_plain_sum(n, L, bad):
    rng = np.random.default_rng(500 + n)
    x, y, z, q = rng.random(n), rng.random(n), rng.random(n), rng.uniform(-1, 1, n)
    at = rng.choice(n, len(bad), replace=False)
    q[at] = bad
    got, ref = _run(x, y, z, q, 4, L), oracle.direct3(x, y, z, q)
    for g, r in zip(got, ref):
        fin = np.isfinite(r)
        assert np.array_equal(g[~fin], r[~fin], equal_nan=True)
        assert np.all(np.isfinite(g[fin]))
    if len(bad) == 1:          # its own potential: the sum over the others
        k, others = at[0], np.arange(n) != at[0]
        r = np.sqrt((x - x[k]) ** 2 + (y - y[k]) ** 2 + (z - z[k]) ** 2)[others]
        assert abs(got[0][k] - ref[0][k]) < 1e-13 * np.sum(np.abs(q[others]) / r)


@pytest.mark.parametrize("n,L,p", [(6000, 3, 6), (60000, 5, 3), (40000, 3, 4), (500, 2, 9)])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_its_own_result(n, L, p, bad):
    rng = np.random.default_rng(600 + n)
    x, y, z, q = rng.random(n), rng.random(n), rng.random(n), rng.uniform(-1, 1, n)
    k, twin = n // 2, n // 3
    x[twin], y[twin], z[twin] = x[k], y[k], z[k]
    q0 = q.copy()
    q0[k] = 0.0
    q[k] = bad
    got, ref = _run(x, y, z, q, p, L), _run(x, y, z, q0, p, L)
    for g, r in zip(got, ref):
        assert np.all(np.isfinite(r))
        assert g[k] == r[k] and g[twin] == r[twin]
    leaf = [np.floor(a * 2 ** L) for a in (x, y, z)]
    near = np.all([np.abs(a - a[k]) <= 1 for a in leaf], axis=0)
    near[[k, twin]] = False
    assert near.sum() > 0 and not np.any(np.isfinite(got[0][near]))
