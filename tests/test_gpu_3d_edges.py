"""The 3D form's kernels at the edges of their work splits: one wavefront per
leaf (8^5 leaves) and four (fewer), leaves of one to several target chunks of
64 whose near sources fill none, one or several stages of 256, every number of
targets per lane, coincident particles, particles outside the cube (behind the
last leaf), degrees with and without folded M2L operators.

Reference: the oracle's 3D FMM of the same degree and depth (the plain sum
where there is no far field), within the 1e-12 of the other parity tests.
Coincident pairs contribute nothing on either side.
"""
import math

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _built():
    oracle.build()


def _points(counts, L, seed):
    """counts[i] particles in leaf i along a row of leaves, the last ones coincident in pairs, and 200 anywhere."""
    rng = np.random.default_rng(seed)
    w = 0.5 ** L
    parts = [rng.random((200, 3))]
    for i, c in enumerate(counts):
        pts = (np.array([i % 2 ** L, 1 % 2 ** L, 0]) + 0.02 + 0.96 * rng.random((c, 3))) * w
        if c >= 4:
            pts[c - 2:] = pts[:2]
        parts.append(pts)
    xyz = np.concatenate(parts)
    return xyz[:, 0].copy(), xyz[:, 1].copy(), xyz[:, 2].copy(), rng.uniform(-1, 1, len(xyz))


@pytest.mark.parametrize("counts,L,p,outside", [
    ([1, 2, 3, 7, 16, 17, 31, 32, 33, 40, 63, 64, 65, 100, 128, 129, 300, 700], 5, 3, 0),
    ([5, 33, 64, 90, 0, 0, 257, 12], 5, 5, 150),
    ([1, 2, 3, 7, 16, 17, 31, 32, 33, 40, 63, 64, 65, 100, 300], 4, 4, 3),
    ([48, 65, 500, 1, 0, 29], 3, 7, 70),
    ([256, 255], 1, 5, 1),
])
def test_leaf_sizes(counts, L, p, outside):
    import torch
    import paper_0905_2637_amd as fm
    x, y, z, q = _points(counts, L, 60 + L)
    n = len(x)
    rng = np.random.default_rng(70)
    xo = np.concatenate([x, 1.0 + rng.random(outside)])
    yo, zo = (np.concatenate([a, rng.random(outside)]) for a in (y, z))
    qo = np.concatenate([q, rng.random(outside)])
    order = rng.permutation(n + outside)
    dev = [torch.as_tensor(np.ascontiguousarray(a[order]), device="cuda") for a in (xo, yo, zo, qo)]
    plan = fm.Plan3D(n + outside, p, L)
    out = plan.evaluate(*dev, check=False)
    torch.cuda.synchronize()
    assert plan.out_of_domain() == outside
    plan.close()
    got = []
    for o in out:
        a = np.empty(n + outside)
        a[order] = o.cpu().numpy()
        assert not a[n:].any()
        got.append(a[:n])
    ref = oracle.fmm3(x, y, z, q, p, L) if L >= 2 else oracle.direct3(x, y, z, q)
    num = sum(np.sum((u - v) ** 2) for u, v in zip(got[1:], ref[1:4]))
    den = sum(np.sum(v ** 2) for v in ref[1:4])
    assert math.sqrt(num / den) < 1e-12
    assert np.linalg.norm(got[0] - ref[0]) / np.linalg.norm(ref[0]) < 1e-12
