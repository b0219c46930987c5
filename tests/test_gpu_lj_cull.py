"""Lennard-Jones forces where the near field leaves staged sources out (those
beyond the cutoff of the target leaf): cutoffs from a small part of a leaf to
its whole width, sparse leaves, quads and leaves of several target chunks,
sources exactly a cutoff away from a leaf's edge, and particles outside the
square (clamped into the edge leaves: there every source is kept).

Reference: the oracle's plain sum, within the 1e-12 (relative L2) of the other
Lennard-Jones tests.  Particles outside lie within a cutoff of the edge, so
all their partners are in the leaves around theirs.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _built():
    oracle.build()


@pytest.mark.parametrize("m,depth,rel_cutoff,outside", [
    (128, 5, 0.55, False),     # quads of 64
    (128, 5, 1.0, True),
    (48, 5, 0.9, True),        # about two per leaf
    (90, 3, 0.2, False),       # about 127 per leaf: two target chunks, three stages of sources
    (90, 3, 0.04, True),       # fewer than one partner each
    (64, 0, 0.05, False),      # one leaf
])
def test_forces(m, depth, rel_cutoff, outside):
    import torch
    import paper_0905_2637_amd as fm
    rng = np.random.default_rng(830 + m + depth)
    a = 1.0 / m
    c = (np.arange(m) + 0.5) * a
    X, Y = np.meshgrid(c, c)
    x = X.ravel() + rng.uniform(-0.2 * a, 0.2 * a, m * m)
    y = Y.ravel() + rng.uniform(-0.2 * a, 0.2 * a, m * m)
    w = 0.5 ** depth
    rc = rel_cutoff * w
    if depth > 0:              # at a cutoff from an edge of leaf column 1, far from other particles' cores
        x[5], x[7] = 2.0 * w + rc, w - rc
    k = 0
    if outside:
        edge = np.concatenate([np.argsort(x)[:6], np.argsort(-y)[:6]])
        k = len(edge)
        x[edge[:6]] = -0.3 * rc * (1.0 + rng.random(6))
        y[edge[6:]] = 1.0 + 0.3 * rc * (1.0 + rng.random(6))
    s, eps = a / 1.12, 0.8
    dev = [torch.as_tensor(v, device="cuda") for v in (x, y, np.zeros(len(x)))]
    plan = fm.Plan(len(x), s, 8, depth, kernel="lennard-jones", lj_epsilon=eps, cutoff=rc)
    fx, fy = plan.evaluate(*dev, check=False)
    torch.cuda.synchronize()
    assert plan.out_of_domain() == k
    plan.close()
    fx, fy = fx.cpu().numpy(), fy.cpu().numpy()
    ox, oy = oracle.lj_forces(x, y, eps, s, rc)
    num = np.sum((fx - ox) ** 2 + (fy - oy) ** 2)
    den = np.sum(ox ** 2 + oy ** 2)
    assert num <= 1e-24 * den
