"""3D form: every degree on deep trees, where the M2L takes 32 targets a
workgroup and the evaluation one wavefront a leaf.  The degrees differ in the
M2L's steps, tiles and classes and in where its sources lie (below 5 a grid with
one zero box, from 5 on a bordered one).

Reference: the oracle's 3D FMM within the 1e-12 of the other parity tests.  Its
time grows with the boxes and the square of the terms, so the costly ones put
all particles into one box of level k: nothing interacts above level k + 2, and
the result is that of a tree k levels shallower on that box.
"""
import math

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _built():
    oracle.build()


def _check(x, y, z, q, p, L, ref):
    import torch
    import paper_0905_2637_amd as fm
    plan = fm.Plan3D(len(x), p, L)
    out = plan.evaluate(*(torch.as_tensor(a, device="cuda") for a in (x, y, z, q)))
    torch.cuda.synchronize()
    plan.close()
    got = [o.cpu().numpy() for o in out]
    assert ref[4] == 0
    num = sum(np.sum((a - b) ** 2) for a, b in zip(got[1:], ref[1:4]))
    den = sum(np.sum(b ** 2) for b in ref[1:4])
    assert math.sqrt(num / den) < 1e-12
    assert np.linalg.norm(got[0] - ref[0]) < 1e-12 * np.linalg.norm(ref[0])


@pytest.mark.parametrize("p,n", [(0, 5000), (1, 3000), (2, 40000), (4, 3000), (6, 3000)])
def test_whole_cube(p, n):
    rng = np.random.default_rng(700 + p)
    x, y, z, q = rng.random(n), rng.random(n), rng.random(n), rng.uniform(-1, 1, n)
    _check(x, y, z, q, p, 5, oracle.fmm3(x, y, z, q, p, 5))


@pytest.mark.parametrize("p,L,k,box", [
    (7, 5, 1, (1, 0, 1)),
    (8, 5, 1, (0, 1, 0)),
    (9, 5, 1, (1, 1, 0)),
    (3, 6, 2, (1, 2, 3)),
    (5, 6, 2, (2, 1, 0)),
    (2, 7, 3, (3, 4, 7)),
    (5, 7, 3, (4, 0, 3)),
    (0, 7, 3, (7, 7, 7)),
])
def test_one_box_of_a_deep_tree(p, L, k, box):
    rng = np.random.default_rng(720 + p + L)
    n, w = 3000, 0.5 ** k
    c = [(b + rng.random(n)) * w for b in box]
    q = rng.uniform(-1, 1, n)
    _check(*c, q, p, L, oracle.fmm3(*c, q, p, L - k, tuple(b * w for b in box), w))
