"""The fast Gauss transform at the compiled sizes below 16, where the matrix
instructions carry unused rows and columns (8 and 12 of 16; 8 takes two boxes
side by side along an axis) and at sizes padded to them, at one, four and sixteen
wavefronts per box, at particles and at points.

Reference: the oracle's fast transform of the same size and range within the
1e-12 of the other parity tests.
"""
import math

import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _built():
    oracle.build()


def _range(sigma, L):
    nc = math.ceil(math.sqrt(math.log(1e16)) * math.sqrt(2.0) * sigma * 2 ** L)
    return min(nc, 2 ** L - 1)


def _dev(*arrays):
    import torch
    return [torch.as_tensor(np.ascontiguousarray(a), device="cuda") for a in arrays]


def _check(G, Go):
    assert np.linalg.norm(G.cpu().numpy() - Go) < 1e-12 * np.linalg.norm(Go)


@pytest.mark.parametrize("L", [4, 5, 6])
@pytest.mark.parametrize("p", [7, 8, 10, 12])
@pytest.mark.parametrize("clustered", [False, True])
def test_particles(p, L, clustered):
    import torch
    import paper_0905_2637_amd as fm
    n, sigma = 9001, 1.3 / 2 ** L
    x, y, q = workloads.gaussian_mixture(n, 3, 950 + L)[:3] if clustered else workloads.uniform_square(n, 950 + L)
    plan = fm.Plan(n, sigma, p, L, kernel="gauss-transform")
    G, v = plan.evaluate(*_dev(x, y, q))
    torch.cuda.synchronize()
    plan.close()
    Go, nbad = oracle.fgt(x, y, q, sigma, p, L, _range(sigma, L))
    assert nbad == 0 and not v.cpu().numpy().any()
    _check(G, Go)


@pytest.mark.parametrize("p", [8, 12])
@pytest.mark.parametrize("n", [1, 100, 5000])
def test_four_boxes(p, n):
    """Depth 1: the shortest line of boxes, one pair wide."""
    import torch
    import paper_0905_2637_amd as fm
    x, y, q = workloads.uniform_square(n, 960 + n)
    plan = fm.Plan(n, 0.6, p, 1, kernel="gauss-transform")
    G, _ = plan.evaluate(*_dev(x, y, q))
    torch.cuda.synchronize()
    plan.close()
    _check(G, oracle.fgt(x, y, q, 0.6, p, 1, _range(0.6, 1))[0])


@pytest.mark.parametrize("p,L,n,m", [(12, 6, 9001, 3001), (8, 6, 3001, 20000), (8, 5, 5000, 300), (12, 4, 700, 5000)])
def test_points(p, L, n, m):
    import torch
    import paper_0905_2637_amd as fm
    sigma = 1.3 / 2 ** L
    x, y, q = workloads.uniform_square(n, 970 + n)
    rng = np.random.default_rng(970 + m)
    tx, ty = rng.random(m), rng.random(m)
    plan = fm.Plan(n, sigma, p, L, kernel="gauss-transform", m_max=m)
    G, _ = plan.evaluate_at(*_dev(x, y, q, tx, ty))
    torch.cuda.synchronize()
    plan.close()
    Go, nbad = oracle.fgt_at(x, y, q, sigma, p, L, _range(sigma, L), tx, ty)
    assert nbad == 0
    _check(G, Go)


@pytest.mark.parametrize("p", [8, 12, 16])
def test_shared_coefficients(p):
    """From 2^18 points on, wavefronts within one box read its coefficients
    through scalar loads: the same values as for a few points, which never do,
    bit for bit."""
    import torch
    import paper_0905_2637_amd as fm
    n, L = (1 << 18) + 77, 4
    dev = _dev(*workloads.uniform_square(n, 985))
    plan = fm.Plan(n, 1.0 / 2 ** L, p, L, kernel="gauss-transform", m_max=n)
    all_at = plan.evaluate(*dev)[0].clone()
    points = [t[:5000].contiguous() for t in dev[:2]]
    few = plan.evaluate_at(*dev, *points)[0].clone()
    at = plan.evaluate_at(*dev, *dev[:2])[0]
    torch.cuda.synchronize()
    assert torch.equal(all_at[:5000], few) and torch.equal(all_at, at)
    plan.close()
