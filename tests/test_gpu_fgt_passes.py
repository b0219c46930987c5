"""The fast Gauss transform's kernels where their work split changes: one, four
and sixteen wavefronts per box in P2H (4^6, 4^5 and fewer boxes), boxes with
no, one and many particles, wavefronts of the Taylor evaluation whose points
lie in few boxes (coefficients through scalar loads) and in many (gathered),
counts that fill no wavefront, ranges clipped at the square's edge.

Reference: the plain sum, at p = 16 and w / sigma = 0.78, where the oracle's
fast form is within 8.5e-15 of it (3.4e-13 at w / sigma = 0.98): what remains
is the rounding of two sums of n terms of mixed sign, 1e-13 relative to the
result's norm, the bound of the other transform tests.
"""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _built():
    oracle.build()


@pytest.mark.parametrize("n,L,sigma,clustered", [
    (257, 6, 0.02, False),       # most boxes empty, every wavefront gathers
    (30011, 6, 0.02, False),    # about seven per box
    (20000, 6, 0.02, True),      # dense and empty boxes side by side
    (20003, 5, 0.04, True),
    (9001, 3, 0.16, False),     # about 140 per box: scalar coefficients
    (4097, 2, 0.32, False),       # the whole square within the range
    (1023, 1, 0.64, True),
])
def test_fgt_against_the_plain_sum(n, L, sigma, clustered):
    import torch
    import paper_0905_2637_amd as fm
    if clustered:
        x, y, q, _, _ = workloads.gaussian_mixture(n, 3, 940 + L)
    else:
        x, y, q = workloads.uniform_square(n, 940 + L)
    dev = [torch.as_tensor(a, device="cuda") for a in (x, y, q)]
    plan = fm.Plan(n, sigma, 16, L, kernel="gauss-transform")
    G, v = plan.evaluate(*dev)
    torch.cuda.synchronize()
    plan.close()
    Gd = oracle.gauss_direct(x, y, q, sigma)
    err = float(np.linalg.norm(G.cpu().numpy() - Gd) / np.linalg.norm(Gd))
    assert not v.cpu().numpy().any()
    assert err < 1e-13, f"rel L2 vs the plain sum {err:.3e}"
