"""The sort of batched plans that keeps the instances apart (by the leaf bits
only) against the oracle's tree, instance by instance, and against the sort by
the whole key, which a plan with room for more instances takes: permutation,
leaf ranges and velocities bit for bit.  Sizes at the edges of the 4096-record
tiles, empty instances first, in the middle and last, unused instance slots,
one to three digits, equal depths and mixed ones, one instance with nearly
every particle, particles outside the square, and sets that replace one
another in one plan.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

INST = 9                       # slots of the plan; past 8192 particles a slot on average the instances stay apart
CAP = 8192 * INST
SETS = [
    [(0, 2), (1, 0), (4095, 4), (4096, 3), (4097, 4), (0, 1), (8192, 2), (12289, 4), (0, 3)],
    [(CAP - 1, 4), (1, 4)],
    [(4096, 4), (4096, 4), (4096, 4)],
    [(63, 1), (30000, 6), (64, 0), (20000, 5), (2, 6)],
    [(CAP // INST, 9)] * INST,
]


@pytest.fixture(scope="module", autouse=True)
def _built():
    oracle.build()


def _run(plan, n_cap, x, y, g, counts, depths):
    import torch
    import paper_0905_2637_amd as fm
    n = len(x)
    X, Y, G, U, V = (torch.zeros(n_cap, dtype=torch.float64, device="cuda") for _ in range(5))
    for dst, src in ((X, x), (Y, y), (G, g)):
        dst[:n] = torch.as_tensor(src, device="cuda")
    plan.evaluate(X[:n], Y[:n], G[:n], U[:n], V[:n], counts=counts, depths=depths, check=False)
    torch.cuda.synchronize()
    entries = sum(4 ** d + 1 for d in depths)
    return (plan.dump(fm.DUMP_PERM)[:n].astype(np.int64), plan.dump(fm.DUMP_LEAF_START)[:entries].astype(np.int64),
            U[:n].cpu().numpy(), V[:n].cpu().numpy(), plan.out_of_domain())


@pytest.mark.parametrize("depth,sets", [(4, [0, 1, 2]), (6, [3, 0, 3]), (9, [4, 3])])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_instances_sorted_apart(depth, sets, precision):
    import paper_0905_2637_amd as fm
    leaves = max(sum(4 ** d for _, d in SETS[k]) for k in sets)
    plans = [fm.BatchPlan([CAP], [depth], 0.3 / (1 << depth), 8, precision=precision, n_max=CAP, max_instances=m,
                          max_depth=depth, max_leaves=max(leaves, 4 ** depth)) for m in (INST, 8 * INST)]
    for k in sets:
        counts, depths = [c for c, _ in SETS[k]], [d for _, d in SETS[k]]
        rng = np.random.default_rng(300 + k)
        n = sum(counts)
        x, y, g = rng.random(n), rng.random(n), rng.uniform(-1.0, 1.0, n)
        x[n // 2], y[n // 3] = 1.25, -0.5
        apart, whole = (_run(p, CAP, x, y, g, counts, depths) for p in plans)
        for a, b in zip(apart, whole):
            assert np.array_equal(a, b), k
        off, seg, nbad = 0, 0, 0
        for c, L in zip(counts, depths):
            ent = 4 ** L + 1
            if c > 0:
                _, perm, ls, bad = oracle.tree(x[off:off + c], y[off:off + c], L)
                assert np.array_equal(apart[0][off:off + c] - off, perm), (k, c, L)
                assert np.array_equal(apart[1][seg:seg + ent] - off, ls), (k, c, L)
                nbad += bad
            else:
                assert np.all(apart[1][seg:seg + ent] == off)
            off, seg = off + c, seg + ent
        assert apart[4] == nbad == 2
    for p in plans:
        p.close()
