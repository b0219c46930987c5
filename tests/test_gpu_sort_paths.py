"""Sorts that only some plans take, against the oracle's trees bit for bit: the
points of small plans over several tiles (with more points than particles and
the reverse, on a given square and on the bounding one), and batched instances
sorted apart on more than 4096 tiles (workgroups of 256 threads).
"""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _built():
    oracle.build()


def _dev(*arrays):
    import torch
    return [torch.as_tensor(np.ascontiguousarray(a), device="cuda") for a in arrays]


@pytest.mark.parametrize("n,m,L", [(5000, 30000, 5), (30000, 5000, 6), (3000, 4097, 1), (4097, 4096, 6), (200, 200000, 6)])
@pytest.mark.parametrize("domain", [(0.0, 0.0, 1.0), None])
def test_points_of_small_plans(n, m, L, domain):
    import torch
    import paper_0905_2637_amd as fm
    x, y, g = workloads.uniform_square(n, 980 + L)
    rng = np.random.default_rng(990 + L)
    tx, ty = rng.random(m), rng.random(m)
    tx[1::7], ty[1::7] = tx[0], ty[0]
    if domain is None:
        tx = 1.3 * tx - 0.2
    plan = fm.Plan(n, 0.3 / 2 ** L, 8, L, domain=domain, m_max=m)
    plan.evaluate_at(*_dev(x, y, g, tx, ty))
    torch.cuda.synchronize()
    d = domain or oracle.bounding_square(np.concatenate([x, tx]), np.concatenate([y, ty]))
    assert tuple(plan.dump(fm.DUMP_DOMAIN)[:3]) == tuple(d)
    for dumps, (a, b) in (((fm.DUMP_KEYS, fm.DUMP_PERM, fm.DUMP_LEAF_START), (x, y)),
                          ((fm.DUMP_TKEYS, fm.DUMP_TPERM, fm.DUMP_TLEAF_START), (tx, ty))):
        key, perm, ls, nbad = oracle.tree(a, b, L, *d)
        got = [plan.dump(k) for k in dumps]
        assert nbad == 0
        assert np.array_equal(got[0], key) and np.array_equal(got[1], perm) and np.array_equal(got[2], ls)
    plan.close()


def test_instances_apart_on_many_tiles():
    import torch
    import paper_0905_2637_amd as fm
    counts, depths = [4096 * 1365 + 1, 0, 4096 * 2731 - 1, 40000], [8, 3, 9, 5]
    n = sum(counts)
    assert n // 4096 + len(counts) > 4096
    rng = np.random.default_rng(995)
    x, y = rng.random(n), rng.random(n)
    plan = fm.BatchPlan(counts, depths, 1e-3, 8)
    xd, yd = _dev(x, y)
    g = torch.zeros(n, dtype=torch.float64, device="cuda")
    plan.evaluate(xd, yd, g)
    torch.cuda.synchronize()
    perm_all = plan.dump(fm.DUMP_PERM)[:n].astype(np.int64)
    ls_all = plan.dump(fm.DUMP_LEAF_START).astype(np.int64)
    plan.close()
    off = seg = 0
    for c, L in zip(counts, depths):
        ent = 4 ** L + 1
        if c > 0:
            _, perm, ls, nbad = oracle.tree(x[off:off + c], y[off:off + c], L)
            assert nbad == 0
            assert np.array_equal(perm_all[off:off + c] - off, perm), (c, L)
            assert np.array_equal(ls_all[seg:seg + ent] - off, ls), (c, L)
        else:
            assert np.all(ls_all[seg:seg + ent] == off)
        off, seg = off + c, seg + ent


@pytest.mark.parametrize("L", [7, 9])
def test_runs_of_empty_leaves(L):
    """Runs around the length from which a wavefront fills them together, long
    ones, and none, side by side and at both ends."""
    import torch
    import paper_0905_2637_amd as fm
    rng = np.random.default_rng(996 + L)
    runs = [0, 1, 7, 8, 9, 30, 31, 32, 33, 34, 63, 64, 65, 66, 127, 128, 129, 300, 2000]
    leaf, at = [], 40
    while True:
        at += 1 + int(rng.choice(runs))
        if at >= 4 ** L - 200:
            break
        leaf += [at] * int(rng.integers(1, 3))
    k = np.array(leaf, dtype=np.uint64)
    a, b = np.zeros(len(k)), np.zeros(len(k))
    for bit in range(L):
        a += ((k >> np.uint64(2 * bit)) & np.uint64(1)) * 2.0 ** bit
        b += ((k >> np.uint64(2 * bit + 1)) & np.uint64(1)) * 2.0 ** bit
    order = rng.permutation(len(k))
    x, y = (((c + 0.1 + 0.8 * rng.random(len(k))) / 2 ** L)[order] for c in (a, b))
    plan = fm.Plan(300000, 1e-4, 8, L)
    plan.evaluate(*_dev(x, y, np.ones(len(x))))
    torch.cuda.synchronize()
    key, perm, ls, nbad = oracle.tree(x, y, L)
    assert nbad == 0 and len(np.unique(np.diff(np.unique(key)))) > 10
    assert np.array_equal(plan.dump(fm.DUMP_KEYS), key) and np.array_equal(plan.dump(fm.DUMP_PERM), perm)
    assert np.array_equal(plan.dump(fm.DUMP_LEAF_START), ls)
    plan.close()
