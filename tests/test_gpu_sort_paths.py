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
