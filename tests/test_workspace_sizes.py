"""Workspace sizes that callers may hold as constants or preallocated buffers:
the bytes these plans asked for before their small and batched sorts got tables
of their own.  A plan may need less, never more, or a buffer that held it is
refused.  No GPU needed.
"""
import pytest

import paper_0905_2637_amd as fm


@pytest.mark.parametrize("n,depth,held,kw", [
    # one sort over the whole key (at most 2^18 points, depth 6)
    (1, 6, 4281088, {}),
    (4097, 6, 4561664, {}),
    (262144, 6, 22233088, {}),
    (100003, 5, 7971584, {}),
    (30000, 1, 2127104, {}),
    (5000, 6, 15014912, dict(m_max=200000)),
    (20000, 6, 43397376, dict(kernel="gauss-transform")),
    (20000, 6, 5967104, dict(precision="mixed")),
    # by digits
    (262145, 6, 22238208, {}),
    (1 << 20, 8, 139264768, {}),
    # batched, the instances sorted apart and not
    (16384, 4, 1715968, dict(max_instances=2)),
    (73728, 6, 43015168, dict(max_instances=9)),
    (1 << 20, 5, 206681088, dict(max_instances=128)),
    (1 << 22, 5, 826528256, dict(max_instances=512)),
    (4095 * 512, 5, 682836224, dict(max_instances=512)),
])
def test_no_larger(n, depth, held, kw):
    prm = fm.make_params(n, 0.3 / 2 ** depth, 12, depth, fp32_fine_levels=min(2, depth - 1), **kw)
    assert fm.workspace_size(prm) <= held


# bytes that 3D plans of 1,000 particles asked for with full sets of coefficients, degrees 0 to 9
HELD_3D = {
    0: [84224, 183552, 520960, 1253632, 2535424, 4519424, 7360512, 11210496, 16225280, 22556160],
    2: [85504, 188416, 532480, 1276928, 2575616, 4584192, 7457536, 11348992, 16415488, 22809856],
    5: [814336, 2711296, 6643456, 13368064, 23636992, 38203904, 57821696, 83241728, 115218944, 154504192],
    7: [46820608, 161963776, 392388352, 776600320, 1353100288, 2160390656, 3236973056, 4621347584, 6352017920,
        8467483648],
}


@pytest.mark.parametrize("depth", sorted(HELD_3D))
@pytest.mark.parametrize("p", range(10))
def test_no_larger_3d(depth, p):
    import ctypes as C
    prm, out = fm.Fmm3dParams(1000, p, depth, 0.0, 0.0, 0.0, 1.0), C.c_size_t(0)
    assert fm.load().fmm3d_workspace_size(C.byref(prm), C.byref(out)) == fm.FMM_OK
    assert out.value <= HELD_3D[depth][p]
