"""The sort's passes end with the highest bit of the keys: particles in the cells next to the box's far
corner (all key bits set) and its origin, and crowds of up to 2048 that share exactly the high bits
that the passes of this many particles cover (levels 8, 10 2/3 and 13 1/3 of the cells), so that no
wider sort is needed.  The order must be (key, input index) exactly, as the oracle's."""
import numpy as np
import pytest

import boxgen

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0910_0121_amd as t
    t.lib()
    return t


@pytest.mark.parametrize("n,level", [(60000, 8), (65536, 8), (65537, 10), (300001, 10),
                                     (2097153, 13)])
def test_sort_order(tp, orc, n, level):
    print(f"[gpu-case] sort key bits n={n} level={level}", flush=True)
    p = list(boxgen.uniform_box(n, 31))
    rng = boxgen.SplitMix64(32)
    side, at = 2.0 ** -level, 0
    for corner in (0.0, 1.0 - side, 0.5 - side, 0.5):
        for a in range(3):
            p[a][at:at + 2000] = corner + side * rng.uniform(2000)
        at += 2000
    perm = np.argsort(rng.next_u64(n), kind="stable")
    x, y, z = (np.ascontiguousarray(p[a][perm]) for a in range(3))
    m = np.full(n, 1.0 / n)
    T = orc.Tree(x, y, z, m, 1.0, 0.1, 0.002, 0.5, 10, 64)
    ctx = tp.treepm_create(tp.make_params(1.0, 0.1 / 3.0, 0.1, 0.002, 0.5, 10, 64,
                                          tp.TREEPM_FP64), 0)
    try:
        for _ in range(2):
            tp.treepm_build(ctx, *[torch.from_numpy(a).cuda() for a in (x, y, z, m)])
            gk, gi = tp.treepm_export_sorted(ctx)
            ok, oi = T.sorted()
            np.testing.assert_array_equal(gk, ok)
            np.testing.assert_array_equal(gi, oi)
    finally:
        tp.treepm_destroy(ctx)
