"""The sort's second half at the lengths where its route changes: runs of equal high key bits up to
64 (in a tile of 1024, wherever they start in it), above that up to 2048 (listed), longer ones
(all of the bits), for boxes sorted by 24 and by 32 high bits.  The order must be (key, input
index) exactly, as the oracle's.
"""
import numpy as np
import pytest

import boxgen
from test_gpu_parity import _clumped_box

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

SHORT = [2, 3, 31, 32, 33, 62, 63, 64] * 40     # many: they start everywhere in a tile
LONG = [65, 66, 127, 128, 129, 1023, 1024, 1025, 2046]


@pytest.fixture(scope="module")
def tp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0910_0121_amd as t
    t.lib()
    return t


@pytest.mark.parametrize("n", [1, 900, 3001, 70001])
@pytest.mark.parametrize("clumps", [SHORT, SHORT + LONG, SHORT + [2048, 2049, 2500]],
                         ids=["short", "long", "too-long"])
def test_sort_order(tp, orc, n, clumps):
    print(f"[gpu-case] sort runs n={n} clumps up to {max(clumps)}", flush=True)
    x, y, z, m = _clumped_box(n, clumps, 17)
    T = orc.Tree(x, y, z, m, 1.0, 0.1, 0.002, 0.5, 10, 64)
    p = tp.treepm_params(1.0, 0.1 / 3.0, 0.1, 0.002, 0.5, 10, 64, tp.TREEPM_FP64)
    ctx = tp.treepm_create(p, 0)
    try:
        for _ in range(2):
            tp.treepm_build(ctx, *[torch.from_numpy(a).cuda() for a in (x, y, z, m)])
            gk, gi = tp.treepm_export_sorted(ctx)
            ok, oi = T.sorted()
            np.testing.assert_array_equal(gk, ok)
            np.testing.assert_array_equal(gi, oi)
    finally:
        tp.treepm_destroy(ctx)
