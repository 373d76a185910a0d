"""Runs of equal high key bits that a workgroup sorts in LDS, at the edges of its powers of two up to
the longest (2048), alone (nothing too long beside them, which would leave all of them to a sort by
more bits), and with coincident particles in them.  The order must be (key, input index) exactly, as
the oracle's."""
import numpy as np
import pytest

from test_gpu_parity import _clumped_box

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0910_0121_amd as t
    t.lib()
    return t


@pytest.mark.parametrize("n", [60, 70001])
@pytest.mark.parametrize("clumps", [[2048], [2047], [1025, 1024, 1023, 513, 512, 511],
                                    [65, 127, 128, 129, 255, 256, 257, 64, 66] * 3])
def test_sort_order(tp, orc, n, clumps):
    print(f"[gpu-case] long runs n={n} clumps {clumps}", flush=True)
    x, y, z, m = _clumped_box(n, clumps, 23)
    p = tp.treepm_params(1.0, 0.1 / 3.0, 0.1, 0.002, 0.5, 10, 64, tp.TREEPM_FP64)
    T = orc.Tree(x, y, z, m, 1.0, 0.1, 0.002, 0.5, 10, 64)
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
