"""FP64 force at the edges of its work split (the clumps of the FP32 test) on both of its routes:
the table of the pair law from the smallest softening that has one to the largest, and the pair by
pair evaluation below and above those and without softening; with the nearest image taken once per
entry, and per pair where a group's cube plus r_cut reaches half the box.

Bound per particle as in the parity suite: 1e-13 of the summed magnitudes of the pairs and of the
noise of their differences.
"""
import numpy as np
import pytest

import test_gpu_force_groups as groups

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

tp = groups.tp


@pytest.mark.parametrize("radius,r_cut,eps_ratio", [
    (0.1, 0.24, 1 / 60),            # every large group is shared by a workgroup
    (0.02, 0.05, 1 / 60),           # the small groups run on single waves
    (0.1, 0.24, 2.0 ** -11.5),      # the smallest softening with a table
    (0.1, 0.24, 2.0 ** -11.51),     # and just below it: pair by pair
    (0.1, 0.24, 0.0),
    (0.1, 0.24, 8.0),               # the largest softening with a table
    (0.1, 0.24, 8.01),
    (0.1, 0.45, 1 / 60),            # nearest images pair by pair
    (0.1, 0.45, 0.0),
], ids=["split", "single", "eps-min", "eps-below", "eps-0", "eps-max", "eps-above", "images",
        "images-eps-0"])
def test_group_sizes(tp, orc, radius, r_cut, eps_ratio):
    print(f"[gpu-case] clumps radius={radius} r_cut={r_cut} eps/r_cut={eps_ratio}", flush=True)
    x, y, z, m = groups.clumps(groups.SIZES, radius, 77)
    eps = r_cut * eps_ratio
    T = orc.Tree(x, y, z, m, 1.0, r_cut, eps, 0.4, 10, 600)
    ref = np.stack(T.force())
    p = tp.treepm_params(1.0, r_cut / 3.0, r_cut, eps, 0.4, 10, 600, tp.TREEPM_FP64)
    ctx = tp.treepm_create(p, 0)
    try:
        tp.treepm_build(ctx, *[torch.from_numpy(a).cuda() for a in (x, y, z, m)])
        st = tp.treepm_walk(ctx)
        assert st.interactions == T.interactions()
        acc = [torch.full((x.size,), 7.0, dtype=torch.float64, device="cuda") for _ in range(3)]
        tp.treepm_force_short(ctx, *acc)
        got = np.stack([a.cpu().numpy() for a in acc])
    finally:
        tp.treepm_destroy(ctx)
    scale = T.error_scale()[None, :]
    err = np.abs(got - ref)
    print(f"[gpu-case]   max err/(1e-13 scale) {np.max(err / (1e-13 * scale + 1e-300)):.3f}",
          flush=True)
    assert np.all(err <= 1e-13 * scale + 1e-300)
