"""FP32 quadrupole terms at the edges of their work split and table: the clumps of the force test
(groups of every size at which the chunks change, shared by a workgroup or run by single waves),
softenings from the smallest to the largest, float and double records.

Bound per particle: 8 u B_i for the monopole part as in the force test, u = 2^-24, and for the
quadrupole part as much again times its size: with cells of l / r <= 0.5 a term is at most 1.2
of what its pair adds to B_i, and the table's error and the rounding of a term are within 8 u of
it (where the table's relative error is larger, near the cutoff, the law itself has fallen by
more): 20 u B_i together.  Float outputs add u of the result.
"""
import numpy as np
import pytest

import test_gpu_force_groups as groups

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

tp = groups.tp


@pytest.mark.parametrize("radius,r_cut,eps_ratio,dtype", [
    (0.12, 0.24, 1 / 60, "float64"),       # every large group is shared by a workgroup
    (0.12, 0.24, 1 / 60, "float32"),
    (0.12, 0.12, 1 / 60, "float64"),       # shorter lists: the small groups run on single waves
    (0.12, 0.24, 2.0 ** -13, "float64"),   # the smallest softening: the longest table
    (0.12, 0.24, 7.9, "float64"),          # the largest: the shortest
], ids=["split", "split-f32", "single", "eps-min", "eps-max"])
def test_group_sizes(tp, orc, radius, r_cut, eps_ratio, dtype):
    from test_gpu_parity import fp32_error_scale
    print(f"[gpu-case] clumps radius={radius} r_cut={r_cut} eps/r_cut={eps_ratio} {dtype}",
          flush=True)
    x, y, z, m = groups.clumps(groups.SIZES, radius, 77)
    eps = r_cut * eps_ratio
    T = orc.Tree(x, y, z, m, 1.0, r_cut, eps, 0.5, 10, 600, quadrupole=True)
    mono = np.stack(orc.Tree(x, y, z, m, 1.0, r_cut, eps, 0.5, 10, 600).force())
    ref = np.stack(T.force())
    assert np.max(np.abs(ref - mono)) > 0
    p = tp.make_params(1.0, r_cut / 3.0, r_cut, eps, 0.5, 10, 600, tp.TREEPM_FP32, quadrupole=1)
    ctx = tp.treepm_create(p, 0)
    try:
        tp.treepm_build(ctx, *[torch.from_numpy(a).cuda() for a in (x, y, z, m)])
        st = tp.treepm_walk(ctx)
        assert st.interactions == T.interactions()
        acc = [torch.full((x.size,), 7.0, dtype=getattr(torch, dtype), device="cuda")
               for _ in range(3)]
        tp.treepm_force_short(ctx, *acc)
        got = np.stack([a.cpu().numpy().astype(np.float64) for a in acc])
    finally:
        tp.treepm_destroy(ctx)
    u = 2.0 ** -24
    bound = 20 * u * fp32_error_scale(T, x, y, z, m, eps)
    if dtype == "float32":
        bound = bound + u * np.linalg.norm(ref, axis=0)
    d = np.linalg.norm(got - ref, axis=0)
    print(f"[gpu-case]   max |da| / bound {np.max(d / bound):.3f}, largest quadrupole part "
          f"{np.max(np.linalg.norm(ref - mono, axis=0) / np.linalg.norm(ref, axis=0)):.1e}",
          flush=True)
    assert np.all(d <= bound)
