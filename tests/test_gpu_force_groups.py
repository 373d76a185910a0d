"""FP32 force at the edges of its work split: groups of every size at which the kernel's chunks
of particles change (1, 4, 8, 16, ... up to groups of several chunks), in pieces or run by
single waves, and pair-law tables from the smallest to the largest softening.

Boxes are isolated clumps, one per level-2 cell, so the groups are exactly the clumps.  Bound per
particle as in the parity suite: |da_i| <= 8 u B_i (rounding of the FP32 relative positions and
of the pair arithmetic), u = 2^-24.
"""
import numpy as np
import pytest

import boxgen

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 4, 5, 8, 9, 13, 14, 16, 17, 26, 27, 32, 33, 53, 54, 64, 65, 106, 107, 128, 129,
         181, 192, 213, 214, 255, 256, 257, 300, 512, 513]


@pytest.fixture(scope="module")
def tp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0910_0121_amd as t
    t.lib()
    return t


def clumps(sizes, radius, seed):
    """One clump per level-2 cell: sizes[k] particles within `radius` of the centre of cell k;
    the cells left over hold 600 particles, so every level-1 octant holds more than n_crit."""
    rng = boxgen.SplitMix64(seed)
    pos = []
    for cell in range(64):
        # spread the sizes over the octants: cell 8 o + j is child j of octant o
        k = (cell % 8) * 8 + cell // 8
        c = sizes[k] if k < len(sizes) else 600
        q = np.array([((cell >> 5) & 1) * 2 + ((cell >> 2) & 1),
                      ((cell >> 4) & 1) * 2 + ((cell >> 1) & 1),
                      ((cell >> 3) & 1) * 2 + (cell & 1)])
        centre = (q + 0.5) / 4.0
        pos.append(centre[:, None] + radius * (2.0 * rng.uniform(3 * c).reshape(3, c) - 1.0))
    p = np.concatenate(pos, axis=1)
    p = p[:, np.argsort(rng.next_u64(p.shape[1]), kind="stable")]
    m = np.exp(rng.uniform(p.shape[1]) * np.log(30.0))
    return p[0].copy(), p[1].copy(), p[2].copy(), m / m.sum()


@pytest.mark.parametrize("radius,r_cut,eps_ratio", [
    (0.1, 0.24, 1 / 60),          # lists of thousands: every large group is shared by a workgroup
    (0.02, 0.05, 1 / 60),         # only the clump itself: the small groups run on single waves
    (0.1, 0.24, 2.0 ** -13),      # the smallest softening: the longest table
    (0.1, 0.24, 7.9),             # the largest: the shortest
    (0.1, 0.24, 0.05),
], ids=["split", "single", "eps-min", "eps-max", "eps-mid"])
def test_group_sizes(tp, orc, radius, r_cut, eps_ratio):
    from test_gpu_parity import fp32_error_scale
    print(f"[gpu-case] clumps radius={radius} r_cut={r_cut} eps/r_cut={eps_ratio}", flush=True)
    x, y, z, m = clumps(SIZES, radius, 77)
    eps = r_cut * eps_ratio
    T = orc.Tree(x, y, z, m, 1.0, r_cut, eps, 0.4, 10, 600)
    assert set(SIZES) <= set(T.groups()["count"].tolist())
    ref = np.stack(T.force())
    p = tp.treepm_params(1.0, r_cut / 3.0, r_cut, eps, 0.4, 10, 600, tp.TREEPM_FP32)
    ctx = tp.treepm_create(p, 0)
    try:
        tp.treepm_build(ctx, *[torch.from_numpy(a).cuda() for a in (x, y, z, m)])
        st = tp.treepm_walk(ctx)
        assert st.interactions == T.interactions()
        acc = [torch.full((x.size,), 7.0, dtype=torch.float64, device="cuda") for _ in range(3)]
        tp.treepm_force_short(ctx, *acc)
        got = np.stack([a.cpu().numpy() for a in acc])
        assert 0 < tp.treepm_get_stats(ctx).evaluated <= st.interactions
    finally:
        tp.treepm_destroy(ctx)
    B = fp32_error_scale(T, x, y, z, m, eps)
    d = np.linalg.norm(got - ref, axis=0)
    print(f"[gpu-case]   max |da|/(u B) {np.max(d / (2.0 ** -24 * B)):.3f}", flush=True)
    assert np.all(d <= 8 * 2.0 ** -24 * B)
