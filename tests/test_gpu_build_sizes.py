"""The build at the sizes where its passes change: one and several tiles of the sort (1024 keys
up to 2^18, 4096 above) and of the octree (1024 up to 2^20), the number of sort passes (2^16,
2^21), the sums over tiles taken in the scatter (up to 256 tiles) or by a scan, levels of few
and of many nodes; and each step of the sort's fallback, for boxes whose clumps make runs of
equal high key bits longer than 2048.

The (key, index) order must equal numpy's, and for the smaller boxes the nodes, groups and lists
the oracle's, bit for bit; a second build on the same context must repeat the first.
"""
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


def box(n, clump, side, seed):
    """n particles, uniform and in halos; `clump` of them inside one cube of the given side."""
    if n < 1000:
        x, y, z, m = boxgen.uniform_box(n, seed)
    else:
        x, y, z, m = boxgen.nfw_box(n, max(1, n // 3000), seed)
    rng = boxgen.SplitMix64(seed + 1)
    c = min(clump, n)
    for a in (x, y, z):
        a[:c] = 0.3 + side * rng.uniform(c)
    m = np.exp(rng.uniform(n) * np.log(20.0))
    return x, y, z, m / m.sum()


@pytest.mark.parametrize("n,clump,side", [
    (1, 0, 0.0), (2, 0, 0.0), (63, 0, 0.0), (1023, 0, 0.0), (1024, 0, 0.0), (1025, 0, 0.0),
    (4097, 700, 2.0 ** -9),
    (65536, 1500, 2.0 ** -9), (65537, 1500, 2.0 ** -12),
    (262144, 0, 0.0), (262145, 0, 0.0), (1048576, 0, 0.0), (1048577, 0, 0.0),
    (2097152, 2000, 2.0 ** -12), (2097153, 2000, 2.0 ** -15),
    (30000, 2500, 2.0 ** -9),     # one cell of level 8 holds more than 2048: wider sort
    (30000, 3000, 2.0 ** -16),    # and so does one of level 13.3: all bits
    (500000, 2500, 2.0 ** -12),
    (500000, 3000, 0.0),          # coincident particles, in index order
])
def test_build_sizes(tp, orc, n, clump, side):
    print(f"[gpu-case] build n={n} clump={clump} side={side}", flush=True)
    x, y, z, m = box(n, clump, side, 900 + n % 97)
    r_cut, eps, theta, n_leaf, n_crit = 0.05, 0.001, 0.5, 8, 64
    p = tp.treepm_params(1.0, r_cut / 3.0, r_cut, eps, theta, n_leaf, n_crit, tp.TREEPM_FP64)
    dev = [torch.from_numpy(a).cuda() for a in (x, y, z, m)]
    ctx = tp.treepm_create(p, 0)
    try:
        from test_gpu_sort import _morton
        keys = _morton(x, y, z)
        order = np.lexsort((np.arange(n), keys))
        nodes = []
        for rep in range(2):
            tp.treepm_build(ctx, *dev)
            gk, gi = tp.treepm_export_sorted(ctx)
            np.testing.assert_array_equal(gi, order, err_msg=f"build {rep}")
            np.testing.assert_array_equal(gk, keys[order])
            nodes.append(tp.treepm_export_nodes(ctx))
        for k in nodes[0]:
            np.testing.assert_array_equal(nodes[0][k], nodes[1][k], err_msg=k)
        groups = tp.treepm_export_groups(ctx)
        st = tp.treepm_get_stats(ctx)
        assert groups["count"].sum() == n
        T = orc.Tree(x, y, z, m, 1.0, r_cut, eps, theta, n_leaf, n_crit)
        on, og = T.nodes(), T.groups()
        assert st.n_nodes == on["code"].size and st.n_groups == og["code"].size
        a, b = np.argsort(nodes[0]["code"]), np.argsort(on["code"])
        for k in ("code", "first", "count", "nchild", "mass", "com"):
            np.testing.assert_array_equal(nodes[0][k][a], on[k][b], err_msg=k)
        for k in ("code", "first", "count", "lo", "hi", "xg"):
            np.testing.assert_array_equal(groups[k], og[k], err_msg=k)
        assert st.max_group == og["count"].max()
        if n <= 70000 and clump < 2500:
            assert tp.treepm_walk(ctx).interactions == T.interactions()
    finally:
        tp.treepm_destroy(ctx)


def test_lists_in_the_room_an_earlier_walk_left(tp, orc):
    """Two-pass walks of a used context write the lists into the room that is there without
    waiting for their lengths: a box with more entries than fit, and then boxes that do fit, must
    leave the oracle's lists, alone and in a batch."""
    r_cut, theta, n_leaf, n_crit = 0.06, 0.5, 10, 64
    eps = r_cut / 60
    boxes = [boxgen.nfw_box(3000, 3, 21), boxgen.nfw_box(60000, 100, 2), boxgen.nfw_box(3000, 3, 22),
             boxgen.nfw_box(90000, 9, 23)]
    trees = [orc.Tree(*b, 1.0, r_cut, eps, theta, n_leaf, n_crit) for b in boxes]
    p = tp.treepm_params(1.0, r_cut / 3.0, r_cut, eps, theta, n_leaf, n_crit, tp.TREEPM_FP32)

    def check(ctx, k, what):
        print(f"[gpu-case] room: box {k} {what}", flush=True)
        off, isc, val = tp.treepm_export_lists(ctx)
        oo, oc, ov = trees[k].lists()
        np.testing.assert_array_equal(np.diff(off), np.diff(oo))
        g = np.repeat(np.arange(oo.size - 1), np.diff(oo))
        a, b = np.lexsort((val, isc, g)), np.lexsort((ov, oc, g))
        np.testing.assert_array_equal(isc[a], oc[b])
        np.testing.assert_array_equal(val[a], ov[b])

    ctxs = [tp.treepm_create(p, 0) for _ in range(3)]
    try:
        for k in (0, 1, 2, 3):
            tp.treepm_build(ctxs[0], *[torch.from_numpy(a).cuda() for a in boxes[k]])
            assert tp.treepm_walk(ctxs[0]).interactions == trees[k].interactions()
            check(ctxs[0], k, "alone")
        # a batch of a used context with too little room, a fresh one, and one that fits
        tp.treepm_build(ctxs[1], *[torch.from_numpy(a).cuda() for a in boxes[0]])
        tp.treepm_walk(ctxs[1])
        use = (3, 1, 2)
        for c, k in zip(ctxs, use):
            tp.treepm_build(c, *[torch.from_numpy(a).cuda() for a in boxes[k]])
        outs = [[torch.zeros(boxes[k][0].size, dtype=torch.float32, device="cuda")
                 for _ in range(3)] for k in use]
        tp.treepm_force_short_batch(ctxs, outs)
        for c, k in zip(ctxs, use):
            check(c, k, "batch")
    finally:
        for c in ctxs:
            tp.treepm_destroy(c)
