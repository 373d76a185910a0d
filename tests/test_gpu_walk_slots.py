"""Walks into a slot per list, sized from the context's last walk: the lists and the forces are
the oracle's when the slots fit, when the next box's lists are too long for them (two passes
again), when they shrink, and for several boxes through shared launches."""
import numpy as np
import pytest

import boxgen
from test_gpu_parity import _assert_lists_equal

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0910_0121_amd as t
    t.lib()
    return t


R_CUT = 0.1


def _boxes():
    dense = boxgen.nfw_box(20011, 3, 5)      # lists several times as long
    return [boxgen.uniform_box(8000, 1), boxgen.uniform_box(9001, 2), dense, dense,
            boxgen.uniform_box(1, 3), boxgen.uniform_box(700, 4)]


def test_slots_follow_the_last_walk(tp, orc):
    p = tp.make_params(1.0, R_CUT / 3.0, R_CUT, R_CUT / 60, 0.5, 8, 64, tp.TREEPM_FP64)
    ctx = tp.treepm_create(p, 0)
    longest = []
    try:
        for k, (x, y, z, m) in enumerate(_boxes()):
            print(f"[gpu-case] slots box {k} n={len(x)}", flush=True)
            T = orc.Tree(x, y, z, m, 1.0, R_CUT, R_CUT / 60, 0.5, 8, 64)
            tp.treepm_build(ctx, *[torch.from_numpy(a).cuda() for a in (x, y, z, m)])
            st = tp.treepm_walk(ctx)
            assert st.interactions == T.interactions()
            _assert_lists_equal(tp, ctx, T, f"box {k}")
            acc = [torch.zeros(len(x), dtype=torch.float64, device="cuda") for _ in range(3)]
            tp.treepm_force_short(ctx, *acc)
            got = np.stack([a.cpu().numpy() for a in acc])
            ref = np.stack(T.force())
            assert np.all(np.abs(got - ref) <= 1e-13 * T.error_scale()[None, :] + 1e-300)
            longest.append(int(np.max(np.diff(T.lists()[0]))))
    finally:
        tp.treepm_destroy(ctx)
    assert longest[2] > 2 * longest[1]       # the dense box did not fit the uniform box's slots


def test_slots_with_room_behind(tp, orc):
    """90,000 groups of one particle: slots of twice the longest list would take 5 GB, so they
    hold four times the mean list and the longer ones go behind them; first sized by a uniform
    box (nothing fits: two passes again), then by the clustered one itself."""
    n, theta = 90000, 0.25
    p = tp.make_params(1.0, R_CUT / 3.0, R_CUT, R_CUT / 60, theta, 2, 1, tp.TREEPM_FP64)
    ctx = tp.treepm_create(p, 0)
    dense = boxgen.nfw_box(n, 6, 5)
    try:
        for k, (x, y, z, m) in enumerate((boxgen.uniform_box(n, 1), dense, dense)):
            print(f"[gpu-case] slots with room behind, box {k}", flush=True)
            T = orc.Tree(x, y, z, m, 1.0, R_CUT, R_CUT / 60, theta, 2, 1)
            length = np.diff(T.lists()[0])
            if k:
                assert 2 * int(length.max()) * len(length) * 4 > 1 << 30
                assert np.any(length > 4 * length.mean())
            tp.treepm_build(ctx, *[torch.from_numpy(a).cuda() for a in (x, y, z, m)])
            st = tp.treepm_walk(ctx)
            assert st.interactions == T.interactions()
            np.testing.assert_array_equal(np.diff(tp.treepm_export_lists(ctx)[0]), length)
            acc = [torch.zeros(n, dtype=torch.float64, device="cuda") for _ in range(3)]
            tp.treepm_force_short(ctx, *acc)
            got = np.stack([a.cpu().numpy() for a in acc])
            ref = np.stack(T.force())
            assert np.all(np.abs(got - ref) <= 1e-13 * T.error_scale()[None, :] + 1e-300)
    finally:
        tp.treepm_destroy(ctx)


def test_slots_in_a_batch(tp, orc):
    boxes = _boxes()[:3]
    p = tp.make_params(1.0, R_CUT / 3.0, R_CUT, R_CUT / 60, 0.5, 8, 64, tp.TREEPM_FP32)
    ctxs = [tp.treepm_create(p, 0) for _ in boxes]
    try:
        # the second round's boxes are rotated: one context's slots are too small, one's fit
        for r in range(3):
            order = [boxes[(k + (r == 1)) % 3] for k in range(3)]
            for c, (x, y, z, m) in zip(ctxs, order):
                tp.treepm_build(c, *[torch.from_numpy(a).cuda() for a in (x, y, z, m)])
            out = [tuple(torch.empty(len(b[0]), dtype=torch.float32, device="cuda")
                         for _ in range(3)) for b in order]
            print(f"[gpu-case] slots batch round {r}", flush=True)
            tp.treepm_force_short_batch(ctxs, out)
            for c, (x, y, z, m) in zip(ctxs, order):
                T = orc.Tree(x, y, z, m, 1.0, R_CUT, R_CUT / 60, 0.5, 8, 64)
                _assert_lists_equal(tp, c, T, f"round {r}")
    finally:
        for c in ctxs:
            tp.treepm_destroy(c)
