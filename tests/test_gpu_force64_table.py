"""The FP64 force from its table, which boxes of at least 2^28 interactions use: a crowd of 17,011
particles that all act on each other (theta = 0), in groups of a few, some dozen and some hundred
particles, inside the box and across its corner, against the oracle."""
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


@pytest.mark.parametrize("centre", [0.37, 0.0])
@pytest.mark.parametrize("n_leaf,n_crit", [(3, 3), (8, 41), (8, 300)])
def test_crowd(tp, orc, n_leaf, n_crit, centre):
    print(f"[gpu-case] fp64 table n_crit={n_crit} centre={centre}", flush=True)
    n, r_cut = 17011, 0.1
    x, y, z, m = boxgen.uniform_box(n, 9)
    # most of it within r_cut / 2 of each other, the rest everywhere
    k = np.arange(n) < n - 500
    p = []
    for a in (x, y, z):
        q = np.where(k, centre + 0.5 * r_cut / np.sqrt(3.0) * (a - 0.5), a) % 1.0
        p.append(np.where(q < 1.0, q, 0.0))
    T = orc.Tree(*p, m, 1.0, r_cut, r_cut / 60, 0.0, n_leaf, n_crit)
    ctx = tp.treepm_create(tp.make_params(1.0, r_cut / 3.0, r_cut, r_cut / 60, 0.0, n_leaf, n_crit,
                                          tp.TREEPM_FP64), 0)
    try:
        tp.treepm_build(ctx, *[torch.from_numpy(a).cuda() for a in (*p, m)])
        st = tp.treepm_walk(ctx)
        assert st.interactions == T.interactions() >= 1 << 28
        acc = [torch.zeros(n, dtype=torch.float64, device="cuda") for _ in range(3)]
        tp.treepm_force_short(ctx, *acc)
        got = np.stack([a.cpu().numpy() for a in acc])
    finally:
        tp.treepm_destroy(ctx)
    ref = np.stack(T.force())
    # the tolerance of the FP64 force everywhere else
    assert np.all(np.abs(got - ref) <= 1e-13 * T.error_scale()[None, :] + 1e-300)
