"""Groups that are taken in pieces (about a 2^13th of the box's pairs or more, at least 2^13): chunks of
128 particles by segments of 64 list entries or more, at the edges of both: groups of one chunk and
of dozens, lists shorter than a round and of many segments, for the FP32, FP64 and quadrupole
kernels, alone and through shared launches.  Bounds as in the parity suite.
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


def _coincident(n, k, seed):
    """k particles at one point (a level-21 leaf of all of them) in a uniform box."""
    x, y, z, m = boxgen.uniform_box(n, seed)
    x[:k], y[:k], z[:k] = 0.3, 0.6, 0.8
    return x, y, z, m


def _run(tp, box, p):
    x, y, z, m = box
    ctx = tp.treepm_create(p, 0)
    try:
        tp.treepm_build(ctx, *[torch.from_numpy(a).cuda() for a in (x, y, z, m)])
        st = tp.treepm_walk(ctx)
        out = []
        for _ in range(2):
            acc = [torch.full((x.size,), 7.0, dtype=torch.float64, device="cuda")
                   for _ in range(3)]
            tp.treepm_force_short(ctx, *acc)
            out.append(np.stack([a.cpu().numpy() for a in acc]))
        np.testing.assert_array_equal(out[0], out[1])
        return st, out[0]
    finally:
        tp.treepm_destroy(ctx)


# box, n_leaf, n_crit: one group of 3000 (24 chunks, the last of 56); 127, 128, 129 and 2000
# particles at one point; groups of up to 1024 of a clustered box
BOXES = [
    (lambda: boxgen.nfw_box(3000, 5, 3), 8, 4096),
    (lambda: _coincident(4000, 127, 5), 8, 64),
    (lambda: _coincident(4000, 128, 5), 8, 64),
    (lambda: _coincident(4000, 129, 5), 8, 64),
    (lambda: _coincident(6000, 2000, 5), 8, 64),
    (lambda: boxgen.nfw_box(20011, 12, 3), 8, 1024),
]
IDS = ["root", "127", "128", "129", "2000", "nfw"]


@pytest.mark.parametrize("k", range(len(BOXES)), ids=IDS)
def test_fp64(tp, orc, k):
    make, n_leaf, n_crit = BOXES[k]
    print(f"[gpu-case] pieces fp64 {IDS[k]}", flush=True)
    box = make()
    T = orc.Tree(*box, 1.0, 0.1, 0.002, 0.5, n_leaf, n_crit)
    st, got = _run(tp, box, tp.treepm_params(1.0, 0.1 / 3.0, 0.1, 0.002, 0.5, n_leaf, n_crit,
                                             tp.TREEPM_FP64))
    assert st.interactions == T.interactions()
    ref = np.stack(T.force())
    assert np.all(np.abs(got - ref) <= 1e-13 * T.error_scale()[None, :] + 1e-300)


@pytest.mark.parametrize("quad", [False, True], ids=["mono", "quad"])
@pytest.mark.parametrize("k", range(1, len(BOXES)), ids=IDS[1:])
def test_fp32(tp, orc, k, quad):
    from test_gpu_parity import fp32_error_scale
    make, n_leaf, n_crit = BOXES[k]
    print(f"[gpu-case] pieces fp32 {IDS[k]} quad={quad}", flush=True)
    box = make()
    T = orc.Tree(*box, 1.0, 0.1, 0.002, 0.5, n_leaf, n_crit, quadrupole=quad)
    p = tp.make_params(1.0, 0.1 / 3.0, 0.1, 0.002, 0.5, n_leaf, n_crit, tp.TREEPM_FP32,
                       quadrupole=1 if quad else 0)
    st, got = _run(tp, box, p)
    assert st.interactions == T.interactions()
    d = np.linalg.norm(got - np.stack(T.force()), axis=0)
    assert np.all(d <= (20 if quad else 8) * 2.0 ** -24 * fp32_error_scale(T, *box, 0.002))


def test_batch_equals_alone(tp):
    """Boxes with pieces and without through one launch: bit for bit each box's own result."""
    print("[gpu-case] pieces batch", flush=True)
    boxes = [BOXES[5][0](), boxgen.uniform_box(400, 2), _coincident(6000, 2000, 5)]
    p = tp.treepm_params(1.0, 0.1 / 3.0, 0.1, 0.002, 0.5, 8, 256, tp.TREEPM_FP32)
    ctxs = [tp.treepm_create(p, 0) for _ in boxes]
    try:
        alone = []
        for c, b in zip(ctxs, boxes):
            tp.treepm_build(c, *[torch.from_numpy(a).cuda() for a in b])
            tp.treepm_walk(c)
            o = tuple(torch.zeros(len(b[0]), dtype=torch.float32, device="cuda") for _ in range(3))
            tp.treepm_force_short(c, *o)
            alone.append([t.cpu().numpy() for t in o])
        for c, b in zip(ctxs, boxes):
            tp.treepm_build(c, *[torch.from_numpy(a).cuda() for a in b])
        out = [tuple(torch.full((len(b[0]),), 3.0, dtype=torch.float32, device="cuda")
                     for _ in range(3)) for b in boxes]
        tp.treepm_force_short_batch(ctxs, out)
        for a, o in zip(alone, out):
            for u, v in zip(a, o):
                np.testing.assert_array_equal(u, v.cpu().numpy())
    finally:
        for c in ctxs:
            tp.treepm_destroy(c)
