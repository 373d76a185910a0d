"""Build, walk and force of one context, each on a stream of its own: a walk that has returned its
statistics has left everything that the force reads, so the results are, bit for bit, those of
one stream.  Boxes whose queues the walk's last workgroup writes (up to 1,024 groups), those whose
queues a launch of their own writes (up to 16,384) and larger ones; each context walks twice, so
that the second force could find the first walk's queues."""
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


def _force(tp, ctx, box, streams, dtype, rounds):
    outs = []
    for k in range(rounds):
        # another box first: its queues are not those of the one that is checked
        p = [a.clone() for a in box]
        if k + 1 < rounds:
            p[0] = torch.remainder(p[0] + 0.37, 1.0)
            p[0][p[0] >= 1.0] = 0.0
            p[1] = torch.flip(p[1], (0,))
        torch.cuda.synchronize()
        tp.treepm_build(ctx, *p, stream=streams[0])
        st = tp.treepm_walk(ctx, stream=streams[1])
        acc = [torch.empty(len(p[0]), dtype=dtype, device="cuda") for _ in range(3)]
        tp.treepm_force_short(ctx, *acc, stream=streams[2])
        torch.cuda.synchronize()
        outs.append((st.interactions, torch.stack(acc).cpu().numpy()))
    return outs[-1]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n,n_crit,lo,hi", [(12011, 64, 1, 1024), (60013, 64, 1025, 16384),
                                            (400009, 128, 1025, 16384), (300007, 8, 16385, 300007)])
def test_three_streams_give_the_result_of_one(tp, n, n_crit, lo, hi, precision):
    print(f"[gpu-case] streams n={n} n_crit={n_crit} {precision}", flush=True)
    x = boxgen.nfw_box(n, max(3, n // 8000), 11)
    box = [torch.from_numpy(a).cuda() for a in x]
    mesh = 1.0 / round(n ** (1 / 3))
    p = tp.make_params(1.0, mesh, 3 * mesh, mesh / 20, 0.5, 8, n_crit,
                       tp.TREEPM_FP64 if precision == "fp64" else tp.TREEPM_FP32)
    dtype = torch.float64 if precision == "fp64" else torch.float32
    one = torch.cuda.Stream()
    got = {}
    for name, streams in (("one", [one] * 3), ("three", [torch.cuda.Stream() for _ in range(3)]),
                          ("default", [torch.cuda.Stream(), torch.cuda.Stream(),
                                       torch.cuda.default_stream()])):
        ctx = tp.treepm_create(p, 0)
        try:
            got[name] = _force(tp, ctx, box, streams, dtype, 3)
            assert lo <= tp.treepm_get_stats(ctx).n_groups <= hi
        finally:
            tp.treepm_destroy(ctx)
    for name in ("three", "default"):
        assert got[name][0] == got["one"][0]
        np.testing.assert_array_equal(got[name][1], got["one"][1])
