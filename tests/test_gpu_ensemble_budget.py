"""A server whose budget is just above its estimate for one clustered box (320 bytes a particle and
64 MiB): repeated requests on the box, whose context sizes its lists from the walk before, keep within
the budget, all come back, and are the box's own forces bit for bit.  A second box then takes its
place."""
import time

import numpy as np
import pytest

import boxgen
from test_gpu_ensemble import _alone, _params

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0910_0121_amd as t
    t.lib()
    return t


def _request(tp, ens, box_id, p, arr):
    t = tp.treepm_ensemble_submit(ens, box_id, p, *arr)
    out = [np.zeros(len(arr[0]), dtype=np.float32) for _ in range(3)]
    for _ in range(3000):
        rc, _st = tp.treepm_ensemble_poll(ens, t, *out)
        if rc != tp.TREEPM_PENDING:
            break
        time.sleep(0.01)
    assert rc == tp.TREEPM_OK, rc
    return np.stack(out)


def test_repeated_requests_keep_to_the_budget(tp):
    n = 300007
    budget = int((n * 320 + (64 << 20)) * 1.02)
    mesh = 1.0 / round(n ** (1 / 3))
    boxes = [boxgen.nfw_box(n, n // 8000, 41), boxgen.nfw_box(n, n // 3000, 42)]
    ref = [_alone(tp, arr, mesh)[0] for arr in boxes]
    p = _params(tp, mesh)
    ens = tp.treepm_ens_create(0, budget, 4)
    try:
        for k, b in enumerate([0, 0, 0, 0, 1, 1, 0, 0]):
            print(f"[gpu-case] budget request {k} box {b}", flush=True)
            np.testing.assert_array_equal(_request(tp, ens, b, p, boxes[b]), ref[b])
            info = tp.treepm_ens_info(ens)
            assert 0 < info["resident_bytes"] <= budget, info
    finally:
        tp.treepm_ens_destroy(ens)
