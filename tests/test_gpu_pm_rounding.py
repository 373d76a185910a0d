"""Rounding of the mesh force on meshes finer than a uniform box needs, where the differences of
neighbouring potentials cancel and the transform's rounding shows.

The yardstick is the FP64 scheme with nothing but its potential rounded to float: a value of white
noise per mesh point.  The library also rounds, after the Green's function, the points once between
the steps of each of the three inverse passes, twice between the passes and once where lines are
paired, each by as much, and the differences and weights of the interpolation: sqrt(1 + 6 + 1) = 2.8
times the yardstick.  4 is asked for.  With the transform's 24 or so additions and its twiddles
rounded to float as well it is over 6."""
import numpy as np
import pytest

import boxgen
import test_gpu_pm as base
from oracle import pm
from oracle.ewald import LongRangeKernel

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

tp = base.tp


@pytest.mark.parametrize("n,n_pm", [(100003, 64), (100003, 128)])
def test_mesh_force_rounding(tp, n, n_pm):
    print(f"[gpu-case] mesh rounding n={n} N={n_pm}", flush=True)
    x, y, z, m = boxgen.uniform_box(n, 5)
    mesh = 1.0 / n_pm
    ctx = tp.treepm_create(tp.make_params(1.0, mesh, 3 * mesh, mesh / 20, 0.5, 10, 128,
                                          tp.TREEPM_FP32), 0)
    try:
        tp.treepm_build(ctx, *[torch.from_numpy(a).cuda() for a in (x, y, z, m)])
        acc = [torch.zeros(n, dtype=torch.float32, device="cuda") for _ in range(3)]
        tp.treepm_force_long(ctx, *acc)
        got = np.stack([a.cpu().numpy() for a in acc], axis=1).astype(np.float64)
    finally:
        tp.treepm_destroy(ctx)
    pos = np.stack([x, y, z], axis=1)
    G = pm.green(n_pm, 1.0, 1.5 * mesh, LongRangeKernel(1.5 * mesh))
    phi = pm.potential(pm.assign(pos, m, 1.0, n_pm), 1.0, G)
    ref = pm.interpolate(pm.mesh_force(phi, 1.0), pos, 1.0)
    one = pm.interpolate(pm.mesh_force(phi.astype(np.float32).astype(np.float64), 1.0), pos, 1.0)
    err, unit = np.sqrt(np.mean((got - ref) ** 2)), np.sqrt(np.mean((one - ref) ** 2))
    print(f"[gpu-case]   {err / unit:.2f} x the rounding of the potential, "
          f"{err / np.sqrt(np.mean(ref ** 2)):.2e} of the force", flush=True)
    assert err <= 4.0 * unit
