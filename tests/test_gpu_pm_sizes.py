"""The long-range force on the larger meshes (the transform's steps of radix 16 x 16, 8 x 8 x 8
and 16 x 8 x 8), against the same scheme in FP64 with torch's FFT on the device: the oracle's
assignment, window and differences, and its kernel through the closed form of the S2 cloud's
transform, which is held against the oracle's quadrature first.  Bar as in the PM suite (a
rounding of about log2(N) u of the mesh's RMS per value).
"""
import math

import numpy as np
import pytest

import boxgen
import test_gpu_pm as base
from oracle import pm
from oracle.ewald import LongRangeKernel

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

tp = base.tp


def _phi_hat(k, eta):
    x = k * eta
    s = 12.0 * (2.0 - 2.0 * torch.cos(x) - x * torch.sin(x)) / x ** 4
    s = torch.where(x < 0.05, 1.0 - x * x / 15.0 + x ** 4 / 560.0, s)
    return -4.0 * math.pi * s * s / (k * k)


def _reference(pos, m, n, eta):
    M = torch.zeros(n ** 3, dtype=torch.float64, device="cuda")
    i0, w = pm.tsc_cloud(pos * n)
    for a in range(3):
        for b in range(3):
            for c in range(3):
                cell = (((i0[:, 0] + a - 1) % n) * n + (i0[:, 1] + b - 1) % n) * n + \
                    (i0[:, 2] + c - 1) % n
                wt = m * w[:, 0, a] * w[:, 1, b] * w[:, 2, c]
                u, inv = np.unique(cell, return_inverse=True)
                M[torch.from_numpy(u).cuda()] += torch.from_numpy(
                    np.bincount(inv, weights=wt)).cuda()
    K = torch.fft.rfftn(M.view(n, n, n))
    del M
    k = 2.0 * math.pi * torch.fft.fftfreq(n, d=1.0 / n, dtype=torch.float64, device="cuda")
    win = torch.sinc(k / (2.0 * math.pi * n)) ** 3  # torch's sinc is sin(pi t) / (pi t)
    kz, wz = k[:n // 2 + 1].abs(), win[:n // 2 + 1]
    for ix in range(n):  # plane by plane: the Green's function is never held as a whole
        kk = torch.sqrt(k[ix] ** 2 + k[:, None] ** 2 + kz[None, :] ** 2)
        G = _phi_hat(kk, eta) / (win[ix] * win[:, None] * wz[None, :]) ** 2
        if ix == 0:
            G[0, 0] = 0.0
        K[ix] *= G
    phi = torch.fft.irfftn(K, s=(n, n, n)) * float(n) ** 3
    del K
    out = np.zeros((len(m), 3))
    for a in range(3):
        for b in range(3):
            for c in range(3):
                p = [torch.from_numpy((i0[:, 0] + a - 1) % n).cuda(),
                     torch.from_numpy((i0[:, 1] + b - 1) % n).cuda(),
                     torch.from_numpy((i0[:, 2] + c - 1) % n).cuda()]
                wt = w[:, 0, a] * w[:, 1, b] * w[:, 2, c]
                for d in range(3):
                    def at(s):
                        q = list(p)
                        q[d] = (q[d] + s) % n
                        return phi[q[0], q[1], q[2]]
                    f = -((2.0 / 3.0) * (at(1) - at(-1)) - (1.0 / 12.0) * (at(2) - at(-2))) * n
                    out[:, d] += wt * f.cpu().numpy()
    return out


@pytest.mark.parametrize("n_pm", [128, 256, 512, 1024])
def test_pm_large_meshes(tp, n_pm):
    base._say(f"pm large mesh N_PM={n_pm}")
    eta = 1.5 / n_pm
    k = np.array([0.3, 1.0, 2.5, 4.0]) / eta
    closed = _phi_hat(torch.from_numpy(k), eta).numpy()
    np.testing.assert_allclose(closed, LongRangeKernel(eta).phi_hat(k), rtol=1e-7)
    x, y, z, m = boxgen.nfw_box(30011, 40, 5)
    got = base._long(tp, x, y, z, m, n_pm)
    ref = _reference(np.stack([x, y, z], axis=1), m, n_pm, eta)
    base._check(got, ref, f"N_PM={n_pm}")
    np.testing.assert_array_equal(got, base._long(tp, x, y, z, m, n_pm))
