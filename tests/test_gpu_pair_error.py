"""Rounding of one pair of the force kernels, against the pair law in extended precision.

u = 2^-53 (FP64) or 2^-24 (FP32); an operation rounds by about 0.4 u RMS.  Below R = r / eta = 0.5
the law's own relative slope in s = (r / r_cut)^2 is at most 1.5.

FP64, isolated pairs on dyadic positions, so that every difference is exact: the law's value (its
edge value, the sum and the product with the mass: 0.4 u each, the mass is 1), s (two operations
and a constant, 0.7 u, times 1.5), the product with d and the scale (0.4 u each) and the scale's own
three constants (0.7 u) make 1.5 u RMS; 2.25 u is asked for.  FP32, treepm_pairwise_f32 along an axis
from the origin, the separation taken as the kernel rounds it: the same with the fit of the table's
pieces (0.4 u RMS) makes 1.3 u; 1.85 u is asked for.  A law whose fifth root is rounded and raised to the
fifth power shows 2 u from that alone, and more from the coefficients."""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

LD = np.longdouble


@pytest.fixture(scope="module")
def tp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0910_0121_amd as t
    t.lib()
    return t


def _law(s, e2):
    """G = g(2 sqrt(s)) / (s + e2)^(3/2), eq. (2)'s first branch."""
    R = 2 * np.sqrt(s)
    g = 1 + R ** 3 * (LD(-8) / 5 + R * R * (LD(8) / 5 + R * (LD(-1) / 2 + R * (
        LD(-12) / 35 + LD(3) / 20 * R))))
    x = s + LD(e2)
    return g / (x * np.sqrt(x))


@pytest.mark.parametrize("crowd", [0, 20000])
@pytest.mark.parametrize("ratio", [1.0 / 256, 1.0 / 60, 1.0 / 8, 1.0])
def test_fp64_pair(tp, ratio, crowd):
    """crowd: so many particles in a far corner, which make the box one of 4e8 interactions."""
    print(f"[gpu-case] fp64 pair eps/r_cut={ratio:.3g} crowd={crowd}", flush=True)
    rng = np.random.default_rng(7)
    r_cut = 2.0 ** -7
    i = np.arange(42)
    c = (np.stack(np.meshgrid(i, i, i, indexing="ij"), -1).reshape(-1, 3) * 2 + 1) / 128.0
    c = c[np.any(np.abs(c - 0.5) > 4 * r_cut, axis=1)]
    n = len(c)
    R = np.where(np.arange(n) % 3 == 0, 10.0 ** rng.uniform(-3, math.log10(0.5), n),
                 rng.uniform(0.0, 0.5, n))
    r = np.maximum(np.round(R * 0.5 * r_cut * 2.0 ** 44), 1.0) / 2.0 ** 44
    h = np.round(r * 2.0 ** 43) / 2.0 ** 44
    a, b = c.copy(), c.copy()
    a[:, 0] -= h
    b[:, 0] = a[:, 0] + r
    pos = np.concatenate([a, b, 0.5 + 0.25 * r_cut * rng.uniform(-0.5, 0.5, (crowd, 3))])
    mesh = r_cut / 3.0
    p = tp.make_params(1.0, mesh, 3.0 * mesh, ratio * r_cut, 0.0, 3, 64, tp.TREEPM_FP64)
    ctx = tp.treepm_create(p, 0)
    try:
        tp.treepm_build(ctx, *[torch.from_numpy(np.ascontiguousarray(pos[:, k])).cuda()
                               for k in range(3)], torch.ones(len(pos), dtype=torch.float64).cuda())
        st = tp.treepm_walk(ctx)
        assert (st.interactions >= 1 << 28) == (crowd > 0)
        acc = [torch.zeros(len(pos), dtype=torch.float64, device="cuda") for _ in range(3)]
        tp.treepm_force_short(ctx, *acc)
        got = acc[0].cpu().numpy()[:n]
    finally:
        tp.treepm_destroy(ctx)
    rc, d = LD(p.r_cut), (b[:, 0] - a[:, 0]).astype(LD)
    ref = _law((d / rc) ** 2, (LD(p.eps) / rc) ** 2) * d / rc ** 3
    rms = float(np.sqrt(np.mean(((got - ref) / ref).astype(np.float64) ** 2)))
    print(f"[gpu-case]   RMS {rms / 2.0 ** -53:.2f} u", flush=True)
    assert rms <= 2.25 * 2.0 ** -53


@pytest.mark.parametrize("ratio", [1.0 / 8000, 1.0 / 256, 1.0 / 60, 1.0 / 8, 1.0])
def test_fp32_pair(tp, ratio):
    print(f"[gpu-case] fp32 pair eps/r_cut={ratio:.3g}", flush=True)
    rng = np.random.default_rng(8)
    r_cut, n = 3.0 / 64, 100000
    p = tp.make_params(1.0, r_cut / 3.0, r_cut, ratio * r_cut, 0.5, 10, 64, tp.TREEPM_FP32)
    R = np.where(np.arange(n) % 3 == 0, 10.0 ** rng.uniform(-3, math.log10(0.5), n),
                 rng.uniform(0.0, 0.5, n))
    xj = np.zeros((n, 3))
    xj[:, 0] = R * 0.5 * r_cut
    got = tp.treepm_pairwise_f32(p, np.zeros((1, 3)), xj, np.ones(n), np.zeros(3))[0][:, 0]
    # the kernel's unit of length, r_cut / sqrt(1 - c) with c the power of two of its table
    e2 = (p.eps / p.r_cut) ** 2
    c = 2.0 ** min(math.floor(math.log2(e2)) - 1, -11)
    d = (xj[:, 0] * (math.sqrt(1.0 - c) / r_cut)).astype(np.float32).astype(LD)
    ref = _law(d * d / (1 - LD(c)), e2) * d / (LD(r_cut) ** 2 * np.sqrt(1 - LD(c)))
    ok = d > 0
    rms = float(np.sqrt(np.mean((((got - ref) / ref)[ok]).astype(np.float64) ** 2)))
    print(f"[gpu-case]   RMS {rms / 2.0 ** -24:.2f} u", flush=True)
    assert rms <= 1.85 * 2.0 ** -24
