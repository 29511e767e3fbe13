"""The arithmetic first guess of the velocity code (FP32 arctangent, the table near the middle of two
codes): the kernel's formula in NumPy against the exact edges, on the CPU, and the kernel itself against
the oracle's codes."""
import numpy as np
import pytest

import synth
from oracle import twin

C = [0.9999993443489075, -0.33329859375953674, 0.19946563243865967, -0.13908620178699493, 0.09642171859741211,
     -0.05591198801994324, 0.021862726658582687, -0.004054504446685314]
F = np.float32


def guess(u, m, ulp):
    """x = (M / pi) atan(u) as the kernel forms it, its reciprocal off by ulp units in the last place."""
    a = np.abs(u)
    with np.errstate(over="ignore", divide="ignore"):
        r = (1.0 / a.astype(np.float64)).astype(F)
    if ulp:
        r = np.nextafter(r, F(np.inf) if ulp > 0 else F(0))
    z = np.minimum(a, r)
    w = z * z
    cs = [F(c * m / np.pi) for c in C]
    p = np.full_like(w, cs[7])
    for c in cs[6::-1]:
        p = (p.astype(np.float64) * w + np.float64(c)).astype(F)
    zp = z * p
    return np.copysign(np.where(a > 1, F(m / 2) - zp, zp), u)


@pytest.mark.parametrize("m,margin", [(255, 1e-4), (65535, 0.012)])
def test_guess_is_the_code_away_from_the_edges(m, margin):
    h = (m - 1) // 2
    e = np.tan(np.pi * (np.arange(-(h - 1), h + 1) - 0.5) / m)
    f = e.astype(F)
    f = np.where(f < e, np.nextafter(f, F(np.inf)), f)  # the smallest float not below the edge
    ext = np.concatenate([[F(-np.inf)], f, [F(np.inf)]])
    g = synth.rng(m)
    u = [f, np.nextafter(f, F(-np.inf)), np.nextafter(f, F(np.inf)), np.tan(np.pi * (g.random(500000) - 0.5)).astype(F),
         (10 ** g.uniform(-30, 30, 500000) * g.choice([-1, 1], 500000)).astype(F),
         np.array([0, -0.0, 1, -1, 3e38, -3e38, 1e-45], F)]
    u = np.concatenate(u)
    want = np.searchsorted(f, u, side="right") - h
    for ulp in (-1, 0, 1):
        x = guess(u, m, ulp)
        r = np.rint(x)
        nu = np.clip(r, -h, h).astype(np.int64)
        near = ~(np.abs(x - r) <= F(0.5) - F(margin))
        step = nu + (u >= ext[nu + h + 1]) - (u < ext[nu + h])
        assert np.array_equal(np.where(near, step, nu), want)


@pytest.mark.gpu
@pytest.mark.parametrize("nchi,nnu", [(1, 1), (2, 1), (1, 2), (2, 2)])
def test_codes_of_heavy_tails(nchi, nnu):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1712_06121_amd import Sim
    g = synth.rng(11 + nnu)
    n, nm = 300007, 32
    x = g.random((n, 3)) * nm
    v = np.clip(np.tan(np.pi * (g.random((n, 3)) - 0.5)), -2000.0, 2000.0) * 0.05
    ref = twin.load(x, v, nm // 4, nchi, nnu, 1)
    with Sim(32, nm, 100.0, x_bytes=nchi, v_bytes=nnu, capacity=n) as sim:
        sim.load_particles(x, v)
        got = sim.get_state()
    assert np.abs(ref.nu.astype(np.int64)).max() > 0.98 * (128 if nnu == 1 else 32768)
    for name in ("cnt", "chi", "nu", "vc", "vs"):
        assert np.array_equal(got[name], getattr(ref, name)), name
