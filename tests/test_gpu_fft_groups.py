"""The Poisson solve at the mesh sizes whose column transforms run in larger workgroups, on densities
whose potential is known exactly."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def Sim():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1712_06121_amd import Sim as S
    return S


# per size the column widths, and the largest size in the scratch layout too. FP32 values through 3 x 10
# radix-2 levels each way: about 60 roundings of 6e-8, 4e-6 of the potential at the most
@pytest.mark.parametrize("nm,variant", [
    (256, dict(fft_col_width=8)), (256, dict(fft_col_width=16)),
    (512, dict(fft_col_width=8, fft_z_order=1)), (512, dict(fft_col_width=16)),
    (1024, dict(fft_col_width=4)), (1024, dict(fft_col_width=8, fft_z_order=1)),
    (1024, dict(fft_col_width=8, fft_z_layout=1, fft_z_width=4))])
def test_solve_plane_waves(Sim, nm, variant):
    h = nm // 2
    waves = [((3, 0, 0), 0.5, 0.3), ((0, h // 2 + 5, 0), 0.2, 1.1), ((0, 0, h - 1), 0.1, -0.7), ((h - 1, 2, 1), 0.3, 2.0)]
    i = 2 * math.pi * np.arange(nm) / nm
    delta = np.zeros((nm, nm, nm), np.float32)  # [z, y, x]
    want = np.zeros((64, nm))  # 64 rows along x through cells all over the box
    g = np.random.default_rng(nm)
    rz, ry = g.integers(0, nm, size=64), g.integers(0, nm, size=64)
    for (nx, ny, nz), amp, ph in waves:
        ey, ez = np.exp(1j * ny * i), np.exp(1j * (nz * i + ph)) * amp
        if nx and (ny or nz):  # one slab at a time
            for z in range(nm):
                delta[z] += (np.exp(1j * nx * i)[None, :] * (ez[z] * ey)[:, None]).real.astype(np.float32)
        elif nx:
            delta += (ez[0] * np.exp(1j * nx * i)).real.astype(np.float32)[None, None, :]
        elif ny:
            delta += (ez[0] * ey).real.astype(np.float32)[None, :, None]
        else:
            delta += ez.real.astype(np.float32)[:, None, None]
        k2 = (2 * math.pi / nm) ** 2 * (nx * nx + ny * ny + nz * nz)
        want += -1.5 * 0.3 / k2 * (np.exp(1j * nx * i)[None, :] * (ez[rz] * ey[ry])[:, None]).real
    with Sim(nm // 2, nm, 100.0, omega_m=0.3, x_bytes=1, v_bytes=1) as sim:
        sim.set_variant(**variant)
        sim.set_mesh(delta)
        sim.stage_solve()
        got = sim.get_mesh()[rz, ry].astype(np.float64)
    assert np.abs(got - want).max() / np.abs(want).max() < 1e-5
