"""The amplitudes of the initial conditions where their table is largest for its launch, of odd length
or steep, against the oracle's displacement field."""
import numpy as np
import pytest

import synth
from oracle import ic
from oracle.cosmology import Cosmology
from oracle.philox import white_noise_grid

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def Sim():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1712_06121_amd import Sim as S
    return S


# 3 (np/2)^2 + 1 entries: 769 (three workgroups and one entry) to 27649; the bound is that of the whole
# displacement field, FP32 transforms of up to 192^3 (60 roundings of 6e-8)
@pytest.mark.parametrize("np_side,box,n_s,omega_m", [(32, 40.0, 1.0, 0.3), (32, 3000.0, 0.8, 1.0), (48, 75.0, 1.1, 0.1),
                                                     (128, 100.0, 0.96, 0.3), (192, 1500.0, 0.9, 0.25)])
def test_displacement_amplitudes(Sim, np_side, box, n_s, omega_m):
    cfg = dict(synth.WORKLOADS["c1_pm32"], np_side=np_side, nm_side=2 * np_side, nc_side=np_side // 2, box=box, n_s=n_s,
               omega_m=omega_m, omega_l=1.0 - omega_m, seed=77)
    with Sim(**cfg) as sim:
        got = sim.get_ic_displacement()
    cosmo = Cosmology(omega_m, 1.0 - omega_m, h=cfg["h"], sigma8=cfg["sigma8"], n_s=n_s)
    ref = np.stack(ic.displacement_field(white_noise_grid(77, np_side), box, cosmo, cfg["a_init"])) * (2 * np_side / box)
    assert np.linalg.norm(got - ref) / np.linalg.norm(ref) < 1e-5
