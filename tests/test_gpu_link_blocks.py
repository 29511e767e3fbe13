"""Offsets and dispersions of a move's new cells where their sums over the link blocks change kind,
against the step reference, bit for bit."""
import numpy as np
import pytest

import synth
from oracle import twin

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def Sim():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1712_06121_amd import Sim as S
    return S


# 2, 54, 1024 (the last without a scan of its own) and 3456 blocks of 256 cells; one particle, and a
# crowded corner whose block holds half of them
@pytest.mark.parametrize("sigma_mode", [0, 1])
@pytest.mark.parametrize("nm,n,clump", [(32, 1, 0.0), (32, 5003, 0.5), (96, 20011, 0.5), (256, 30011, 0.5), (384, 30011, 0.5)])
def test_offsets_and_dispersion(Sim, nm, n, clump, sigma_mode):
    x, v = synth.particle_cloud(17 + n, n, nm, vscale=0.6, clump_frac=clump, n_clumps=1, clump_radius=1.0)
    st = twin.load(x, v, nm // 4, 1, 1, sigma_mode)
    kf, df = np.float32(0.0), np.float32(0.7)
    exp = twin.move(st, np.zeros((nm, nm, nm), np.float32), kf, df, sigma_mode=sigma_mode)
    with Sim(max(32, nm // 2), nm, 100.0, x_bytes=1, v_bytes=1, sigma_mode=sigma_mode, capacity=n) as sim:
        sim.set_state(st.cnt, st.chi, st.nu, st.vc, st.vs)
        sim.set_mesh(np.zeros((nm, nm, nm), np.float32))
        sim.stage_move(kf, df)
        got = sim.get_state()
    for name in ("cnt", "chi", "nu", "vc", "vs"):
        assert np.array_equal(got[name], getattr(exp, name)), name
