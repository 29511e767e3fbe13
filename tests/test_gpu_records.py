"""The two scatters of a move: from the records of the count pass, and recomputing the move (the one
of boxes whose records do not fit). Same codes, counts, order and IDs, bit for bit, as the FP32 step
reference."""
import numpy as np
import pytest

import synth
from oracle import twin

pytestmark = pytest.mark.gpu

RECOMPUTE = (1 << 22) + 1  # a poll limit other than the default selects the recomputing scatter


@pytest.fixture(scope="module")
def Sim():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1712_06121_amd import Sim as S
    return S


# particles: one, fewer than a wavefront, one short of and one past whole chunks, a crowded cell, many
# cells of few; both meshes put tiles at every face of the box
@pytest.mark.parametrize("nchi,nnu,pid,nm,n,clump", [
    (1, 1, 0, 32, 1, 0.0), (1, 1, 8, 32, 63, 0.0), (1, 1, 0, 32, 4097, 0.95), (1, 1, 4, 64, 100003, 0.5),
    (1, 2, 0, 32, 20011, 0.5), (2, 1, 8, 64, 30011, 0.25), (2, 2, 0, 32, 65, 0.0), (2, 2, 4, 64, 50021, 0.9)])
def test_scatters_agree(Sim, nchi, nnu, pid, nm, n, clump):
    x, v = synth.particle_cloud(301 + n, n, nm, vscale=0.6, clump_frac=clump, n_clumps=2, clump_radius=1.0)
    st = twin.load(x, v, nm // 4, nchi, nnu, 1)
    phi = synth.smooth_potential(11, nm, amp=0.5)
    kf, df = np.float32(-1.3 / 12.0), np.float32(0.5)
    exp = twin.move(st, phi, kf, df, sigma_mode=1)
    got = {}
    for variant in (0, 1):
        for limit in (1 << 22, RECOMPUTE):
            with Sim(32, nm, 100.0, x_bytes=nchi, v_bytes=nnu, capacity=n) as sim:
                sim.set_state(st.cnt, st.chi, st.nu, st.vc, st.vs)
                if pid:
                    sim.enable_pids(pid)
                    sim.set_pids(np.arange(n)[::-1] + 5)
                sim.set_variant(move_variant=variant)
                sim.debug_set_turn_limit(limit)
                sim.set_mesh(phi)
                sim.stage_move(kf, df)
                got[variant, limit] = sim.get_state(), sim.get_pids() if pid else None
    for key, (s, ids) in got.items():
        for name in ("cnt", "chi", "nu", "vc", "vs"):
            assert np.array_equal(s[name], getattr(exp, name)), (key, name)
        if pid:
            assert np.array_equal(ids, got[0, RECOMPUTE][1]) and np.array_equal(np.sort(ids), np.arange(n) + 5), key
