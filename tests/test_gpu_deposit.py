"""The deposit where its sums and its wavefront sums change kind, against the exact integer CIC of the
same codes, bit for bit."""
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


# columns of 4 and of 8 coarse cells; knots of particles around one point in the middle of a cell, at its
# corner (eight cells, at the box's edge too) and spread over some fine cells: fewer and more than 12 lanes
# of a wavefront on one corner cell, below and above the 32-bit sums' 2047 particles in 2^3 cells
@pytest.mark.parametrize("nchi", [1, 2])
@pytest.mark.parametrize("nm,knot,radius,centre", [
    (64, 300, 0.01, 30.4), (64, 2047, 0.01, 34.5), (64, 2048, 0.01, 32.0), (64, 30000, 0.3, 0.0),
    (192, 2047, 0.01, 96.5), (192, 2100, 0.01, 96.0), (192, 40000, 0.4, 191.9), (192, 100000, 2.0, 64.0)])
def test_deposit_knots_bit_exact(Sim, nchi, nm, knot, radius, centre):
    g = synth.rng(7 + knot)
    n = knot + 5003
    x = g.uniform(0.0, nm, size=(n, 3))
    x[:knot] = np.mod(centre + radius * g.uniform(-1.0, 1.0, size=(knot, 3)), nm)
    ref = twin.load(np.where(x >= nm, 0.0, x), np.zeros((n, 3)), nm // 4, nchi, 1)
    with Sim(96 if nm == 192 else 32, nm, 100.0, x_bytes=nchi, capacity=n) as sim:
        sim.set_state(ref.cnt, ref.chi, ref.nu, ref.vc, ref.vs)
        sim.stage_deposit()
        got = sim.get_mesh()
    assert np.array_equal(got, twin.delta_from_rho(twin.deposit_int(ref, nm), n, nchi))
