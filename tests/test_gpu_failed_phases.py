"""Phases enqueued behind a failed one: their state is the buffer that the failed phase left unwritten,
or holding its new counts beside old offsets. They must not follow it; the state before the failed phase
stays, and the simulation goes on from new particles as if nothing had happened."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

KEYS = ("cnt", "chi", "nu", "vc", "vs")
# four steps of 5e-4 in a: a half drift moves a particle of v = 6000 by 1.5 fine cells
CFG = dict(np_side=32, nm_side=64, box=100.0, omega_m=0.3, a_init=0.998, a_final=1.0, n_steps=4, spacing=1)


@pytest.fixture(scope="module")
def lib():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1712_06121_amd as m
    return m


def cold_cloud(drift0, seed):
    """Uniform particles at rest (but for a little)."""
    g = synth.rng(seed)
    return g.uniform(0.0, 64.0, size=(20011, 3)), g.normal(size=(20011, 3)) * 10.0


def too_fast(drift0, seed):
    """One particle that a half drift carries past the next coarse cell."""
    x, v = cold_cloud(drift0, seed)
    x[7], v[7] = (30.0, 30.0, 31.5), (0.0, 0.0, 6.0 / drift0)
    assert v[7, 2] < 32768.0
    return x, v


def colliding(drift0, seed):
    """Two cold groups that a half drift brings into one cell from either side: the number of particles
    there times their velocity variance passes 2^34, found only after the new counts are written."""
    x, v = cold_cloud(drift0, seed)
    g = synth.rng(seed + 1)
    speed = 1.5 / drift0
    assert 700 * speed**2 > 2.0**34 and speed < 10000.0
    x[:700] = g.uniform(1.0, 3.0, size=(700, 3))
    x[:350, 0] = g.uniform(3.2, 3.9, size=350)
    x[350:700, 0] = g.uniform(8.1, 8.7, size=350)
    v[:700] = 0.0
    v[:350, 0], v[350:700, 0] = speed, -speed
    return x, v


def same(a, b, what):
    for key in KEYS:
        assert np.array_equal(a[key], b[key]), (what, key)


@pytest.mark.parametrize("x_bytes,v_bytes,pid", [(1, 1, 0), (2, 2, 8)])
@pytest.mark.parametrize("cloud,code", [(too_fast, -5), (colliding, -7)])
def test_steps_behind_a_failed_half_drift(lib, cloud, code, x_bytes, v_bytes, pid):
    cfg = dict(CFG, x_bytes=x_bytes, v_bytes=v_bytes)
    with lib.Sim(**cfg) as sim:
        drift0 = sim.get_schedule()[0]
        if pid:
            sim.enable_pids(pid)
        sim.load_particles(*cloud(drift0, 3))
        before, ids = sim.get_state(), sim.get_pids() if pid else None
        with pytest.raises(lib.CubeError) as e:
            sim.step(4)
        assert e.value.code == code and "half drift" in str(e.value)
        assert sim.steps_done == 0
        same(sim.get_state(), before, "after the failed call")
        if pid:
            assert np.array_equal(sim.get_pids(), ids)
        sim.load_particles(*cold_cloud(drift0, 5))
        sim.step(4)
        got = sim.get_state()
    with lib.Sim(**cfg) as sim:
        sim.load_particles(*cold_cloud(drift0, 5))
        sim.step(4)
        same(got, sim.get_state(), "a later run")


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("cloud,code", [(too_fast, -5), (colliding, -7)])
def test_batch_steps_behind_a_failed_half_drift(lib, cloud, code, mode):
    cfgs = [dict(CFG, seed=1), dict(CFG, seed=2)]
    with lib.Batch(cfgs) as b:
        b.set_mode(mode)
        drift0 = b.boxes[0].get_schedule()[0]
        b.boxes[0].load_particles(*cold_cloud(drift0, 5))
        b.boxes[1].load_particles(*cloud(drift0, 3))
        before = b.boxes[1].get_state()
        with pytest.raises(lib.CubeError) as e:
            b.step(4)
        assert e.value.code == code and "box 1" in str(e.value) and "half drift" in str(e.value)
        assert [box.steps_done for box in b.boxes] == [4, 0]
        same(b.boxes[1].get_state(), before, "after the failed call")
        got = b.boxes[0].get_state()
    with lib.Sim(**cfgs[0]) as sim:
        sim.load_particles(*cold_cloud(drift0, 5))
        sim.step(4)
        same(got, sim.get_state(), "the other box")


def test_refused_initial_conditions_leave_no_particles(lib):
    """Displacements of many coarse cells: the new counts and offsets were not written, so nothing may
    take them for a state."""
    cfg = dict(np_side=32, nm_side=64, box=50.0, omega_m=0.3, n_steps=10, spacing=1, seed=5)
    with lib.Sim(**cfg) as sim:
        sim.init_ic()
        want = sim.get_state()
    with lib.Sim(**dict(cfg, sigma8=500.0)) as sim:
        for _ in range(2):
            with pytest.raises(lib.CubeError) as e:
                sim.init_ic()
            assert e.value.code == -5 and sim.n == 0
            for call in (lambda: sim.step(3), sim.get_state, sim.stage_deposit, lambda: sim.stage_move(0.0, 0.0)):
                with pytest.raises(lib.CubeError) as e:
                    call()
                assert e.value.code == -8
        sim.set_state(*(want[key] for key in KEYS))
        same(sim.get_state(), want, "a state set afterwards")


@pytest.mark.parametrize("bad,code", [(float("nan"), -7), (40000.0, -7)])
def test_refused_particles_leave_the_ones_that_were_there(lib, bad, code):
    x, v = cold_cloud(0.0, 9)
    v[11, 1] = bad
    with lib.Sim(**CFG) as sim:
        with pytest.raises(lib.CubeError) as e:
            sim.load_particles(x, v)
        assert e.value.code == code
        with pytest.raises(lib.CubeError) as e:
            sim.step(1)
        assert e.value.code == -8  # there were none
        sim.load_particles(*cold_cloud(0.0, 5))
        sim.step(1)
        before = sim.get_state()
        with pytest.raises(lib.CubeError) as e:
            sim.load_particles(x[:5000], v[:5000])
        assert e.value.code == code and sim.n == 20011 and sim.steps_done == 1
        same(sim.get_state(), before, "after the refused load")
        sim.step(3)
        got = sim.get_state()
    with lib.Sim(**CFG) as sim:
        sim.load_particles(*cold_cloud(0.0, 5))
        sim.step(4)
        same(got, sim.get_state(), "the run goes on")
