"""Device memory of the step calls: the records of moved particles are there for the length of a call only,
and a simulation or ensemble whose allocator refuses them recomputes the move with the same result. Every
scatter kernel of whole runs is reached here with and without records: per-corner gradient and gradient
tile, single boxes and ensembles in every launch mode, particle IDs, adaptive steps, the half drift."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KEYS = ("cnt", "chi", "nu", "vc", "vs")
BASE = dict(omega_m=0.3, h=0.7, a_init=0.02, a_final=1.0, n_steps=16, spacing=1)
BOXES = [dict(BASE, np_side=32, nm_side=64, box=50.0, x_bytes=1, v_bytes=1, seed=11),
         dict(BASE, np_side=48, nm_side=96, box=75.0, x_bytes=2, v_bytes=2, seed=12),
         dict(BASE, np_side=64, nm_side=64, box=64.0, x_bytes=1, v_bytes=1, seed=13),
         dict(BASE, np_side=32, nm_side=32, box=32.0, x_bytes=1, v_bytes=2, sigma_mode=0, seed=14),
         dict(BASE, np_side=64, nm_side=64, box=64.0, x_bytes=2, v_bytes=1, seed=15)]


def record_bytes(cfg):
    return (16 if cfg["x_bytes"] == 1 else 20) * cfg["np_side"]**3


@pytest.fixture(scope="module")
def lib():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1712_06121_amd as m
    return m


class Memory:
    """A counting device allocator for the library over PyTorch's, with a limit and, on request, another
    place for every allocation."""

    def __init__(self, binding):
        import torch
        self.torch, self.live, self.total, self.peak, self.limit, self.spacers = torch, {}, 0, 0, None, None
        dev, stream = torch.cuda.current_device(), torch.cuda.current_stream()

        def alloc(n, _user):
            if self.limit is not None and self.total + n > self.limit:
                return None
            p = torch.cuda.caching_allocator_alloc(int(n), dev, stream)
            if self.spacers is not None:  # what lies at this address stays taken: the next one is another
                self.spacers.append(p)
                p = torch.cuda.caching_allocator_alloc(int(n), dev, stream)
            self.live[p] = n
            self.total += n
            self.peak = max(self.peak, self.total)
            return p

        def free(p, _user):
            self.total -= self.live.pop(p)
            torch.cuda.caching_allocator_delete(p)

        self.table = binding.CubeAllocator(binding.ALLOC_FN(alloc), binding.FREE_FN(free), None)
        self.stream = binding.c_void_p(stream.cuda_stream)

    def close(self):
        for p in self.spacers or ():
            self.torch.cuda.caching_allocator_delete(p)
        self.spacers = None


@pytest.fixture
def memory(lib, monkeypatch):
    from paper_1712_06121_amd import binding
    m = Memory(binding)
    monkeypatch.setattr(binding, "_torch_env", lambda torch_memory: (m.stream, binding.byref(m.table), [m]))
    yield m
    m.close()


def same(a, b, what):
    for key in KEYS:
        assert np.array_equal(a[key], b[key]), (what, key)


@pytest.mark.parametrize("cfg", BOXES, ids=lambda c: "%d_%d_x%dv%d" % (c["np_side"], c["nm_side"], c["x_bytes"], c["v_bytes"]))
def test_records_live_as_long_as_the_call(lib, memory, cfg):
    with lib.Sim(**cfg) as sim:
        created = memory.total
        assert sim.device_bytes == created
        sim.init_ic()
        assert memory.total == created
        memory.peak = memory.total
        sim.step(6)
        assert memory.total == sim.device_bytes == created  # given back
        assert memory.peak >= created + record_bytes(cfg)  # and there meanwhile
        sim.step(3)
        sim.stage_deposit()
        sim.stage_solve()
        sim.stage_move(0.0, 0.001)
        assert memory.total == created
        want = sim.get_state()
    for variant in (-1, 0, 1):  # refused: by density, per-corner gradient, gradient tile
        with lib.Sim(**cfg) as sim:
            sim.init_ic()
            sim.set_variant(move_variant=variant)
            memory.limit = memory.total
            sim.step(6)
            sim.step(3)
            sim.stage_deposit()
            sim.stage_solve()
            sim.stage_move(0.0, 0.001)
            memory.limit = None
            same(sim.get_state(), want, f"without records, move_variant {variant}")


@pytest.mark.parametrize("pid", [4, 8])
def test_ids_with_and_without_records(lib, memory, pid):
    out = []
    for refuse in (False, True):
        for variant in (0, 1):
            with lib.Sim(**BOXES[2]) as sim:
                sim.enable_pids(pid)
                sim.init_ic()
                sim.set_variant(move_variant=variant)
                memory.limit = memory.total if refuse else None
                sim.step(9)
                memory.limit = None
                out.append((sim.get_state(), sim.get_pids()))
    for state, ids in out[1:]:
        same(state, out[0][0], pid)
        assert np.array_equal(ids, out[0][1])


def test_adaptive_steps_with_and_without_records(lib, memory):
    out = []
    for refuse, variant in ((False, 0), (True, 0), (True, 1)):
        with lib.Sim(**dict(BOXES[2], n_steps=200)) as sim:
            sim.set_adaptive(0.5, 0.05, 0.08)
            sim.init_ic()
            sim.set_variant(move_variant=variant)
            memory.limit = memory.total if refuse else None
            sim.step(12)
            memory.limit = None
            out.append((sim.get_state(), sim.a))
    for state, a in out[1:]:
        same(state, out[0][0], "adaptive")
        assert a == out[0][1]


@pytest.fixture(scope="module")
def alone(lib):
    out = []
    for cfg in BOXES:
        with lib.Sim(**cfg) as sim:
            sim.init_ic()
            sim.step(12)
            out.append(sim.get_state())
    return out


# refused, granted, moved or refused again from call to call: the captured steps follow
@pytest.mark.parametrize("calls", ["rrrr", "gggg", "grgr", "mmmm", "rmgr"])
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_ensembles_with_and_without_records(lib, memory, alone, mode, calls):
    with lib.Batch(BOXES) as b:
        b.set_mode(mode)
        b.init_ic()
        for box, variant in zip(b.boxes, (0, 1, -1, 0, 1)):
            box.set_variant(move_variant=variant)
        created = memory.total
        for what in calls:
            memory.limit = created if what == "r" else None
            memory.spacers = (memory.spacers or []) if what == "m" else memory.spacers
            memory.peak = created
            b.step(3)
            assert memory.total == created
            assert (memory.peak >= created + sum(map(record_bytes, BOXES))) == (what != "r")
        memory.limit = None
        got = [box.get_state() for box in b.boxes]
    for i, state in enumerate(got):
        same(state, alone[i], f"box {i}")


def test_a_job_keeps_within_its_footprint(lib, memory, alone):
    import time
    for i in (0, 1, 2):
        fp = lib.footprint(**BOXES[i])
        memory.peak = 0
        with lib.Server(fp, max_active=2, slice_steps=5) as srv:
            srv.submit(BOXES[i], 7)
            t0, done = time.time(), []
            while not done and time.time() - t0 < 60:
                done = srv.poll()
                time.sleep(0.001)
            assert done == [7] and srv.status(7)[0] == srv.FINISHED
            assert memory.peak <= fp
            with lib.Sim(**BOXES[i]) as sim:  # what the finished job holds: no records
                assert memory.total == 2 * sim.device_bytes
            got = srv.job(7).get_state()
            srv.release(7)
        with lib.Sim(**BOXES[i]) as sim:
            sim.init_ic()
            sim.step(BASE["n_steps"])
            same(got, sim.get_state(), f"job {i}")


@pytest.mark.parametrize("i", [0, 2])
def test_autotune_chooses_the_scatter_for_steps_without_records(lib, memory, alone, i):
    with lib.Sim(**BOXES[i]) as sim:
        sim.init_ic()
        sim.autotune()
        assert sim.variant["move_variant"] == -1  # not timed: by density
        created = memory.total
        memory.limit = created
        sim.step(12)
        memory.limit = None
        same(sim.get_state(), alone[i], "chosen by density")
    with lib.Sim(**BOXES[i]) as sim:
        sim.init_ic()
        memory.limit = memory.total
        sim.autotune()
        assert sim.variant["move_variant"] in (0, 2)  # timed
        sim.step(12)
        memory.limit = None
        same(sim.get_state(), alone[i], "timed")


@pytest.mark.parametrize("mode", [0, 1, 2])
def test_records_wait_for_the_work_that_still_uses_their_memory(lib, alone, mode):
    """PyTorch's allocator hands out the memory of a tensor that has been dropped before the kernels on it
    have run; a batch steps on streams of its own and has to go behind them."""
    import torch
    a = torch.randn(6144, 6144, device="cuda")
    need = sum((record_bytes(c) + 255) // 256 * 256 for c in BOXES)
    with lib.Batch(BOXES) as b:
        b.set_mode(mode)
        b.init_ic()
        for _ in range(4):
            torch.cuda.synchronize()
            x = torch.empty(need // 4, dtype=torch.int32, device="cuda")
            for _ in range(12):  # some tens of milliseconds before the fill
                c = a @ a
            x.fill_(-1)
            x.add_(c[0, 0].to(torch.int32) * 0)
            del x, c
            b.step(3)
        got = [box.get_state() for box in b.boxes]
    for i, state in enumerate(got):
        same(state, alone[i], f"box {i}")
