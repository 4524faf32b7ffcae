"""What calls promise beside their results: what has ended when they return,
and what they do where device memory is short."""
import ctypes
import os
import shutil
import subprocess
import threading

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2506_16240_amd import micsa as M
from paper_2506_16240_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", [M.LAYOUT_BYTE, M.LAYOUT_BITPLANE])
def test_writes_have_ended_when_they_return(layout):
    """The tally of written spins too, so that work on another stream (a
    replayed graph) may follow a write."""
    stream = torch.cuda.Stream()
    g = M.Lattice(256, 128, 128, 1, 4, 3, layout=layout, stream=stream)
    spins, daemons = g.spins(), g.daemons()
    for _ in range(3):
        g.write_spins(spins)
        assert stream.query()
        g.write_daemons(daemons)
        assert stream.query()
    assert np.array_equal(g.energy(), g.energy_tally())
    g.close()


class Memory:
    """What the library holds of device memory, and a bound on it."""

    def __init__(self, shim):
        self.shim = shim
        shim.alloc_live.restype = ctypes.c_size_t
        shim.pinned_calls.restype = ctypes.c_long
        shim.alloc_limit.argtypes = [ctypes.c_size_t]

    def pinned(self):
        return self.shim.pinned_calls()

    def held(self):
        return self.shim.alloc_live()

    def bound(self, more=None):
        """At most `more` bytes beyond what is held now; None: no bound."""
        self.shim.alloc_limit(2 ** 64 - 1 if more is None else self.held() + more)


@pytest.fixture(scope="module")
def counted(tmp_path_factory):
    """A copy of the library whose device allocations can be counted and bounded."""
    d = tmp_path_factory.mktemp("alloc")
    M.lib()
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-o", str(d / "alloc.so"),
                           os.path.join(os.path.dirname(__file__), "alloc_limit.c"), "-ldl", "-lpthread"])
    shim = ctypes.CDLL(str(d / "alloc.so"), ctypes.RTLD_GLOBAL)
    shutil.copy(M.LIB_PATH, d / "libmicsa.so")
    return Memory(shim), str(d / "libmicsa.so")


@pytest.fixture
def memory(counted, monkeypatch):
    mem, path = counted
    monkeypatch.setattr(M, "LIB_PATH", path)
    monkeypatch.setattr(M, "_lib", None)
    before = mem.held()
    yield mem
    mem.bound()
    mem.shim.pinned_refuse(0)
    assert mem.held() == before


@pytest.mark.parametrize("shape,gamma", [((16, 16, 16, 1, 3), 1), ((64, 64, 64, 1, 1), 1), ((16, 16, 16, 1, 3), 3)])
def test_walkers_without_room_for_their_wandering(memory, shape, gamma):
    """A walker call without memory changes nothing or is made, and leaves
    nothing owed that a read would lack room for."""
    with M.Lattice(*shape, 5, gamma=gamma) as g:
        o = O.Lattice(*shape, 5, gamma=gamma)
        g.set_schedule(M.Schedule(M.SCHED_CONST, 0.9, 0.9, 200, 4))
        os_ = O.Schedule(O.SCHED_CONST, 0.9, 0.9, 200, 4)
        for n in (2 * gamma + 1, 3 * gamma):
            memory.bound(0)
            try:
                g.sweep(M.ALGO_WALKERS, n)
            except M.MicsaError as e:
                assert e.status == M.ENOMEM and g.counters() == (o.k, o.k // gamma // 4)
                memory.bound()
                g.sweep(M.ALGO_WALKERS, n)
            o.run(O.ALGO_WALKERS, os_, n, 0)
            memory.bound(0)
            assert np.array_equal(g.daemon_energy(), o.daemon_energy())
            assert np.array_equal(g.daemons(), o.m) and np.array_equal(g.spins(), o.sigma)
            memory.bound()


@pytest.mark.parametrize("shape,gamma", [((16, 16, 16, 1, 3), 1), ((96, 40, 20, 1, 1), 1), ((16, 16, 16, 1, 3), 6),
                                         ((128, 64, 8, 1, 1), 1)])
def test_walker_calls_allocate_nothing(memory, shape, gamma):
    """The wandering that a call leaves owed needs no second copy of the levels."""
    with M.Lattice(*shape, 5, gamma=gamma) as g:
        g.set_schedule(M.Schedule(M.SCHED_CONST, 0.9, 0.9, 200, 4))
        held = memory.held()
        g.sweep(M.ALGO_WALKERS, 2 * gamma + 1)
        assert memory.held() == held


def _home_bytes(shape, layout):
    """The state's own arrays and the slots of the reductions."""
    N, L, S, R = shape[0] * shape[1] * shape[2], shape[3] * shape[4], shape[3], shape[4]
    G = (S + 63) // 64
    state = 2 * L * N if layout == M.LAYOUT_BYTE else 3 * G * R * N * 8 + G * 6 * N // 2 * 8
    return state + 2 * 512 * max(L, S) + 2048


@pytest.mark.parametrize("part", [0.0, 0.3, 0.7])
@pytest.mark.parametrize("shape,layout", [((32, 32, 32, 1, 16), M.LAYOUT_BYTE), ((64, 64, 64, 1, 2), M.LAYOUT_BYTE),
                                          ((8, 64, 60, 1, 4), M.LAYOUT_BYTE), ((32, 16, 16, 70, 2), M.LAYOUT_BITPLANE)])
def test_sweeps_without_room_for_planes(memory, shape, layout, part):
    """Room for the state alone, or for a part of the planes and drawn levels:
    every call runs, on fewer drawn refreshes or on the state's own arrays."""
    start = memory.held()
    with M.Lattice(*shape, 5, layout=layout) as g:
        full = memory.held() - start
    home = _home_bytes(shape, layout)
    assert full > home
    # 192 KiB for the schedule's tables and small workspaces
    memory.bound(int(home + part * (full - home)) + (192 << 10))
    if layout == M.LAYOUT_BITPLANE:  # the word-wise sweep goes from one copy to the other
        memory.bound(int(home + part * (full - home)) + (192 << 10) + home)
    with M.Lattice(*shape, 5, layout=layout) as g:
        o = O.Lattice(*shape, 5)
        g.set_schedule(M.Schedule(M.SCHED_LINEAR, 2.5, 0.5, 100, 3))
        os_ = O.Schedule(O.SCHED_LINEAR, 2.5, 0.5, 100, 3)
        algos = (M.ALGO_MICSA, M.ALGO_HEATBATH, M.ALGO_METROPOLIS) if layout == M.LAYOUT_BYTE else (M.ALGO_MICSA,)
        for algo in algos:
            g.sweep(algo, 11)
            o.run(algo, os_, 11, 0)
            E, D = g.sweep_logged(algo, 4, 2)
            Eo, Do = o.run(algo, os_, 4, 2)
            assert np.array_equal(E, Eo) and np.array_equal(D, Do)
        memory.bound()  # room again: the next schedule finds it
        g.set_schedule(M.Schedule(M.SCHED_CONST, 0.9, 0.9, 100, 5))
        os_ = O.Schedule(O.SCHED_CONST, 0.9, 0.9, 100, 5)
        g.sweep(M.ALGO_MICSA, 12)
        o.run(O.ALGO_MICSA, os_, 12, 0)
        assert np.array_equal(g.energy(), o.energy())
        assert np.array_equal(g.spins(), o.sigma) and np.array_equal(g.daemons(), o.m)


JOBS = [(8, 1, M.LAYOUT_BYTE), (16, 1, M.LAYOUT_BYTE), (16, 64, M.LAYOUT_BYTE), (32, 5, M.LAYOUT_BYTE),
        (64, 1, M.LAYOUT_BYTE), (64, 3, M.LAYOUT_BYTE), (128, 1, M.LAYOUT_BYTE), (128, 20, M.LAYOUT_BYTE),
        (64, 37, M.LAYOUT_BITPLANE), (16, 100, M.LAYOUT_BITPLANE)]


def _lanes(layout):
    return M.LANES_REPLICAS if layout == M.LAYOUT_BITPLANE else M.LANES_SAMPLES


def _footprint(L, R, layout):
    size = ctypes.c_size_t()
    p = M._params(L, L, L, 1, R, layout, 0, 1, _lanes(layout))
    assert M.lib().micsa_pool_footprint(ctypes.byref(p), ctypes.byref(size)) == M.OK
    return size.value


def _finish(pool, jobs, sweeps, check=lambda: None):
    left = set(jobs)
    for _ in range(100_000):
        pool.step(sweeps)
        check()
        for j in [j for j in left if pool.state(j)[0] == M.JOB_DONE]:
            left.discard(j)
            yield j
        if not left:
            return
    raise AssertionError("jobs left")


def _beside(R, refreshes):
    """Tables, slots of further replicas, padding."""
    return 136 * refreshes + 512 * (R - 1) + 8192


@pytest.mark.parametrize("times", [1, 1.4, 10])
@pytest.mark.parametrize("L,R,layout", JOBS)
def test_a_job_keeps_to_the_budget(memory, L, R, layout, times):
    """Alone in a pool whose budget is its footprint, little more, or plenty, with
    chunks too short for the planes and long ones: never more than the budget is
    held, and nothing once the pool holds no job; the job ends as it does alone."""
    budget = int(_footprint(L, R, layout) * times)
    pool = M.Pool(budget)
    base = memory.held()
    for n, period, sweeps in ((40, 10, 20), (12, 4, 3), (60, 1, 60)):
        sched = M.Schedule(M.SCHED_LINEAR, 2.0, 0.5, n, period)
        memory.bound()
        with M.Lattice(L, L, L, 1, R, 7, layout=layout, lane_mode=_lanes(layout)) as g:
            g.set_schedule(sched)
            g.sweep(M.ALGO_MICSA, n)
            want = g.energy()
        tables = 1 << 20  # of the batched launches, the pool's own (two of them)
        job = pool.submit(L, L, L, 1, R, 7, sched, layout=layout, lane_mode=_lanes(layout))
        most = []
        for j in _finish(pool, [job], sweeps, lambda: most.append(memory.held() - base)):
            assert np.array_equal(pool.lattice(j).energy(), want)
            pool.release(j)
        assert max(most) <= budget + _beside(R, n // period) + 2 * tables
        assert memory.held() - base in (0, tables, 2 * tables)
    pool.close()


def test_a_pool_keeps_to_its_budget(memory):
    """Jobs of many sizes through a budget of a few: what they hold, with what
    lies idle between them, stays within it."""
    budget = int(2.3 * max(_footprint(*j) for j in JOBS))
    pool = M.Pool(budget)
    rng = np.random.default_rng(5)
    specs = [JOBS[k] for k in rng.integers(0, len(JOBS), 40)]
    sched = M.Schedule(M.SCHED_LINEAR, 2.0, 0.5, 30, 10)
    jobs = [pool.submit(L, L, L, 1, R, 7 + i, sched, layout=lay, lane_mode=_lanes(lay))
            for i, (L, R, lay) in enumerate(specs)]
    beside = sum(_beside(R, 3) for _, R, _ in specs) + (2 << 20)

    def check():
        assert memory.held() <= budget + beside

    for j in _finish(pool, jobs, 10, check):
        pool.release(j)
        check()
    pool.close()


@pytest.mark.parametrize("room", [1.05, 0.5])
def test_a_device_with_less_room_than_the_budget(memory, room):
    """Room for little more than one job at a time, and for less than one job's
    planes: every job ends as it does alone."""
    specs = [(32, 6, M.LAYOUT_BYTE), (64, 2, M.LAYOUT_BYTE), (32, 6, M.LAYOUT_BYTE), (64, 2, M.LAYOUT_BYTE)]
    sched = M.Schedule(M.SCHED_LINEAR, 2.0, 0.5, 30, 10)
    alone = []
    for i, (L, R, _) in enumerate(specs):
        with M.Lattice(L, L, L, 1, R, 7 + i) as g:
            g.set_schedule(sched)
            g.sweep(M.ALGO_MICSA, 30)
            alone.append((g.energy(), g.daemon_energy()))
    pool = M.Pool(1 << 34)
    for j in _finish(pool, [pool.submit(8, 8, 8, 1, 1, 1, sched)], 5):
        pool.release(j)
    memory.bound(int(room * max(_footprint(*s) for s in specs)))
    jobs = {pool.submit(L, L, L, 1, R, 7 + i, sched): i for i, (L, R, _) in enumerate(specs)}
    for j in _finish(pool, jobs, 10):
        lat = pool.lattice(j)
        for got, want in zip((lat.energy(), lat.daemon_energy()), alone[jobs[j]]):
            assert np.array_equal(got, want)
        pool.release(j)
    pool.close()


def test_contexts_of_a_pool_in_several_threads():
    """Finished jobs read, swept on and released from threads of their own
    (releases under the pool's caller's lock) while the pool admits others."""
    pool, lock = M.Pool(1 << 30), threading.Lock()
    s1, s2 = M.Schedule(M.SCHED_LINEAR, 2.0, 0.5, 30, 10), M.Schedule(M.SCHED_CONST, 0.8, 0.8, 40, 5)
    specs = [(16, 3), (64, 1), (32, 2), (16, 40), (64, 2), (32, 1)] * 4
    jobs = {pool.submit(L, L, L, 1, R, 50 + i, s1): (L, R, 50 + i) for i, (L, R) in enumerate(specs)}
    got, threads = {}, []

    def use(j, lat):
        a = lat.energy()
        lat.set_schedule(s2)
        lat.sweep(M.ALGO_HEATBATH, 3)
        lat.sweep(M.ALGO_MICSA, 7)
        got[j] = a, lat.energy(), lat.spins(), lat.daemons()
        with lock:
            pool.release(j)

    left = set(jobs)
    for _ in range(100_000):
        with lock:
            pool.step(10)
            done = [j for j in left if pool.state(j)[0] == M.JOB_DONE]
            views = {j: pool.lattice(j) for j in done}
        for j in done:
            left.discard(j)
            threads.append(threading.Thread(target=use, args=(j, views[j])))
            threads[-1].start()
        if not left:
            break
    for t in threads:
        t.join(60)
    assert sorted(got) == sorted(jobs)
    pool.close()
    for j, (L, R, seed) in jobs.items():
        with M.Lattice(L, L, L, 1, R, seed) as g:
            g.set_schedule(s1)
            g.sweep(M.ALGO_MICSA, 30)
            want = [g.energy()]
            g.set_schedule(s2)
            g.sweep(M.ALGO_HEATBATH, 3)
            g.sweep(M.ALGO_MICSA, 7)
            want += [g.energy(), g.spins(), g.daemons()]
        for a, b in zip(got[j], want):
            assert np.array_equal(a, b)


def test_contexts_one_after_another_share_what_is_dear_to_allocate(memory):
    """A short life costs no pinned allocation after the first, and little device
    memory; contexts that live at once read through buffers of their own."""
    def life(seed, L=16):
        g = M.Lattice(L, L, L, 1, 1, seed)
        g.set_schedule(M.Schedule(M.SCHED_CONST, 1.5, 1.5, 100, 10))
        g.sweep(M.ALGO_MICSA, 10)
        return g

    life(1).energy()
    before = memory.pinned()
    for seed in range(6):
        with life(seed) as g:
            o = O.Lattice(16, 16, 16, 1, 1, seed)
            o.run(O.ALGO_MICSA, O.Schedule(O.SCHED_CONST, 1.5, 1.5, 100, 10), 10, 0)
            assert np.array_equal(g.energy(), o.energy()) and np.array_equal(g.spins(), o.sigma)
            assert memory.held() < 2 << 20
    assert memory.pinned() == before
    many = [life(s) for s in range(12)]
    for _ in range(2):
        for g, want in zip(many, [M.Lattice(16, 16, 16, 1, 1, s) for s in range(12)]):
            want.set_schedule(M.Schedule(M.SCHED_CONST, 1.5, 1.5, 100, 10))
            want.sweep(M.ALGO_MICSA, 10)
            assert np.array_equal(g.energy(), want.energy()) and np.array_equal(g.daemons(), want.daemons())
            want.close()
    for g in many:
        g.close()


def test_tempering_reads_with_and_without_pinned_memory(memory):
    """Contexts one after another read through one buffer (runs in several pieces);
    where there is no pinned memory a read goes by way of the device."""
    dims, T = (4, 4, 4), np.linspace(0.3, 2.0, 64)
    J = W.gaussian_couplings(*dims, 3)
    o = O.PTLattice(*dims, runs=200, T=T, J=J, seed=9, sweeps=2, algo=O.PT_WALKERS, houdayer=False)
    o.run(2)
    want = o.energies(), o.overlaps()
    pinned = []
    for refuse in (0, 0, 1, 0):
        memory.shim.pinned_refuse(refuse)
        held = [M.PT(*dims, 1, T, J, 1, 2, M.PT_WALKERS, False) for _ in range(9 if refuse else 0)]
        for h in held:
            h.read()  # (idle buffers go to these)
        g = M.PT(*dims, 200, T, J, 9, 2, M.PT_WALKERS, False)
        g.step(2)
        E, Q = g.read()
        assert np.array_equal(E, want[0]) and np.array_equal(Q, want[1])
        g.close()
        for h in held:
            h.close()
        pinned.append(memory.pinned())
    assert pinned[1] == pinned[0]
