"""What calls promise beside their results: what has ended when they return,
and what they do where device memory is short."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2506_16240_amd import micsa as M

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
        shim.alloc_limit.argtypes = [ctypes.c_size_t]

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
    assert mem.held() == before


@pytest.mark.parametrize("shape,gamma", [((16, 16, 16, 1, 3), 1), ((64, 64, 64, 1, 1), 1), ((16, 16, 16, 1, 3), 3)])
def test_walkers_without_room_for_their_wandering(memory, shape, gamma):
    """A walker call takes the room that its wandering will need before it
    changes anything, so that a read never lacks it."""
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
