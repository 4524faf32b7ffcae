"""Sweep calls captured into a graph and replayed, against the oracle: what the
graph holds outlives later calls, and every replay starts where the last call
or replay left the state."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2506_16240_amd import micsa as M

pytestmark = pytest.mark.gpu


class Run:
    """A lattice on a stream of its own beside the oracle."""

    def __init__(self, shape, n_sweeps=400, gamma=1, period=4, layout=M.LAYOUT_BYTE, kernel=M.KERNEL_AUTO):
        self.stream = torch.cuda.Stream()
        self.gamma, self.period, self.n = gamma, period, n_sweeps
        self.g = M.Lattice(*shape, 0x6AF, stream=self.stream, gamma=gamma, layout=layout)
        self.g.set_option(M.OPT_SWEEP_KERNEL, kernel)
        self.o = O.Lattice(*shape, 0x6AF, gamma=gamma)
        self.schedule(2.5, 0.5)

    def schedule(self, T0, T1):
        self.g.set_schedule(M.Schedule(M.SCHED_LINEAR, T0, T1, self.n, self.period))
        self.os = O.Schedule(O.SCHED_LINEAR, T0, T1, self.n, self.period)

    def eager(self, algo, n):
        self.g.sweep(algo, n)
        self.o.run(algo, self.os, n, 0)

    def capture(self, call, n):
        """call(lattice) of n sweeps into a graph; the counter moves on."""
        graph, k, sched = torch.cuda.CUDAGraph(), self.o.k, self.os
        with torch.cuda.graph(graph, stream=self.stream):
            call(self.g)
        self.o.k += n
        return graph, k, n, sched

    def replay(self, algo, cap, stride=0):
        graph, k, n, sched = cap
        with torch.cuda.stream(self.stream):
            graph.replay()
        torch.cuda.synchronize()
        after, self.o.k = self.o.k, k
        out = self.o.run(algo, sched, n, stride)
        self.o.k = after
        return out

    def logs(self, algo, n, stride):
        """A call that logs to device memory, its logs on the host."""
        E, D = self.rows(n // stride), self.rows(n // stride)
        self.g.sweep_logged_d(algo, n, stride, E, D)
        torch.cuda.synchronize()
        return E.cpu().numpy(), D.cpu().numpy()

    def rows(self, n):
        return torch.zeros((n, self.g.S * self.g.R), dtype=torch.int64, device="cuda")

    def same(self):
        E, D = self.o.energy(), self.o.daemon_energy()
        assert np.array_equal(self.g.energy(), E) and np.array_equal(self.g.daemon_energy(), D)
        assert np.array_equal(self.g.spins(), self.o.sigma), "spins differ"
        assert np.array_equal(self.g.daemons(), self.o.m), "daemons differ"
        assert np.array_equal(self.g.energy(), E) and np.array_equal(self.g.energy_tally(), E)


def same_logs(got, want):
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])


@pytest.mark.parametrize("algo", [M.ALGO_MICSA, M.ALGO_HEATBATH, M.ALGO_METROPOLIS])
@pytest.mark.parametrize("shape", [(16, 16, 16, 1, 512), (64, 64, 64, 1, 2)])
def test_a_graph_outlives_larger_calls_and_other_schedules(shape, algo):
    """A short call is captured; longer calls, which need larger buffers for
    their draws, and a schedule of other temperatures follow; then a replay."""
    r = Run(shape)
    r.eager(algo, 1)
    r.same()
    cap = r.capture(lambda g: g.sweep(algo, 5), 5)
    r.eager(algo, 20)
    r.schedule(1.1, 0.9)
    r.eager(algo, 9)
    r.same()
    r.replay(algo, cap)
    r.same()
    big = r.capture(lambda g: g.sweep(algo, 20), 20)  # grows inside the capture where it has to
    r.replay(algo, big)
    r.same()
    r.replay(algo, cap)
    r.same()
    r.g.close()


@pytest.mark.parametrize("algo", [M.ALGO_MICSA, M.ALGO_HEATBATH])
@pytest.mark.parametrize("shape", [(16, 16, 16, 1, 3), (64, 64, 64, 1, 2)])
def test_captured_logs_outlive_longer_logs(shape, algo):
    """A call that logs to device memory, captured; longer logged calls, to the
    host and to the device, follow."""
    r = Run(shape)
    E, D = r.rows(3), r.rows(3)
    r.eager(algo, 2)
    r.same()
    cap = r.capture(lambda g: g.sweep_logged_d(algo, 6, 2, E, D), 6)
    same_logs(r.g.sweep_logged(algo, 40, 1), r.o.run(algo, r.os, 40, 1))
    same_logs(r.logs(algo, 60, 1), r.o.run(algo, r.os, 60, 1))
    for _ in range(2):
        want = r.replay(algo, cap, 2)
        same_logs((E.cpu().numpy(), D.cpu().numpy()), want)
        r.same()
    r.g.close()


CASES = [  # shape, gamma, algorithm, kernel, layout, sweeps captured
    ((16, 16, 16, 1, 3), 1, M.ALGO_MICSA, M.KERNEL_AUTO, M.LAYOUT_BYTE, 3),      # one work-group, in place
    ((64, 64, 64, 1, 2), 1, M.ALGO_MICSA, M.KERNEL_AUTO, M.LAYOUT_BYTE, 3),      # tiles, one launch: the other copy
    ((64, 64, 64, 1, 2), 1, M.ALGO_HEATBATH, M.KERNEL_AUTO, M.LAYOUT_BYTE, 3),   # the same, levels stay
    ((16, 16, 16, 1, 3), 1, M.ALGO_WALKERS, M.KERNEL_AUTO, M.LAYOUT_BYTE, 3),    # a wandering owed, of either parity
    ((64, 64, 64, 1, 1), 1, M.ALGO_WALKERS, M.KERNEL_AUTO, M.LAYOUT_BYTE, 4),
    ((16, 16, 16, 1, 3), 3, M.ALGO_WALKERS, M.KERNEL_AUTO, M.LAYOUT_BYTE, 4),    # families owe, a call inside a timestep
    ((72, 34, 34, 1, 2), 2, M.ALGO_WALKERS, M.KERNEL_AUTO, M.LAYOUT_BYTE, 6),
    ((24, 4, 600, 1, 1), 2, M.ALGO_MICSA, M.KERNEL_AUTO, M.LAYOUT_BYTE, 3),      # families in the other copy, tiles
    ((32, 16, 8, 1, 2), 1, M.ALGO_WALKERS, M.KERNEL_SIMPLE, M.LAYOUT_BYTE, 3),   # byte arrays
    ((128, 16, 8, 1, 2), 1, M.ALGO_MICSA, M.KERNEL_FUSED, M.LAYOUT_BYTE, 5),     # byte arrays in the other copy
    ((128, 16, 8, 1, 2), 1, M.ALGO_WALKERS, M.KERNEL_FUSED, M.LAYOUT_BYTE, 5),
    ((128, 16, 8, 1, 2), 1, M.ALGO_METROPOLIS, M.KERNEL_FUSED, M.LAYOUT_BYTE, 3),
    ((256, 16, 8, 1, 1), 1, M.ALGO_MICSA, M.KERNEL_MULTISPIN, M.LAYOUT_BYTE, 9),
    ((256, 16, 8, 1, 1), 1, M.ALGO_WALKERS, M.KERNEL_MULTISPIN, M.LAYOUT_BYTE, 5),
    ((16, 6, 10, 65, 2), 1, M.ALGO_MICSA, M.KERNEL_AUTO, M.LAYOUT_BITPLANE, 9),  # cell planes
    ((16, 6, 10, 65, 2), 1, M.ALGO_MICSA, M.KERNEL_AUTO, M.LAYOUT_BITPLANE, 3),  # words, other copy, on a fresh state
]


@pytest.mark.parametrize("start", ["fresh", "swept", "read"])
@pytest.mark.parametrize("case", CASES)
def test_replays_start_where_the_state_is(case, start):
    """Captured on a fresh state, after sweeps that nothing has read yet, and
    after a read: reads before the first replay, two replays in a row, replays
    after calls of other lengths and another algorithm, after written spins and
    written daemons."""
    shape, gamma, algo, kernel, layout, n = case
    r = Run(shape, gamma=gamma, kernel=kernel, layout=layout)
    if start != "fresh":
        r.eager(algo, 2 * gamma + 3)
    if start == "read":
        r.same()
    cap = r.capture(lambda g: g.sweep(algo, n), n)
    r.same()
    for before in (0, 0, 1, 2 * gamma + 2):
        if before:
            r.eager(algo, before)
        r.replay(algo, cap)
        if before != 1:
            r.same()
    if layout == M.LAYOUT_BYTE:
        r.eager(M.ALGO_HEATBATH, 3)
        r.replay(algo, cap)
    r.g.write_spins(1 - r.o.sigma)
    r.o.sigma = 1 - r.o.sigma
    r.replay(algo, cap)
    r.same()
    m = np.ascontiguousarray(r.o.m[..., ::-1])
    r.g.write_daemons(m)
    r.o.m[...] = m
    r.replay(algo, cap)
    r.replay(algo, cap)
    assert np.array_equal(r.g.energy(), r.o.energy())
    image = r.g.save()
    r.replay(algo, cap)
    r.same()
    r.g.load(image)
    r.eager(algo, 2)
    r.g.close()


def test_calls_that_wait_are_refused_in_a_capture():
    """Reads, writes, schedules and host logs inside a capture: ESTATE, nothing
    changed, and the capture goes on."""
    r = Run((16, 16, 16, 1, 2))
    r.eager(M.ALGO_MICSA, 3)
    state = r.o.sigma.copy()

    def call(g):
        for refused in (g.energy, g.daemon_energy, g.energy_tally, lambda: g.overlap(0, 1), g.spins, g.daemons, g.couplings,
                        g.c4_sums, g.c4_sums_static, g.xi, g.save, lambda: g.write_spins(state),
                        lambda: g.write_daemons(state), lambda: r.schedule(1.0, 1.0),
                        lambda: g.sweep_logged(M.ALGO_MICSA, 4, 2)):
            with pytest.raises(M.MicsaError) as e:
                refused()
            assert e.value.status == M.ESTATE
        g.sweep(M.ALGO_MICSA, 3)

    cap = r.capture(call, 3)
    r.same()
    r.replay(M.ALGO_MICSA, cap)
    r.same()
    r.g.close()
