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
        assert np.array_equal(self.g.spins(), self.o.sigma), "spins differ"
        assert np.array_equal(self.g.daemons(), self.o.m), "daemons differ"
        assert np.array_equal(self.g.energy_tally(), self.o.energy())


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
