"""The tempering kernel with field tables, and the reads on the device, at the
sizes where their layouts change: rows of each register length, sides of 2,
work-groups of several temperatures with a last one that is not full, tables
that just fit LDS and ones that do not, odd numbers of sweeps, several lots of
runs per read.  Integer trajectories: parity with the oracle is equality."""
import numpy as np
import pytest

from test_gpu_pt import make, same

pytestmark = pytest.mark.gpu

CASES = [
    # dims, runs, temperatures, sweeps, EMCS
    ((4, 2, 2), 700, 7, 5, 3),
    ((6, 2, 4), 900, 5, 1, 3),
    ((8, 4, 2), 500, 11, 4, 3),
    ((10, 6, 4), 260, 7, 3, 2),
    ((12, 4, 6), 200, 6, 10, 2),
    ((16, 2, 6), 300, 5, 7, 2),
    ((16, 6, 10), 40, 9, 2, 2),   # four temperatures of 60 rows in a work-group
    ((16, 16, 8), 1, 3, 3, 2),    # 128 rows of 16: tables of 132 kB
    ((8, 16, 16), 1, 2, 3, 2),    # 256 rows of 8
    ((12, 14, 12), 2, 3, 5, 2),
    ((16, 16, 16), 1, 2, 2, 1),   # tables too large: the records
]


@pytest.mark.parametrize("dims,runs,temps,sweeps,n", CASES, ids=["x".join(map(str, c[0])) for c in CASES])
def test_walkers_with_field_tables(dims, runs, temps, sweeps, n):
    g, o = make(dims, runs, np.linspace(0.25, 1.9, temps), 77, sweeps)
    assert g.kernel_name == "k_pt_emcs_reg"
    swaps = np.zeros((runs, 2, temps - 1), np.int64)
    g.step(n)
    o.run(n, swaps)
    same(g, o, swaps)
    g.close()


def test_reads_in_several_lots():
    """800 runs of 30 temperatures: more results than the read buffer holds."""
    g, o = make((2, 2, 2), 800, np.linspace(0.5, 2.0, 30), 5, 2)
    swaps = np.zeros((800, 2, 29), np.int64)
    g.step(2)
    o.run(2, swaps)
    same(g, o, swaps)
    g.close()
