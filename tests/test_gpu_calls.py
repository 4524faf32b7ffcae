"""What calls promise beside their results: what has ended when they return,
and what they do where device memory is short."""
import numpy as np
import pytest
import torch

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
