"""A cell's increment reaches only the cells that the sweep couples it to,
whatever it is.  In mixed precision an SA right-hand side beyond the FP32
range (a wall cell with an eddy viscosity of 1e18: -1.2e39) makes that cell's
SA increment minus infinity, which the clip of nu-tilde at 0 takes; the cell
is its group's first, whose increment lies in the first slot of the ring that
the group sweep keeps.  Cells that are not coupled to it get what the launch
per wavefront gives them, bit for bit."""
import numpy as np
import pytest

from paper_1709_00803_amd import meshgen as mg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def igks():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1709_00803_amd import igks as m
    return m


def plate_wall_cell_first():
    """A plate in colour order, a wall cell of the plate's middle first."""
    m = mg.flat_plate(24, 20)
    colour, x = mg.greedy_colouring(m), 12
    n = np.arange(m.n_cells)
    order = np.lexsort((n, n != x, colour, colour != colour[x]))
    assert order[0] == x
    return mg.renumber(m, order)


def test_infinite_increment_stays_with_its_neighbours(igks):
    m = plate_wall_cell_first()
    out = []
    for sweep in (1, 2):
        print("case sweep", sweep, flush=True)
        g = igks.Solver(m, precision=1, cfl_init=5.0, chunk=1, sweep=sweep, flux_lanes=1)
        g.set_freestream(0.3, 0.0, 1e6, 3.0)
        W = g.get_state()
        W[3] -= 0.5 * (W[1] ** 2 + W[2] ** 2) / W[0]   # gas at rest: the flow's own residual stays small
        W[1:3] = 0.0
        W[4, 0] = 1e18
        g.set_state(W)
        M = g.compute_residual()[4]
        big = np.abs(M) > np.finfo(np.float32).max
        assert M[0] < 0.0 and big[0] and big.sum() == 1
        g.iterate(1)
        out.append(g.get_state())
        g.close()
    assert out[0][4, 0] == 0.0 and (out[0][4] > 0.0).sum() > m.n_cells // 2
    assert np.array_equal(out[0], out[1])
