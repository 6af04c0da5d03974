"""Groups whose couplings span more cells than the ring of increments in LDS
holds (152 KiB: 3889 cells in FP64, 7780 in FP32) pass them through global
memory: with polygons (entries beyond the fourth) in colour order, and in
natural order over hundreds of wavefronts, against one launch per wavefront,
bit for bit (the Roe operator to rounding); in two block passes, one block of
which is too large for the ring, against the oracle."""
import numpy as np
import pytest

from oracle import pyoracle as po
from paper_1709_00803_amd import meshgen as mg

pytestmark = pytest.mark.gpu
TAGS = dict(bottom=mg.WALL, top=mg.FARFIELD, left=mg.FREESTREAM, right=mg.OUTFLOW)
FLOW = (0.3, 2.0, 3e3, 3.0)


def polygons(precision):
    """Quadtree cells in colour order: 7606 or 14842 of them (the first colour
    couples to the last), a third with more than four faces."""
    return mg.colour_order(mg.random_quadtree(56 if precision else 40, 2, seed=3, tags=TAGS))[0]


@pytest.fixture(scope="module")
def igks():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1709_00803_amd import igks as m
    return m


def span(mesh):
    """The largest distance in sweep order between coupled cells of a mesh in
    colour order (its sweep order is its own)."""
    _, nb = mg.cell_adjacency(mesh)
    return max(abs(i - j) for i in range(mesh.n_cells) for j in nb[i] if j >= 0)


@pytest.mark.parametrize("mesh,precision,op", [("polygons", 0, 0), ("polygons", 1, 0), ("polygons", 0, 1),
                                               ("polygons", 1, 1), ("natural", 0, 0)])
def test_against_launch_per_wavefront(igks, mesh, precision, op):
    if mesh == "polygons":
        m = polygons(precision)
        assert (np.diff(m.cell_ptr) > 4).sum() > m.n_cells // 4 and span(m) > (7780 if precision else 3889)
        flow = FLOW
    else:
        m = mg.cavity_adaptive(60)   # 576 wavefronts; spans 4912 cells
        flow = (0.17, 0.0, 1000.0)
    out = []
    for sweep in (1, 2):
        print("case", mesh, precision, op, "sweep", sweep, flush=True)
        g = igks.Solver(m, precision=precision, lusgs_op=op, cfl_init=5.0, chunk=3, sweep=sweep, flux_lanes=1)
        g.set_freestream(*flow)
        g.iterate(3)
        out.append(g.get_state())
        g.close()
    assert np.isfinite(out[0]).all()
    if op == 0:
        assert np.array_equal(out[0], out[1])
    else:
        # rounding of the increments (at most the state's size), a few ulp a step
        err = (np.abs(out[0] - out[1]) / np.abs(out[0]).max(axis=1, keepdims=True)).max()
        assert err <= (1e-13 if precision == 0 else 1e-5), err


@pytest.mark.parametrize("precision,op", [(0, 0), (0, 1), (1, 0)])
def test_two_passes_against_oracle(igks, precision, op):
    print("case two passes", precision, op, flush=True)
    m = polygons(precision)
    x = m.centroids_approx()[:, 0]
    blk = (x > np.quantile(x, 0.94)).astype(np.int32)   # the first block's couplings span nearly all of its cells
    o = po.Oracle(m, cfl_init=5.0, lusgs_op=op)
    o.set_sweep_blocks(blk)
    o.set_block_passes(2)
    o.set_freestream(*FLOW)
    g = igks.Solver(m, sweep_blocks=blk, block_passes=2, precision=precision, lusgs_op=op, cfl_init=5.0, chunk=2)
    g.set_freestream(*FLOW)
    o.iterate(2)
    g.iterate(2)
    Wo, Wg = o.get_state(), g.get_state()
    err = (np.abs(Wg - Wo) / np.abs(Wo).max(axis=1, keepdims=True)).max()
    assert err <= (1e-9 if precision == 0 else 1e-5), err
