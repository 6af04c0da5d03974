"""The ends of the CFL range (Eq.24, Omega/dt = Lambda_c/CFL): with an infinite
CFL number the time term leaves the LU-SGS diagonal and the iteration runs on
what is left, as the oracle's does; with CFL 0 (a checkpoint that carries
none, under a fixed CFL) the diagonal is infinite and the state stays as it
is, bit for bit.  Every sweep schedule forms both."""
import numpy as np
import pytest

from oracle import pyoracle as po
from paper_1709_00803_amd import meshgen as mg

pytestmark = pytest.mark.gpu
TAGS = dict(bottom=mg.WALL, top=mg.FARFIELD, left=mg.FREESTREAM, right=mg.OUTFLOW)
FLOW = (0.4, 3.0, 5e4, 3.0)
MESHES = {
    "colour": lambda: (mg.colour_order(mg.random_hybrid(20, 16, seed=3, tags=TAGS))[0], None),
    "natural": lambda: (mg.random_hybrid(20, 16, seed=3, tags=TAGS), None),
    "polygons": lambda: (mg.random_quadtree(4, 1, seed=1, tags=TAGS), None),
    "blocks": lambda: mg.block_order(mg.random_hybrid(20, 16, seed=3, tags=TAGS), 40, "coupled"),
}


@pytest.fixture(scope="module")
def igks():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1709_00803_amd import igks as m
    return m


def solver(igks, name, **opt):
    m, blk = MESHES[name]()
    g = igks.Solver(m, sweep_blocks=blk, chunk=2, **opt)
    g.set_freestream(*FLOW)
    return m, blk, g


@pytest.mark.parametrize("op", [0, 1])
@pytest.mark.parametrize("name,sweep,passes", [("colour", 1, 1), ("natural", 2, 1), ("polygons", 2, 1),
                                               ("blocks", 3, 1), ("blocks", 3, 2)])
def test_infinite_cfl(igks, name, sweep, passes, op):
    print("case", name, sweep, passes, op, flush=True)
    m, blk, g = solver(igks, name, sweep=sweep, block_passes=passes, lusgs_op=op, cfl_init=np.inf, cfl_max=np.inf)
    o = po.Oracle(m, cfl_init=np.inf, cfl_max=np.inf, lusgs_op=op)
    if blk is not None:
        o.set_sweep_blocks(blk)
        o.set_block_passes(passes)
    o.set_freestream(*FLOW)
    o.iterate(2)
    g.iterate(2)
    Wo, Wg = o.get_state(), g.get_state()
    assert g.scalars().iteration == 2 and np.isinf(g.scalars().cfl)
    err = (np.abs(Wg - Wo) / np.abs(Wo).max(axis=1, keepdims=True)).max()
    assert err <= 1e-9, err


@pytest.mark.parametrize("op", [0, 1])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name,sweep,passes", [("colour", 1, 1), ("natural", 2, 1), ("polygons", 2, 1),
                                               ("blocks", 3, 2)])
def test_zero_cfl(igks, name, sweep, passes, precision, op):
    print("case", name, sweep, passes, precision, op, flush=True)
    m, blk, g = solver(igks, name, sweep=sweep, block_passes=passes, precision=precision, lusgs_op=op, cfl_init=5.0,
                       cfl_mode=1)
    g.iterate(2)
    W, sc = g.get_state(), g.scalars()
    sc.cfl = 0.0
    g.set_state(W, sc)
    g.iterate(2)
    assert g.scalars().iteration == 4 and g.scalars().cfl == 0.0
    assert np.array_equal(g.get_state(), W)
