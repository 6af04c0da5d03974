"""The group sweep with the update in the backward sweep and in a launch of its
own, on both sides of the rule that picks (chunks of 16 cells in the largest
group beyond one a wavefront: more than 80 and a thousandth of the cells):
against one launch per wavefront, bit for bit (the Roe operator to rounding),
with polygons, in a batch with a frozen instance, and in two block passes
against the oracle."""
import numpy as np
import pytest

from oracle import pyoracle as po
from paper_1709_00803_amd import meshgen as mg

pytestmark = pytest.mark.gpu
TAGS = dict(bottom=mg.WALL, top=mg.FARFIELD, left=mg.FREESTREAM, right=mg.OUTFLOW)


@pytest.fixture(scope="module")
def igks():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1709_00803_amd import igks as m
    return m


def spare_chunks(mesh, blk=None):
    """Chunks beyond the first of each wavefront, of the largest block."""
    _, nb = mg.cell_adjacency(mesh)
    blk = np.zeros(mesh.n_cells, int) if blk is None else np.asarray(blk)
    lev = np.zeros(mesh.n_cells, int)
    for i in range(mesh.n_cells):
        low = [lev[j] for j in nb[i] if 0 <= j < i and blk[j] == blk[i]]
        lev[i] = 1 + max(low) if low else 0
    return max((-(-np.bincount(lev[blk == b]) // 16) - 1).sum() for b in np.unique(blk))


# name -> (meshes, update in a launch of its own)
CASES = {
    "below": lambda: ([mg.flat_plate(90, 20)], False),
    "above": lambda: ([mg.flat_plate(100, 20)], True),
    "polygons": lambda: ([mg.cavity_adaptive(40)], True),
    "batch": lambda: ([mg.flat_plate(100, 20), mg.random_hybrid(9, 7, seed=1, tags=TAGS),
                       mg.random_hybrid(40, 30, seed=2, tags=TAGS)], True),
}


@pytest.mark.parametrize("op", [0, 1])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", list(CASES))
def test_update_with_and_after_the_sweep(igks, name, precision, op):
    meshes, split = CASES[name]()
    assert (max(map(spare_chunks, meshes)) > 80 + sum(m.n_cells for m in meshes) // 1000) == split
    out = []
    for sweep in (1, 2):
        print("case", name, precision, op, "sweep", sweep, flush=True)
        b = igks.BatchSolver(meshes, precision=precision, lusgs_op=op, cfl_init=5.0, chunk=3, sweep=sweep, flux_lanes=1)
        for i in range(len(meshes)):
            b.set_freestream(i, 0.3, 0.0, 2e3 * (1 + 9 * (i % 2)), 3.0 if i % 2 else -1.0)
        if name == "batch":
            # a cell of near-vacuum pressure beside one of 1e5 times the others: the update is rejected
            W = b.get_state(2)
            c, kin = W.shape[1] // 2, 0.5 * (W[1] ** 2 + W[2] ** 2) / W[0]
            W[3, c] = kin[c] + 1e-6 * (W[3, c] - kin[c])
            W[3, c + 1] = kin[c + 1] + 1e5 * (W[3, c + 1] - kin[c + 1])
            b.set_state(2, W)
        try:
            b.iterate(6)
        except igks.IgksError as e:
            assert name == "batch", e
        hist = [b.history(i)[:, 4] for i in range(len(meshes))]   # Eq.40
        out.append([(b.get_state(i), hist[i], b.scalars(i).iteration) for i in range(len(meshes))])
        b.close()
    for i, ((x, hx, nx), (y, hy, ny)) in enumerate(zip(*out)):
        assert np.isfinite(x).all() and nx == ny and (nx == 6) == (i < 2)
        if op == 0:
            assert np.array_equal(x, y) and np.array_equal(hx, hy), (name, i)
        else:
            # rounding of the increments (at most the state's size), a few ulp a step
            err = (np.abs(x - y) / np.abs(x).max(axis=1, keepdims=True).clip(1e-300)).max()
            assert err <= (1e-13 if precision == 0 else 1e-5), (name, i, err)


@pytest.mark.parametrize("op", [0, 1])
def test_two_passes_against_oracle(igks, op):
    m = mg.random_hybrid(90, 40, seed=4, tags=TAGS)
    blk = (m.centroids_approx()[:, 0] > 0.8 * m.centroids_approx()[:, 0].max()).astype(np.int32)
    assert spare_chunks(m, blk) > 80 + m.n_cells // 1000
    o = po.Oracle(m, cfl_init=5.0, lusgs_op=op)
    o.set_sweep_blocks(blk)
    o.set_block_passes(2)
    o.set_freestream(0.3, 2.0, 3e3, 3.0)
    g = igks.Solver(m, sweep_blocks=blk, block_passes=2, lusgs_op=op, cfl_init=5.0, chunk=2)
    g.set_freestream(0.3, 2.0, 3e3, 3.0)
    o.iterate(3)
    g.iterate(3)
    Wo, Wg = o.get_state(), g.get_state()
    err = (np.abs(Wg - Wo) / np.abs(Wo).max(axis=1, keepdims=True)).max()
    assert err <= 1e-9, err
