"""The autotuner times the group sweep once: what it reports is a launch per
wavefront (1) or, with sweep blocks, a workgroup per block (3), else a
workgroup per instance (2).  The 64x32 plate has 50 and more narrow wavefronts,
which the group sweep takes several times faster, in natural order and in
blocks, so that 2 and 3 are also what it finds."""
import pytest

from paper_1709_00803_amd import meshgen as mg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def igks():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1709_00803_amd import igks as m
    return m


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("blocks", [False, True])
def test_one_group_sweep_candidate(igks, blocks, precision):
    m, blk = mg.flat_plate(64, 32), None
    if blocks:
        m, blk = mg.block_order(m, 128, "coupled")
    s = igks.Solver(m, sweep_blocks=blk, precision=precision, cfl_init=5.0)
    s.set_freestream(0.3, 0.0, 1e4)
    for _ in range(4):
        print("case", blocks, precision, flush=True)
        assert s.autotune(2)[4] == (3 if blocks else 2)
    s.close()
