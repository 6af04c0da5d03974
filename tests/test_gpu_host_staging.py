"""States through the pinned staging memory: what set_state put in comes back
from get_state bit for bit, at the edges of a slot of 16384 cells, of the
eight slots and of the sizes from which several threads copy; residuals, which
take the same way, against those of the context that copies without it (the
static workspace) on a mesh of two slots."""
import ctypes as C

import numpy as np
import pytest

from paper_1709_00803_amd import meshgen as mg

pytestmark = pytest.mark.gpu
SLOT = 16384


@pytest.fixture(scope="module")
def igks():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1709_00803_amd import igks as m
    return m


def random_state(n, seed):
    g = np.random.default_rng(seed)
    W = np.empty((5, n))
    W[0] = g.uniform(0.5, 2.0, n)
    W[1:3] = g.uniform(-1.0, 1.0, (2, n))
    W[3] = g.uniform(5.0, 9.0, n)
    W[4] = g.uniform(0.0, 1e-3, n)
    return W


@pytest.mark.parametrize("nx,ny", [(1, 1), (127, 129), (128, 128), (113, 145), (256, 448), (241, 476), (393, 417)])
def test_state_round_trip(igks, nx, ny):
    m = mg.flat_plate(nx, ny) if nx > 1 else mg.cavity(1)
    print("case", nx, ny, "slots", -(-m.n_cells // SLOT), flush=True)
    s = igks.Solver(m, sweep=1)
    s.set_freestream(0.4, 1.0, 2e3, 3.0)
    for seed in (1, 2):
        W = random_state(m.n_cells, seed)
        s.set_state(W)
        assert np.array_equal(s.get_state(), W)
    s.close()


def test_residual_with_and_without_staging(igks):
    import torch
    m = mg.flat_plate(128, 200)
    W = random_state(m.n_cells, 3)
    s = igks.Solver(m)
    s.set_freestream(0.4, 1.0, 2e3, 3.0)
    s.set_state(W)
    stream, ctx, o = torch.cuda.Stream(), C.c_void_p(), igks.default_options()
    assert igks.igks_create(C.byref(ctx), C.byref(o), C.c_void_p(stream.cuda_stream)) == igks.IGKS_OK
    try:
        keep, args = igks._mesh_args(m)
        assert igks.igks_mesh_upload(ctx, *args) == igks.IGKS_OK
        assert igks.igks_bind_static_workspace(ctx) == igks.IGKS_OK
        assert igks.igks_set_freestream(ctx, 0.4, 1.0, 2e3, 3.0) == igks.IGKS_OK
        dp = C.POINTER(C.c_double)
        assert igks.igks_set_state(ctx, W.ctypes.data_as(dp), None) == igks.IGKS_OK
        M = np.empty_like(W)
        for _ in range(3):   # the first leaves the slots as it found them
            assert igks.igks_compute_residual(ctx, M.ctypes.data_as(dp)) == igks.IGKS_OK
            assert np.array_equal(s.compute_residual(), M)
    finally:
        igks.igks_destroy(ctx)
    s.close()
