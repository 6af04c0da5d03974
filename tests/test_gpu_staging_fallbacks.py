"""What a context hands out with and without its pinned host memory: states,
wall loads, scalars and histories of the static workspace, whose binding may
allocate nothing, against those of a caller's workspace, and of a batch whose
chunk's results exceed the 4 MiB mailbox against those of short chunks."""
import ctypes as C

import numpy as np
import pytest

from paper_1709_00803_amd import meshgen as mg

pytestmark = pytest.mark.gpu
FLOW = (0.4, 1.0, 2e3, 3.0)


@pytest.fixture(scope="module")
def igks():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1709_00803_amd import igks as m
    return m


def test_static_workspace_copies_the_same(igks):
    import torch
    m = mg.flat_plate(128, 200)   # two slots
    s = igks.Solver(m, chunk=4, cfl_init=5.0)
    s.set_freestream(*FLOW)
    # the same calls on the static workspace, whose context is not one of the class's
    t = object.__new__(igks.Solver)
    t.ctx, stream, o = C.c_void_p(), torch.cuda.Stream(), igks.default_options(chunk=4, cfl_init=5.0)
    assert igks.igks_create(C.byref(t.ctx), C.byref(o), C.c_void_p(stream.cuda_stream)) == igks.IGKS_OK
    try:
        keep, args = igks._mesh_args(m)
        assert igks.igks_mesh_upload(t.ctx, *args) == igks.IGKS_OK
        assert igks.igks_bind_static_workspace(t.ctx) == igks.IGKS_OK
        t.n, t.nwall = s.n, s.nwall
        t.set_freestream(*FLOW)
        for step in range(3):
            print("step", step, flush=True)
            assert s.iterate(6) == t.iterate(6) == 6   # a whole chunk and a part of one
            assert np.array_equal(s.history(), t.history()) and len(s.history()) == 6
            W, V = s.get_state(), t.get_state()
            assert np.array_equal(W, V)
            a, b = s.wall_loads(), t.wall_loads()
            assert a["cl"] == b["cl"] and a["cd"] == b["cd"]
            assert all(np.array_equal(a[k], b[k]) for k in ("cf", "cp", "xw")) and len(a["cf"]) == s.nwall > 0
            sc = s.scalars()
            assert (sc.iteration, sc.cfl, sc.res_inf_prev, sc.res0) == tuple(
                getattr(t.scalars(), k) for k in ("iteration", "cfl", "res_inf_prev", "res0"))
            W[0, ::7] *= 1.0 + 1e-3 * (step + 1)
            s.set_state(W, sc)
            t.set_state(W, sc)
    finally:
        t.close()
    s.close()


def test_results_beyond_the_mailbox(igks):
    n, iters = 300, 12
    out = []
    for chunk in (300, 4):   # 300 x (96 + 48 x 300) bytes: 4.1 MiB; 80 KiB
        print("case chunk", chunk, flush=True)
        b = igks.BatchSolver([mg.cavity(3 + i % 3) for i in range(n)], chunk=chunk, cfl_init=5.0, flux_lanes=1, sweep=2)
        for i in range(n):
            b.set_freestream(i, 0.1 + 1e-3 * (i % 50), 0.0, 100.0 + i)
        hist = [[] for _ in range(n)]
        for _ in range(iters // 4):
            assert b.iterate(4) == 4
            for i in range(n):
                hist[i].append(b.history(i))
        out.append([(np.concatenate(hist[i]), b.get_state(i), b.scalars(i).cfl) for i in range(n)])
        b.close()
    for (ha, Wa, ca), (hb, Wb, cb) in zip(*out):
        assert ha.shape == (iters, igks.HIST_W) and np.array_equal(ha, hb)
        assert np.array_equal(Wa, Wb) and ca == cb
