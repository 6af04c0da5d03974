"""The launches of an iteration that igks_graph_chunk reports, and cuts the
captured graphs by, are none too few with the Roe-matrix operator, whose
inverted diagonal blocks take a launch of their own: prep, flux, gather,
reduce, the blocks, the sweeps, commit."""
import ctypes as C

import pytest

from paper_1709_00803_amd import meshgen as mg

igks = pytest.importorskip("paper_1709_00803_amd.igks")


@pytest.mark.parametrize("sweep", [1, 2])
def test_roe_operator_launches(sweep):
    mesh = mg.flat_plate(8, 300)   # row by row: a wavefront per row and column step, 307
    ctx, o = C.c_void_p(), igks.default_options(sweep=sweep, chunk=100, lusgs_op=1)
    assert igks.igks_create(C.byref(ctx), C.byref(o), C.c_void_p(0x1)) == igks.IGKS_OK
    try:
        keep, args = igks._mesh_args(mesh)
        assert igks.igks_mesh_upload(ctx, *args) == igks.IGKS_OK
        v = [C.c_int32() for _ in range(4)]
        assert igks.igks_mesh_info(ctx, *(C.byref(x) for x in v)) == igks.IGKS_OK
        nlev, it, nl = v[3].value, C.c_int32(), C.c_int32()
        assert nlev == 307
        assert igks.igks_graph_chunk(ctx, C.byref(it), C.byref(nl)) == igks.IGKS_OK
        assert nl.value == (6 + 2 * (nlev - 1) if sweep == 1 else 8)
        assert it.value == min(100, 8192 // nl.value)
    finally:
        igks.igks_destroy(ctx)
