"""The sweep schedule that binding picks, read from the launches of an
iteration before any binding: a launch per wavefront where the wavefronts of
the largest instance are wide (one workgroup takes 0.31 us for 16 cells of
them), a workgroup per instance where they are many and narrow, however many
instances there are."""
import ctypes as C

import numpy as np
import pytest

from paper_1709_00803_amd import meshgen as mg

igks = pytest.importorskip("paper_1709_00803_amd.igks")


def columns(nx, ny):
    """A plate numbered column by column, the even rows of a column first:
    nx + 1 wavefronts of about ny cells."""
    m = mg.flat_plate(nx, ny, ratio=1.001)
    i, j = np.tile(np.arange(nx), ny), np.repeat(np.arange(ny), nx)
    return mg.renumber(m, np.lexsort((j, j % 2, i)))


@pytest.mark.parametrize("meshes,launched", [
    (lambda: [columns(18, 600)], True),
    (lambda: [columns(18, 300)], False),
    (lambda: [columns(14, 300)], True),                              # 15 wavefronts
    (lambda: [mg.flat_plate(200, 40)] * 40, False),                  # 40 instances of narrow ones
    (lambda: [mg.flat_plate(200, 40), columns(18, 600)], False),     # the wide ones are few beside 239
    (lambda: [columns(18, 200)] * 257, False),                       # two instances on a CU
    (lambda: [columns(18, 300)] * 257, True),
])
def test_picked_schedule(meshes, launched):
    meshes = meshes()
    ctx, o = C.c_void_p(), igks.default_options()
    assert igks.igks_batch_create(C.byref(ctx), C.byref(o), C.c_void_p(0x1), len(meshes)) == igks.IGKS_OK
    try:
        for i, m in enumerate(meshes):
            keep, args = igks._mesh_args(m)
            assert igks.igks_batch_mesh_upload(ctx, i, *args) == igks.IGKS_OK
        v = [C.c_int32() for _ in range(4)]
        assert igks.igks_mesh_info(ctx, *(C.byref(x) for x in v)) == igks.IGKS_OK
        it, nl = C.c_int32(), C.c_int32()
        assert igks.igks_graph_chunk(ctx, C.byref(it), C.byref(nl)) == igks.IGKS_OK
        assert nl.value == (5 + 2 * (v[3].value - 1) if launched else 8)
    finally:
        igks.igks_destroy(ctx)
