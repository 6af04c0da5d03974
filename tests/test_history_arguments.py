"""history(max_entries) of a context that has none: an empty array of the
history's width, and a negative count is refused (it sized an array once)."""
import ctypes as C

import pytest

igks = pytest.importorskip("paper_1709_00803_amd.igks")


@pytest.mark.parametrize("cls,args", [("Solver", ()), ("BatchSolver", (1,))])
def test_history_entries(cls, args):
    s = object.__new__(getattr(igks, cls))
    s.ctx = C.c_void_p()
    o = igks.default_options()
    # a context with a caller's stream touches no device before a workspace is bound
    assert igks.igks_batch_create(C.byref(s.ctx), C.byref(o), C.c_void_p(0x1), 2) == igks.IGKS_OK
    try:
        for n in (0, 1, 1 << 20):
            assert s.history(*args, max_entries=n).shape == (0, igks.HIST_W)
        with pytest.raises(ValueError):
            s.history(*args, max_entries=-1)
    finally:
        s.close()
