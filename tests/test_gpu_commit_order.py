"""Whether an iteration is committed by a launch of its own (the last of a
chunk) or by the reduction of the next one makes no difference: chunks of one
against a chunk of all iterations, bit for bit, with an instance that is
frozen by a rejected update on the way and one that is not."""
import numpy as np
import pytest

from paper_1709_00803_amd import meshgen as mg

pytestmark = pytest.mark.gpu
TAGS = dict(bottom=mg.WALL, top=mg.FARFIELD, left=mg.FREESTREAM, right=mg.OUTFLOW)
ITERS = 12


@pytest.fixture(scope="module")
def igks():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1709_00803_amd import igks as m
    return m


def run(igks, meshes, starts, chunk, scheme, sweep):
    b = igks.BatchSolver(meshes, scheme=scheme, cfl_init=0.5 if scheme else 5.0, cfl_mode=1, chunk=chunk, sweep=sweep,
                         limiter=1)
    for i in range(len(meshes)):
        b.set_freestream(i, 0.4, 1.0, 2e3, 3.0)
        if starts[i] is not None:
            b.set_state(i, starts[i](b.get_state(i)))
    hist = [[] for _ in meshes]
    for _ in range(ITERS // chunk):
        try:
            b.iterate(chunk)
        except igks.IgksError as e:
            print("frozen:", e, flush=True)
        for i, h in enumerate(hist):
            h.extend(b.history(i))   # of the last call
    out = [(b.get_state(i), np.array(hist[i]), b.scalars(i).iteration, b.scalars(i).cfl) for i in range(len(meshes))]
    b.close()
    return out


def spike(W):
    # a cell of near-vacuum pressure beside one of 1e5 times the others: its update is rejected
    W = W.copy()
    c = W.shape[1] // 2
    kin = 0.5 * (W[1] ** 2 + W[2] ** 2) / W[0]
    W[3, c] = kin[c] + 1e-6 * (W[3, c] - kin[c])
    W[3, c + 1] = kin[c + 1] + 1e5 * (W[3, c + 1] - kin[c + 1])
    return W


@pytest.mark.parametrize("starts", [(None,), (spike,), (None, spike, None)], ids=["one", "frozen", "batch"])
@pytest.mark.parametrize("scheme,sweep", [(1, 0), (0, 1), (0, 2)])
def test_commit_in_next_reduction(igks, starts, scheme, sweep):
    meshes = [mg.random_hybrid(9 + i, 7, seed=i, tags=TAGS, jitter=0.2) for i in range(len(starts))]
    print("case", len(starts), scheme, sweep, flush=True)
    a = run(igks, meshes, starts, 1, scheme, sweep)
    b = run(igks, meshes, starts, ITERS, scheme, sweep)
    for (Wa, ha, na, ca), (Wb, hb, nb, cb), start in zip(a, b, starts):
        assert na == nb and ca == cb
        assert (na < ITERS) == (start is spike)
        assert np.array_equal(Wa, Wb)
        assert len(ha) == min(na + 1, ITERS) and np.array_equal(ha, hb)
