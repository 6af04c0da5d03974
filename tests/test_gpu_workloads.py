"""The workloads that the solver's throughput is followed on (perf/cases.py)
against the array evaluation of the scheme that stands beside them, which
shares no code with the library: states and histories to 1e-9 of each
component's largest value, as elsewhere; a single residual and its wall loads,
where only the cancellation of the face fluxes amplifies rounding (a per cent
and more of them is left), to 1e-10."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cases():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from perf import cases as m
    return m


# name -> what is changed: few iterations, the smaller meshes
PICKED = {
    "loads_hybrid_2k": {},
    "plate_blocks": dict(iters=4),
    "cavity_adaptive_natural": dict(n=12, iters=2),
    "cavity_explicit": dict(iters=10),
    "turbulent_plate_blocks": dict(iters=2),
    "jouk40k_colour": dict(cells=8000, iters=4),
    "jouk250k_two_pass": dict(n_wall=64, layers=30, h1=2e-5, cells=6000, iters=2),
}


def compare(got, want, tol, what):
    got, want = np.atleast_1d(got), np.atleast_1d(want)
    assert got.shape == want.shape, what
    axis = 0 if what == "history" else -1   # per column, per component, or of the whole array
    scale = np.abs(want).max(axis=axis, keepdims=True)
    assert np.isfinite(got).all() and (np.abs(got - want) <= tol * scale).all(), (
        what, (np.abs(got - want) / np.maximum(scale, 1e-300)).max())


@pytest.mark.parametrize("name", list(PICKED))
def test_against_the_array_evaluation(cases, name):
    print("case", name, flush=True)
    case = dict(next(c for c in cases.listed() if c["name"] == name), **PICKED[name])
    want = cases.exact(case, 1)
    assert want is not None
    state = cases.prepare(case, 1)
    got = cases.run(state)
    state["solver"].close()
    assert set(got) == set(want)
    for k in want:
        compare(got[k], want[k], 1e-10 if case.get("call") == "loads" else 1e-9, k)
