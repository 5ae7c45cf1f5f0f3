"""Forward mode over groups of parameters and strips of walks.

The derivative of a walk's terminal value is linear in the vertices'
velocities: with one parameter per vertex coordinate it gives every other
Jacobian's result.  Jacobians with empty rows, full rows and rows with gaps,
and numbers of parameters and walks on both sides of the kernel's groups (64
parameters, 256 / 64 to 256 walks at a time), against that; sums of doubles in
another order, 1e-12 of their scale.
"""
import numpy as np
import pytest

import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

NSEG = 24


@pytest.fixture(scope="module")
def solver():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2405_12964_amd import Solver
    return Solver.from_scene(scenes.c2_star(n=NSEG, K=2), "fp32")


@pytest.mark.parametrize("N,W", [(1, 1), (1, 257), (2, 127), (3, 65), (23, 9), (32, 8), (33, 5), (64, 4), (65, 3),
                                 (130, 2)])
def test_parameter_groups(solver, N, W):
    rng = np.random.default_rng(N)
    X = torch.tensor(scenes.star_points(5, 3), device="cuda")
    n2 = 2 * NSEG
    solver.set_parameters(n2, np.arange(NSEG + 1) * 2, np.arange(n2), np.tile(np.eye(2), (NSEG, 1)))
    basis = solver.walk_records(X, W, 9, 1, udot=True)["udot"].reshape(-1, n2).cpu().numpy()
    J = rng.normal(size=(NSEG, N, 2)) * (rng.random((NSEG, N, 1)) < rng.choice([0.0, 0.4, 1.0], (NSEG, 1, 1)))
    rows, cols = np.nonzero(J.any(axis=2))
    solver.set_parameters(N, np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=NSEG))]), cols, J[rows, cols])
    want = np.einsum("wvc,vnc->wn", basis.reshape(-1, NSEG, 2), J).reshape(5, W, N)
    scale = np.abs(basis).max() * 10
    got = solver.walk_records(X, W, 9, 1, udot=True)["udot"].reshape(5, W, N).cpu().numpy()
    assert np.abs(got - want).max() <= 1e-12 * scale
    ud, uv, _ = solver.jvp(X, W, 9)
    assert np.abs(ud.cpu().numpy() - got.mean(1)).max() <= 1e-12 * scale
    var = got.var(1, ddof=1) / W if W > 1 else 0 * got[:, 0]
    assert np.abs(uv.cpu().numpy() - var).max() <= 1e-12 * scale ** 2
