"""Reflecting-boundary queries at every bound a caller can pass: a negative
cap, zero, an infinite one and one that is not a number answer at once or as
the capped query does (silhouette_d2 takes the cap's square; no ray hit has a
t below zero), beside rows with ordinary caps in the same wavefront."""
import numpy as np
import pytest

import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("dim", [2, 3])
def test_caps_without_a_range(dev, dim, precision):
    from paper_2405_12964_amd import Solver
    sc = scenes.thermal_scene(n_slice=300, K=1) if dim == 2 else scenes.thermal3d_scene(nu_slice=4, nu_wire=2, K=1)
    s = Solver.from_scene(sc, precision)
    rng = np.random.default_rng(5)
    n = 30
    t = lambda a, dt=torch.float64: torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device=dev)  # noqa: E731
    X, D = rng.uniform(-1.8, 1.8, (n, dim)), rng.normal(size=(n, dim))
    D /= np.linalg.norm(D, axis=1, keepdims=True)
    on, nin = t(-np.ones(n), torch.int32), t(np.zeros((n, dim)))

    def ask(cap):
        return s.reflect_query(t(X), t(D), t(cap), on, nin).cpu().numpy()

    cap = np.tile([1.5, np.nan, -1.0, -0.25, 0.0, np.inf], n // 6)
    got, plain = ask(cap), ask(np.where(np.isfinite(cap), np.abs(cap), 1e6))
    nan, neg, zero, rest = np.isnan(cap), cap < 0, cap == 0, (cap > 0)
    assert np.isnan(got[nan, :2]).all() and (got[nan, 2] == -1).all()
    assert np.array_equal(got[neg, 0], plain[neg, 0])
    assert np.array_equal(got[neg, 1], cap[neg]) and (got[neg, 2] == -1).all()
    assert np.array_equal(got[zero], np.array([[0.0, 0.0, -1.0]] * zero.sum()))
    hit = rest & (plain[:, 2] >= 0)
    assert hit.any() and np.array_equal(got[hit, 1:], plain[hit, 1:])
    assert np.array_equal(got[rest, 2], plain[rest, 2])
    near = rest & (plain[:, 0] < 1e5)
    assert near.any() and np.array_equal(got[near, 0], plain[near, 0])
