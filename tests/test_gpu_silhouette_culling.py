"""Silhouette queries from points just outside the bounding circles (2D) and
spheres (3D) of runs of the reflecting boundary, where the cones' margins are
tightest: the angle under which such a circle is seen is next to a right one.

FP32 answers against every vertex (edge) in FP64: at most the distance of the
nearest one that is clearly a silhouette (both sides 1e-2 from edge-on, the
test's own tolerance being 1e-4), at least that of the nearest one that may be
(within 1e-3 of edge-on), both to 1e-5 of the coordinates' size (16 units of
FP32 rounding, squared distances included).
"""
import numpy as np
import pytest

import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHELLS = np.array([0.0, 1e-7, 3e-7, 1e-6, 1e-5, 1e-4, 1e-3, 1e-2, 0.1])
TOL = 1e-5 * 2.0


def _around(P, sets, rng):
    """Points just outside the bounding circle of each set's box."""
    out = []
    for s in sets:
        lo, hi = P[s].min(0), P[s].max(0)
        n = rng.normal(size=(len(SHELLS), P.shape[1]))
        n /= np.linalg.norm(n, axis=1, keepdims=True)
        out.append(0.5 * (lo + hi) + n * (0.5 * np.linalg.norm(hi - lo) * (1 + SHELLS))[:, None])
    return np.concatenate(out).astype(np.float32).astype(np.float64)


def _query(sc, X):
    from paper_2405_12964_amd import Solver
    s = Solver.from_scene(sc, "fp32")
    t = lambda a, dt=torch.float64: torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device="cuda")  # noqa: E731
    n, zero = len(X), np.zeros_like(X)
    cap = np.full(n, 10.0)
    return s.reflect_query(t(X), t(zero + np.eye(X.shape[1])[0]), t(cap), t(-np.ones(n), torch.int32),
                           t(zero)).cpu().numpy()[:, 0]


def _check(got, d, clear, maybe):
    lo = np.where(maybe, d, 10.0).min(1)
    hi = np.where(clear, d, 10.0).min(1)
    assert (hi < 10.0).mean() > 0.5
    assert (got <= hi + TOL).all(), (got - hi).max()
    assert (got >= lo - TOL).all(), (lo - got).max()


@pytest.mark.parametrize("n", [40, 700])
def test_culling_2d(n):
    sc = scenes.thermal_scene(n_slice=n, n_wire=8, K=1)
    V = np.asarray(sc.NV, np.float32).astype(np.float64)
    rng = np.random.default_rng(n)
    runs = [(rng.integers(0, n) + np.arange(rng.choice([2, 3, 5, 9, 17, 33]) + 1)) % n for _ in range(300)]
    X = _around(V, runs, rng)
    got = _query(sc, X)
    nxt, prv = np.roll(V, -1, 0), np.roll(V, 1, 0)
    v = V[None] - X[:, None]
    d = np.linalg.norm(v, axis=2)
    def side(far):
        w = far - V
        return (v[..., 0] * w[:, 1] - v[..., 1] * w[:, 0]) / np.maximum(d * np.linalg.norm(w, axis=1), 1e-300)
    a, b = side(nxt), side(prv)
    clear = ((a > 1e-2) & (b > 1e-2)) | ((a < -1e-2) & (b < -1e-2))
    maybe = ((a > -1e-3) & (b > -1e-3)) | ((a < 1e-3) & (b < 1e-3))
    _check(got, d, clear, maybe)


@pytest.mark.parametrize("nu", [2, 6])
def test_culling_3d(nu):
    sc = scenes.thermal3d_scene(nu_slice=nu, nu_wire=1, K=1)
    V, F = np.asarray(sc.NV, np.float32).astype(np.float64), np.asarray(sc.nsegs)
    rng = np.random.default_rng(nu)
    near = [np.argsort(np.linalg.norm(V - V[rng.integers(0, len(V))], axis=1))[:rng.choice([3, 5, 9, 17])]
            for _ in range(200)]
    X = _around(V, near, rng)
    got = _query(sc, X)
    edges = {}
    for f, tri in enumerate(F):
        for k in range(3):
            edges.setdefault(tuple(sorted((tri[k], tri[(k + 1) % 3]))), []).append(f)
    e = np.array(list(edges))
    fs = np.array(list(edges.values()))
    assert fs.shape[1] == 2
    A, B = V[e[:, 0]], V[e[:, 1]]
    t = np.clip(((X[:, None] - A) * (B - A)).sum(-1) / ((B - A) ** 2).sum(-1), 0, 1)
    foot = A + t[..., None] * (B - A)
    d = np.linalg.norm(X[:, None] - foot, axis=2)
    third = np.array([[[v for v in F[f] if v not in pq][0] for f in ff] for pq, ff in zip(e, fs)])
    rr = X[:, None] - A
    m = np.cross((B - A)[None], rr)                       # normal of the plane through x and the edge
    lm = np.linalg.norm(m, axis=2)
    def side(k):
        w = V[third[:, k]] - A
        return (m * w).sum(-1) / np.maximum(lm * np.linalg.norm(w, axis=1), 1e-300)
    a, b = side(0), side(1)
    # x on the edge's line: the plane is rounding alone
    line = lm < 1e-3 * np.linalg.norm(B - A, axis=1) * np.linalg.norm(rr, axis=2)
    clear = (((a > 1e-2) & (b > 1e-2)) | ((a < -1e-2) & (b < -1e-2))) & ~line
    maybe = ((a > -1e-3) & (b > -1e-3)) | ((a < 1e-3) & (b < 1e-3)) | line
    _check(got, d, clear, maybe)
