"""Closest points by a wavefront per point, and the refit of large nodes.

A list of up to 16,384 (2D) or 65,536 (3D) points is answered by a wavefront
per point, a longer one by a lane per point.  In FP32 the answer is the lowest
original index at the least distance in any order of the visits, so that both
agree exactly, also at points equally far from many primitives (the centre of
a sphere or a polygon, where every node is visited and the traversal stack is
at its longest) and at points that are not finite.

Refitting cuts nodes of more than 1,024 primitives into parts: after an update
of the vertices, the answers are those of a boundary set to them.
"""
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


def polygon(n):
    t = 2 * np.pi * np.arange(n) / n
    return np.stack([np.cos(t), np.sin(t)], 1), np.stack([np.arange(n), (np.arange(n) + 1) % n], 1).astype(np.int32)


def solver(dim, V, prims, precision="fp32"):
    import paper_2405_12964_amd as dwos
    s = dwos.Solver(dim, precision=precision)
    s.set_boundary(V, prims)
    return s


@pytest.mark.parametrize("dim,size,count", [(2, 3, 16385), (2, 9, 16385), (2, 3000, 16385), (3, 1, 65537),
                                            (3, 40, 65537)])
def test_wavefront_and_lane_agree(dev, dim, size, count):
    V, prims = polygon(size) if dim == 2 else scenes.icosphere(size)
    s = solver(dim, V, prims)
    rng = np.random.default_rng(size)
    X = rng.uniform(-1.2, 1.2, (count, dim))
    X[:64] = 0.0
    X[64:128] *= 1e-6
    X[128:192] = V[rng.integers(0, len(V), 64)]
    X[192:194] = np.nan
    X[194:196] = np.inf
    X[196:198, 0] = -np.inf
    X[198:200] *= 1e30
    X = torch.tensor(X, device=dev)
    lane = s.closest(X)
    wave = torch.cat([s.closest(X[:1]), s.closest(X[1:6]), s.closest(X[6:])])
    assert torch.equal(lane.nan_to_num(nan=-7.0), wave.nan_to_num(nan=-7.0))


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("dim,size", [(2, 1024), (2, 1025), (2, 5000), (3, 7), (3, 8), (3, 30)])
def test_refit_answers_as_a_new_boundary(dev, dim, size, precision):
    V, prims = polygon(size) if dim == 2 else scenes.icosphere(size)
    s = solver(dim, V, prims, precision)
    V2 = V * (1.0 + 0.3 * np.sin(3.0 * V[:, :1])) + 0.1
    s.update_vertices(torch.tensor(V2, device=dev))
    X = torch.tensor(np.random.default_rng(1).uniform(-1.2, 1.2, (3000, dim)), device=dev)
    assert torch.equal(s.closest(X), solver(dim, V2, prims, precision).closest(X))
