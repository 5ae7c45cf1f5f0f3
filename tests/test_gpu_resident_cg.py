"""The Laplacian solve as one resident launch, and beyond what the device holds.

Rows per thread block are 512 and partial sums run over 256 rows, so the
meshes have sizes on both sides of these; vertices of more neighbours than
the kernel's registers hold (2 in 2D, 8 in 3D) and isolated vertices are
among them, and the longest 2D chain is solved by the kernels that take one
launch per part of an iteration.  Against scipy's sparse direct solve: with
tol 1e-14 the residual in the M^-1-like norm falls by that factor, and the
condition number of M is at most 1 + 2 lambda deg < 1e4, hence 1e-9.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def ring(n):
    return n, np.stack([np.arange(n), (np.arange(n) + 1) % n], 1)


def star2(n):                       # one vertex joined to every other, one vertex alone
    return n + 1, np.stack([np.zeros(n - 1, int), np.arange(1, n)], 1)


def fan3(n):                        # a cone over a ring: the apex has n - 1 neighbours
    i = np.arange(1, n)
    return n, np.stack([np.zeros(n - 1, int), i, i % (n - 1) + 1], 1)


def grid3(n):                       # a triangulated square, n x n vertices
    a = (np.arange(n - 1)[:, None] * n + np.arange(n - 1)).ravel()
    return n * n, np.concatenate([np.stack([a, a + 1, a + n], 1), np.stack([a + 1, a + n + 1, a + n], 1)])


MESHES = [(2, ring(3)), (2, ring(256)), (2, ring(257)), (2, ring(513)), (2, star2(600)), (2, ring(300000)),
          (3, fan3(4)), (3, fan3(9)), (3, fan3(10)), (3, fan3(700)), (3, grid3(16)), (3, grid3(33))]


@pytest.mark.parametrize("dim,mesh", MESHES, ids=[f"{d}d-{m[0]}" for d, m in MESHES])
def test_solve_matches_direct(dev, dim, mesh):
    import paper_2405_12964_amd as dwos
    from oracle import largesteps as ls
    from scipy.sparse import linalg as spla
    nv, F = mesh
    F = F.astype(np.int32)
    lam = 5.0
    b = np.random.default_rng(nv).normal(size=(nv, dim))
    M = ls.system_matrix(nv, F, lam).tocsc()
    lu = spla.splu(M)
    ref = np.stack([lu.solve(b[:, c]) for c in range(dim)], 1)
    o = dwos.LargeSteps(dim, nv, F, lam)
    x = torch.zeros(nv, dim, dtype=torch.float64, device=dev)
    tb = torch.tensor(b, dtype=torch.float64, device=dev)
    it = o.solve(tb, x, max_iters=2000, tol=1e-14)
    err = np.abs(x.cpu().numpy() - ref).max() / np.abs(ref).max()
    assert err < 1e-9, (err, it)
    assert it % 16 == 0 and 0 < it < 2000
    # a solve that stops early stops where asked, and a second one goes on from there
    y = torch.zeros_like(x)
    assert o.solve(tb, y, max_iters=1, tol=1e-14) == 1
    assert o.solve(tb, y, max_iters=0, tol=1e-14) == 0
    o.solve(tb, y, max_iters=2000, tol=1e-14)
    assert np.abs(y.cpu().numpy() - ref).max() / np.abs(ref).max() < 1e-9
