"""The one-launch Laplacian solve at the sizes where its blocks are many, and
when they miss each other.

* Against the launches per part of an iteration, bit for bit, with as many
  iterations: on both sides of 65,536 rows (a thread then collects a second
  partial sum), at some 100,000 rows, and on both sides of what the device holds.
  The residual of both, in the norm that stops them, is at most twice the 1e-10
  asked for (the recurrence drifts by less than its own size in FP64).
* Given up: a wait of one tick expires at once in every block, which all end
  normally; the launches that follow reach the residual asked for, relative to the
  start of the solve and within its iterations, and so does the next solve.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LAM = 20.0


def ring(n):
    return 2, n, np.stack([np.arange(n), (np.arange(n) + 1) % n], 1)


def grid3(n, m):                       # a triangulated rectangle of n x m vertices
    a = (np.arange(n - 1)[:, None] * m + np.arange(m - 1)).ravel()
    return 3, n * m, np.concatenate([np.stack([a, a + 1, a + m], 1), np.stack([a + 1, a + m + 1, a + m], 1)])


def problem(mesh):
    import paper_2405_12964_amd as dwos
    from oracle import largesteps as ls
    dim, nv, F = mesh
    F = F.astype(np.int32)
    b = np.random.default_rng(nv).normal(size=(nv, dim))
    M = ls.system_matrix(nv, F, LAM).tocsr()
    return dwos.LargeSteps(dim, nv, F, LAM), torch.tensor(b, device="cuda"), M, b


def residual(M, b, x):
    r = b - M @ x.cpu().numpy()
    d = M.diagonal()[:, None]
    return np.sqrt((r * r / d).sum() / (b * b / d).sum())


@pytest.mark.parametrize("mesh", [grid3(256, 256), grid3(3, 21846), grid3(316, 317), grid3(2, 65536), grid3(3, 43691),
                                  ring(65537), ring(262144), ring(262145)],
                         ids=lambda m: f"{m[0]}d-{m[1]}")
def test_same_as_a_launch_per_part(mesh):
    o, b, M, bh = problem(mesh)
    got = []
    for wait in (10.0, 0.0):
        o.set_wait(wait)
        x = torch.zeros_like(b)
        it = o.solve(b, x, max_iters=4000, tol=1e-10)
        assert 0 < it < 4000
        y = torch.zeros_like(b)
        o.solve(b, y, max_iters=5, tol=1e-10)           # an early end
        got.append((it, x, y))
    assert got[0][0] == got[1][0]
    assert torch.equal(got[0][1], got[1][1]) and torch.equal(got[0][2], got[1][2])
    assert residual(M, bh, got[0][1]) <= 2e-10


@pytest.mark.parametrize("mesh", [ring(300), grid3(20, 20), grid3(316, 317)], ids=lambda m: f"{m[0]}d-{m[1]}")
def test_blocks_that_miss_each_other(mesh):
    o, b, M, bh = problem(mesh)
    x = torch.zeros_like(b)
    o.solve(b, x, max_iters=4000, tol=1e-6)             # a start with a residual of its own
    y = x.clone()
    o.set_wait(1e-8)
    it = o.solve(b, x, max_iters=4000, tol=1e-4)
    start = residual(M, bh, y)
    assert 0 < it < 4000 and residual(M, bh, x) <= 2e-4 * start
    # few iterations are few
    z = torch.zeros_like(b)
    assert o.solve(b, z, max_iters=3, tol=1e-12) <= 3
    # the resident solve again
    o.set_wait(10.0)
    one = torch.zeros_like(b)
    it1 = o.solve(b, one, max_iters=4000, tol=1e-10)
    o.set_wait(0.0)
    parts = torch.zeros_like(b)
    assert o.solve(b, parts, max_iters=4000, tol=1e-10) == it1 and torch.equal(one, parts)


def test_wait_arguments():
    from paper_2405_12964_amd.capi import DwosError, DWOS_EINVAL
    o = problem(ring(8))[0]
    for bad in (-1.0, float("nan"), float("inf"), 3601.0):
        with pytest.raises(DwosError) as e:
            o.set_wait(bad)
        assert e.value.code == DWOS_EINVAL
