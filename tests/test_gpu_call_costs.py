"""Costs of calls that a launch's shape can spoil: short walks, few walks a
point, boundaries just past what fits a block's LDS.  Best of several calls,
against bounds between what the call takes and what it took with the fault that
each test names.
"""
import numpy as np
import pytest

import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def best_us(call, repeats=12):
    """Least device time of a call, us (the first two are not counted)."""
    out = []
    for k in range(repeats):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        call()
        b.record()
        torch.cuda.synchronize()
        if k > 1:
            out.append(a.elapsed_time(b) * 1e3)
    return min(out)


def test_star_blocks_per_cu():
    """Walk on stars keeps four blocks per CU whatever the Dirichlet boundary:
    1,004 segments take what 1,284 take (1.34 times as long when their tree
    and primitives were staged at two blocks per CU)."""
    from paper_2405_12964_amd import Solver
    t = []
    for n_wire in (250, 320):
        sc = scenes.thermal_scene(n_slice=8192, n_wire=n_wire, K=1)
        X, seg = scenes.points_on_segments(sc.NV, sc.nsegs, 4096, 3)
        X = torch.as_tensor(X, dtype=torch.float64, device="cuda").contiguous()
        s = Solver.from_scene(sc, "fp32")
        s.set_start_segments(seg)
        t.append(best_us(lambda: s.solve(X, 16, 3, var=False), 5))
    assert t[0] < 1.17 * t[1], t


def test_short_walks():
    """65,536 walks of one step: the statistics are a few atomics a block, 31 us in
    all (529 us with a dozen a wavefront, of which small launches have four times
    as many as launches of full wavefronts)."""
    from paper_2405_12964_amd import Solver
    s = Solver.from_scene(scenes.c3_icosphere(nu=20, n_basis=64, h=0.4).with_(eps=1e3, delta=1e2), "fp32")
    X = torch.as_tensor(scenes.points_on_box_faces(65536, 3), device="cuda").contiguous()
    ms = []
    for _ in range(12):
        s.walk_timing(0, reset=True)
        s.solve(X, 1, 3, var=False)
        ms.append(s.walk_timing(0)[0])
    assert min(ms) < 0.27, ms


@pytest.mark.parametrize("kind", ["wos2d", "wos3d", "wost2d", "wost3d", "implicit"])
def test_statistics_add_up(kind):
    """The blocks' statistics lose and double nothing: walks, and the steps of
    the records, at block counts from one to more than the chip holds."""
    from paper_2405_12964_amd import Solver
    start = None
    if kind == "wos2d":
        sc, X = scenes.c2_star(n=301, K=1), scenes.star_points(20000, 3)
    elif kind == "wos3d":
        sc, X = scenes.c3_icosphere(nu=6, n_basis=64, h=0.4, K=1), scenes.points_on_box_faces(20000, 3)
    elif kind == "wost2d":
        sc = scenes.thermal_scene(n_slice=600, K=1)
        X, start = scenes.points_on_segments(sc.NV, sc.nsegs, 9000, 3)
    elif kind == "wost3d":
        sc = scenes.thermal3d_scene(nu_slice=6, nu_wire=2, K=1).with_(kmax=40)
        X, start = scenes.points_on_triangles(sc.NV, sc.nsegs, 9000, 3)
    else:
        sc = scenes.inflation_scene(n=9, seed=1)
        X = 0.02 * np.random.default_rng(0).normal(size=(20000, 2)) + sc.mono[0, 1:]
    s = Solver.from_scene(sc, "fp32")
    X = torch.as_tensor(X, dtype=torch.float64, device="cuda").contiguous()
    for P, W in ((1, 1), (1, 17), (3, 100), (300, 33), (len(X), 40)):
        if start is not None:
            s.set_start_segments(start[:P])
        Xp = X[:P].contiguous()
        s.walk_timing(0, reset=True)
        st = s.solve(Xp, W, 7, stats=True)[-1]
        steps = s.walk_records(Xp, W, 7, 0)["steps"]
        shared = 0 if kind == "implicit" else P * (W - 1)   # a point's first query counts once
        assert st["walks"] == P * W and st["steps"] == int(steps.sum()) - shared, (P, W)
        assert (st["nodes"] > 0) == (kind != "implicit")
        total = s.walk_timing(0)[-1]
        assert total["walks"] == 2 * P * W and total["steps"] == 2 * st["steps"]


def test_repeated_first_queries():
    """65,536 one-step walks again from the same points around 200,000 triangles:
    109 us, the first queries 17 of them (83 by a wavefront per point, 678 in all
    with the statistics by wavefront)."""
    from paper_2405_12964_amd import Solver
    s = Solver.from_scene(scenes.c3_icosphere(nu=100, n_basis=64, h=0.4).with_(eps=1e3, delta=1e2), "fp32")
    X = torch.as_tensor(scenes.points_on_box_faces(65536, 3), device="cuda").contiguous()
    assert best_us(lambda: s.solve(X, 1, 3, var=False)) < 165


def test_queries_of_a_small_tree():
    """65,536 points and 32 triangles: a lane per point, 34 us (127 by a wavefront)."""
    from paper_2405_12964_amd import Solver
    V, prims = scenes.icosphere(1)
    s = Solver(3)
    s.set_boundary(V, prims)
    X = torch.as_tensor(np.random.default_rng(1).uniform(-1.9, 1.9, (65536, 3)), device="cuda")
    assert best_us(lambda: s.closest(X)) < 80


def test_forward_mode_of_few_walks():
    """65,536 points of one walk and one parameter: a wavefront per point, 173 us
    in all (with four, three of them without a walk, the reduction alone takes
    245 instead of 65)."""
    from paper_2405_12964_amd import Solver
    n = 128
    s = Solver.from_scene(scenes.c1_polygon(n).with_(eps=1e3, delta=1e2), "fp32")
    s.set_parameters(1, np.arange(n + 1), np.zeros(n, np.int32), np.ones((n, 2)))
    X = torch.as_tensor(scenes.points_in_disk(65536, 0.8, 1), device="cuda").contiguous()
    assert best_us(lambda: s.jvp(X, 1, 3)) < 260
