"""Launches that fill every lane of the chip and refill them from the shared
counter, for every walk kernel: no walk is lost, doubled or changed.  The records
of P x W walks hold, for each point, those of launches with fewer walks a point,
which fit without a refill or leave lanes idle; the contexts' buffers held other
walks before, so that a walk that was not run shows."""
import pytest
import torch

import scenes
from paper_2405_12964_amd import Solver

pytestmark = pytest.mark.gpu


def _case(kind):
    """(scene, points, start primitives or None, walks a point): more than 64
    walks for every resident wavefront (at most 8,192 of them)."""
    if kind == "wos2d":
        return scenes.c2_star(n=301, K=1), scenes.star_points(14000, 3), None, 40
    if kind == "wos3d":
        return (scenes.c3_icosphere(nu=6, n_basis=64, h=0.4, K=1).with_(kmax=12), scenes.points_on_box_faces(14000, 3),
                None, 40)
    if kind == "wost2d":
        sc = scenes.thermal_scene(n_slice=600, K=1).with_(kmax=25)
        return sc, *scenes.points_on_segments(sc.NV, sc.nsegs, 14000, 3), 40
    if kind == "wost3d":
        sc = scenes.thermal3d_scene(nu_slice=6, nu_wire=2, K=1).with_(kmax=12)
        return sc, *scenes.points_on_triangles(sc.NV, sc.nsegs, 14000, 3), 40
    sc = scenes.inflation_scene(n=9, seed=1).with_(K=1)
    return sc, scenes.points_in_disk(14000, 0.02, 1) + sc.mono[0, 1:], None, 40


@pytest.mark.parametrize("kind", ["wos2d", "wos3d", "wost2d", "wost3d", "implicit"])
def test_full_launches(kind):
    sc, X, start, W = _case(kind)
    X = torch.as_tensor(X, dtype=torch.float64, device="cuda").contiguous()
    P = X.shape[0]
    full, few = Solver.from_scene(sc, "fp32"), Solver.from_scene(sc, "fp32")
    for s in (full, few):
        if start is not None:
            s.set_start_segments(start)
    st = full.solve(X, W, 5, stats=True)[-1]
    assert st["walks"] == P * W
    for mode in (0, 1):
        full.walk_records(X, W, 12, mode)
        a = full.walk_records(X, W, 11, mode)
        for w in (1, 9, 20):
            few.walk_records(X, w, 13, mode)
            b = few.walk_records(X, w, 11, mode)
            for key in ("u", "steps", "prim", "uoff"):
                assert torch.equal(a[key][:, :w].nan_to_num(nan=-7), b[key].nan_to_num(nan=-7)), (mode, w, key)
