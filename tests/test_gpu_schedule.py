"""A walk is a function of (seed, point, walk) alone: launches that spread few
walks over many wavefronts give the walks of launches that fill them."""
import numpy as np
import pytest
import torch

import scenes
from paper_2405_12964_amd import Solver

pytestmark = pytest.mark.gpu


def _case(kind):
    """(scene, points, start primitives or None) of more walks than the chip holds at once."""
    if kind == "wos2d":
        sc = scenes.c2_star(n=301, K=2)
        return sc, scenes.star_points(6000, 3), None
    if kind == "wos3d":
        sc = scenes.c3_icosphere(nu=6, n_basis=64, h=0.4, K=2)
        return sc, scenes.points_on_box_faces(6000, 3), None
    if kind == "wost2d":
        sc = scenes.thermal_scene(n_slice=600, K=2)
        X, seg = scenes.points_on_segments(sc.NV, sc.nsegs, 3000, 3)
        return sc, X, seg
    if kind == "wost3d":
        sc = scenes.thermal3d_scene(nu_slice=6, nu_wire=2, K=2)
        X, tri = scenes.points_on_triangles(sc.NV, sc.nsegs, 600, 3)
        return sc, X, tri
    sc = scenes.inflation_scene(n=9, seed=1).with_(K=2)
    return sc, 0.02 * np.random.default_rng(0).normal(size=(3000, 2)) + sc.mono[0, 1:], None


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("kind", ["wos2d", "wos3d", "wost2d", "wost3d", "implicit"])
def test_walks_do_not_depend_on_the_split(kind, precision):
    sc, X, start = _case(kind)
    s = Solver.from_scene(sc, precision)
    X = torch.as_tensor(X, dtype=torch.float64, device="cuda").contiguous()
    W = 48

    def records(n, W, mode):
        if start is not None:
            s.set_start_segments(start[:n])
        return s.walk_records(X[:n].contiguous(), W, 11, mode)

    for mode in (0, 1):
        full = records(X.shape[0], W, mode)
        # one walk; a wavefront's lanes and one more or less; a share of the
        # chip's lanes; the rest in between
        for n, w in ((1, 1), (1, 15), (1, 16), (1, 17), (3, 21), (4, 16), (5, 13), (97, 48), (599, 48)):
            got = records(n, w, mode)
            for key in ("u", "steps", "prim", "uoff"):
                a, b = got[key], full[key][:n, :w]
                assert torch.equal(a, b), (kind, precision, mode, n, w, key, int((a != b).sum()))
