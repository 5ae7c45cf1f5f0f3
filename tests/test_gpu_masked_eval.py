"""The control variate's network on the walks that run nested walks: a walk's
values do not depend on how many others there are or where they lie, so that the
records of a large call's first points are those of a small one, bit for bit, on
both sides of the points that a block looks through at a time."""
import numpy as np
import pytest

import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,q", [(2, 1.0), (3, 1.0), (3, 0.25)])
def test_records_do_not_depend_on_the_call(dim, q):
    from paper_2405_12964_amd import Network, Solver
    if dim == 2:
        sc, pts = scenes.c2_star(200, K=2, sigma=4.0), scenes.star_points(40000, 3)
    else:
        sc, pts = scenes.c3_icosphere(nu=8, n_basis=64, h=0.4, K=2), scenes.points_on_box_faces(40000, 3)
    B, th = scenes.mlp_init(dim, 31, 1.0)
    X = torch.as_tensor(pts, dtype=torch.float64, device="cuda").contiguous()
    W = 16

    def records(n):
        s = Solver.from_scene(sc, "fp32")
        net = Network(dim, B, th)
        s.attach_cv(net, q)
        return s.cv_walk_records(X[:n].contiguous(), W, 7)

    full = records(len(X))
    ran = 0
    for n in (1, 15, 17, 700, 8000):
        part = records(n)
        for key, b in part.items():
            a = full[key][:b.shape[0]] if full[key].shape[0] != b.shape[0] else full[key]
            assert torch.equal(a.nan_to_num(nan=-7.0), b.nan_to_num(nan=-7.0)), (n, key)
        ran = part
    assert len(ran) > 3
