"""Lanes that share a walk change nothing: launches of few walks (four lanes per
walk), of some more (two) and of enough to fill the chip (one) give the same
records, bit for bit, in every mode of the walk kernel and with the tree in LDS,
partly in LDS and in global memory."""
import pytest
import torch

import scenes
from paper_2405_12964_amd import Solver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,size,variant", [(2, 3, 0), (2, 301, 0), (2, 301, 1), (2, 5000, 0), (3, 1, 0), (3, 6, 1),
                                              (3, 30, 0)])
@pytest.mark.parametrize("dudn", [0, 1])
def test_groups_of_lanes(dim, size, variant, dudn):
    if dim == 2:
        sc, X = scenes.c2_star(n=size, K=2), scenes.star_points(7000, 3) * 0.3
    else:
        sc, X = scenes.c3_icosphere(nu=size, n_basis=64, h=0.4, K=2), scenes.points_on_box_faces(7000, 3)
    if dudn:
        sc = sc.with_(dudn=1, sigma=0.0, src_c0=0.0, gauss=None)
    s = Solver.from_scene(sc, "fp32")
    s.set_variant(variant)
    X = torch.as_tensor(X, dtype=torch.float64, device="cuda").contiguous()
    for mode in (0, 1):
        full = s.walk_records(X, 48, 5, mode)              # 336,000 walks
        for n, w in ((2, 1), (3, 7), (700, 48), (1650, 48), (2100, 48)):
            got = s.walk_records(X[:n].contiguous(), w, 5, mode)
            for key in ("u", "steps", "prim", "uoff"):
                a, b = got[key], full[key][:n, :w]
                assert torch.equal(a.nan_to_num(nan=-7), b.nan_to_num(nan=-7)), (mode, n, w, key, int((a != b).sum()))
