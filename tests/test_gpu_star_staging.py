"""Walk on stars in 2D with Dirichlet boundaries on both sides of what a block
keeps in LDS (the whole tree, its nodes without the primitives, the first
nodes): the walks are the same, bit for bit, however much of it is staged."""
import pytest

import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_wire", [4, 125, 200, 320, 1000])
def test_same_walks_however_much_is_staged(n_wire):
    from paper_2405_12964_amd import Solver
    sc = scenes.thermal_scene(n_slice=2000, n_wire=n_wire, K=2)
    X, seg = scenes.points_on_segments(sc.NV, sc.nsegs, 200, 3)
    X = torch.as_tensor(X, dtype=torch.float64, device="cuda").contiguous()
    s = Solver.from_scene(sc, "fp32")
    s.set_start_segments(seg)
    for mode in (0, 1):
        full = s.walk_records(X, 8, 11, mode)
        for cap in (0, 1, 30):
            s.set_tuning(stage_nodes=cap)
            got = s.walk_records(X, 8, 11, mode)
            for key in ("u", "steps", "prim", "uoff"):
                assert torch.equal(got[key], full[key]), (mode, cap, key)
        s.set_tuning(stage_nodes=-1)
