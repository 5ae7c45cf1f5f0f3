"""What a block of the 2D walk kernel keeps in LDS: the whole tree as long as
two stack entries a lane fit beside it, else its first nodes beside five.  The
plan is reported as the launch uses it, and the walks do not depend on it."""
import pytest

import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LDS = 160 * 1024
ENTRY = 1024 * 8          # one stack entry of every lane of a block


@pytest.mark.parametrize("n", [128, 3000, 4096, 4300, 4600, 4800, 5400, 9000])
def test_plan_and_walks(n):
    from paper_2405_12964_amd import Solver
    s = Solver.from_scene(scenes.c2_star(n=n, K=2), "fp32")
    i = s.scene_info()
    whole = i["node_bytes"] + i["prim_bytes"]
    fits = whole + 2 * ENTRY + 512 <= LDS
    assert fits == (n <= 4600)
    assert (i["staged_prims"] == 1 and i["staged_nodes"] == i["nodes"]) == fits
    tree = whole if fits else i["staged_nodes"] * (i["node_bytes"] // i["nodes"])
    entries, rest = divmod(i["lds_bytes"] - tree, ENTRY)
    assert (2 if fits else 5) <= entries <= 15 and 0 < rest <= 512 and i["lds_bytes"] <= LDS
    X = torch.as_tensor(scenes.star_points(700, 3), dtype=torch.float64, device="cuda").contiguous()
    for mode in (0, 1):
        a = s.walk_records(X, 48, 11, mode)
        s.set_variant(1)
        b = s.walk_records(X, 48, 11, mode)
        s.set_variant(0)
        for key in ("u", "steps", "prim", "uoff"):
            assert torch.equal(a[key], b[key]), (mode, key)
