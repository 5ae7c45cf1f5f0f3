"""What a block of the 2D walk kernel keeps in LDS, as scene_info reports it: the
tree or its first nodes, the traversal stacks and the statistics."""
import pytest

import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LDS = 160 * 1024
ENTRY = 1024 * 8          # one stack entry of every lane of a block


@pytest.mark.parametrize("n", [128, 3000, 4096, 9000])
def test_reported_bytes(n):
    from paper_2405_12964_amd import Solver
    s = Solver.from_scene(scenes.c2_star(n=n, K=2), "fp32")
    i = s.scene_info()
    tree = i["staged_nodes"] * (i["node_bytes"] // i["nodes"]) + i["staged_prims"] * i["prim_bytes"]
    entries, rest = divmod(i["lds_bytes"] - tree, ENTRY)
    assert 5 <= entries <= 15 and 0 < rest <= 512 and i["lds_bytes"] <= LDS
