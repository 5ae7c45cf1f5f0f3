"""Forward mode over more points than one launch has blocks (2^24 points took
more threads than a launch holds).  Walks of one step: a point's derivative then
depends on its position alone, so that repeated points repeat their results."""
import numpy as np
import pytest

import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,W", [((1 << 22) + 3, 2), ((1 << 24) + 5, 1)])
def test_more_points_than_blocks(P, W):
    from paper_2405_12964_amd import Solver
    n, period = 24, 1009
    s = Solver.from_scene(scenes.c2_star(n=n, K=1).with_(eps=1e3, delta=1e2), "fp32")
    s.set_parameters(1, np.arange(n + 1), np.zeros(n, np.int32), np.random.default_rng(1).normal(size=(n, 2)))
    X = torch.as_tensor(scenes.star_points(period, 3), dtype=torch.float64, device="cuda").contiguous()
    few = s.jvp(X, W, 3)[0]
    many = s.jvp(X.repeat(P // period + 1, 1)[:P].contiguous(), W, 3)[0]
    assert few.abs().max() > 0
    assert torch.equal(many.reshape(-1), few.reshape(-1).repeat(P // period + 1)[:P])
