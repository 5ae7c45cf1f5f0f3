"""The network kernels at the edges of their tiling, against the FP64 oracle.

Evaluation with derivatives and the adjoint gradient take 16 points at a time,
the value alone and the loss gradient 64, in persistent launches whose blocks
take a second round from 512 (evaluation) and 256 (gradients) groups on; the
sizes lie on both sides of these.

Tolerance: the split products drop what lies 2^-17 below each operand; through
four layers forward and back that is at most 16 such terms of random sign per
result, 1.2e-4 of the results' norm.
"""
import numpy as np
import pytest

import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIZES = [1, 15, 16, 17, 63, 64, 65, 4097, 8193, 16385, 32769]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def rel(a, b):
    return np.linalg.norm(a.cpu().numpy().astype(np.float64) - b) / np.linalg.norm(b)


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("dim", [2, 3])
def test_network_sizes(dev, oracle_mod, dim, n):
    import paper_2405_12964_amd as dwos
    B, th = (a.astype(np.float32).astype(np.float64) for a in scenes.mlp_init(dim, 7 * dim, 1.0))
    rng = np.random.default_rng(n)
    f32 = lambda *s: rng.normal(size=s).astype(np.float32)  # noqa: E731
    X, t, nb, lb = rng.uniform(-1.5, 1.5, (n, dim)).astype(np.float32), f32(n), f32(n), 0.05 * f32(n)
    w = rng.uniform(0.5, 1.5, n).astype(np.float32)
    d = lambda a: torch.tensor(a, device=dev)  # noqa: E731
    net, ref = dwos.Network(dim, B, th), oracle_mod.Net(dim, B, th)
    X64, t64, w64, nb64, lb64 = (a.astype(np.float64) for a in (X, t, w, nb, lb))
    No, Go, Lo = ref.eval(X64)
    for got, want in zip(net.eval(d(X), derivatives=True), (No, Go, Lo)):
        assert rel(got, want) < 1.2e-4
    assert rel(net.eval(d(X)), No) < 1.2e-4
    g = net.vjp(d(X), d(nb), d(lb))
    assert rel(g, ref.vjp(X64, nb64, lb64)) < 1.2e-4
    assert torch.equal(g, net.vjp(d(X), d(nb), d(lb)))     # one order of addition
    loss, g = net.loss_grad(d(X), d(t), d(w))
    loss_o, go = ref.loss_grad(X64, t64, w64)
    assert rel(g, go) < 1.2e-4 and abs(loss.item() - loss_o) <= 1.2e-4 * abs(loss_o)
