"""Network kernels at the edges of their tiles, against forward and the FP64 oracle.

Tolerance of the gradient: every product sum has at most 256 FP32 terms (random-walk error
below 1e-6 of its value, worst case 256 * 2^-24 = 1.5e-5), and the sums over the batch add
terms of random sign whose errors and values grow alike, so 1e-4 of the largest value holds
for every batch size.
"""
import numpy as np
import pytest

from gpu_util import dev, host
from oracle import mlp as om
from paper_1810_08142_amd.synthetic import draw_matrix

pytestmark = pytest.mark.gpu


def _net(d_in, hidden, layers, seed=1):
    from paper_1810_08142_amd import mlp
    net = mlp.Net(d_in, hidden, layers)
    theta = mlp.init_params(d_in, hidden, layers, seed)
    theta += 0.05 * draw_matrix(theta.size, seed + 50).astype(theta.dtype)  # biases too
    net.set_params(theta)
    return net, theta.astype(np.float64)


@pytest.mark.parametrize("hidden", [64, 128, 192, 256])
@pytest.mark.parametrize("d_in,layers,n", [(4, 1, 1), (20, 2, 63), (64, 3, 65), (256, 1, 64), (16, 2, 129)])
def test_infer_in_registers_equals_forward(d_in, hidden, layers, n):
    """Row remainders, inputs of one and of several weight chunks, one to three layers."""
    net, _ = _net(d_in, hidden, layers, seed=hidden + layers)
    X = dev(draw_matrix((n, d_in), 17).astype(np.float32))
    assert np.array_equal(host(net.infer(X)), host(net.forward(X)))


# row tiles of 16 and 32 (from 8192 rows on), remainders of both, more row tiles than
# workgroups (65536 rows), ranges of the weight gradients with and without rows
CASES = ([(8, 256, 2, n) for n in (1, 15, 16, 17, 65, 8191, 8192, 8200, 65600)] +
         [(d, h, l, n) for d, h, l, n in ((1, 64, 1, 33), (17, 64, 3, 100), (64, 64, 2, 2049), (5, 128, 2, 8209),
                                          (128, 128, 1, 40), (33, 192, 3, 333), (3, 192, 2, 9001),
                                          (256, 256, 1, 129), (100, 256, 4, 70), (80, 16, 2, 50))])


@pytest.mark.parametrize("d_in,hidden,layers,n", CASES)
def test_gradient_matches_oracle_at_the_edges(d_in, hidden, layers, n):
    net, theta = _net(d_in, hidden, layers, seed=d_in + layers)
    X = draw_matrix((n, d_in), 5).astype(np.float32)
    Y = (0.5 * draw_matrix(n, 6)).astype(np.float32)
    Lr, gr = om.gradient(theta, X.astype(np.float64), Y.astype(np.float64), d_in, hidden, layers)
    first = None
    for _ in range(2):  # the same bits from used scratch
        loss, g = net.gradient(dev(X), dev(Y))
        g = host(g)
        assert abs(loss - Lr) <= 1e-4 * Lr
        assert np.abs(g - gr).max() <= 1e-4 * np.abs(gr).max()
        assert first is None or np.array_equal(first, g)
        first = g


def test_gradient_after_forward_and_at_odd_addresses():
    """A scratch first made for forward alone grows for the gradient; inputs that are only
    4-byte aligned are taken."""
    import torch
    d_in, hidden, layers, n = 7, 128, 3, 77
    net, theta = _net(d_in, hidden, layers, seed=3)
    X = draw_matrix((n, d_in), 8).astype(np.float32)
    Y = draw_matrix(n, 9).astype(np.float32)
    Xd = torch.empty(n * d_in + 1, dtype=torch.float32, device="cuda")[1:].view(n, d_in)
    Yd = torch.empty(n + 3, dtype=torch.float32, device="cuda")[3:]
    Xd.copy_(torch.from_numpy(X))
    Yd.copy_(torch.from_numpy(Y))
    net.forward(Xd)
    loss, g = net.gradient(Xd, Yd)
    Lr, gr = om.gradient(theta, X.astype(np.float64), Y.astype(np.float64), d_in, hidden, layers)
    assert abs(loss - Lr) <= 1e-4 * Lr
    assert np.abs(host(g) - gr).max() <= 1e-4 * np.abs(gr).max()
