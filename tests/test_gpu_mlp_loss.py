"""The loss and the sums of the gradient against their 64-bit values.

With zero weights the network's output is its output bias, so the FP32 residuals are known
exactly.  Their squares and sums are formed in FP64 (error at most n 2^-53) and rounded once:
2^-24 of the loss."""
import numpy as np
import pytest

from gpu_util import dev, host
from paper_1810_08142_amd.synthetic import draw_matrix

pytestmark = pytest.mark.gpu


# one row, row remainders, several workgroups, several row tiles per workgroup (65536 rows)
@pytest.mark.parametrize("hidden,layers", [(64, 1), (256, 2)])
@pytest.mark.parametrize("n", [1, 17, 4096, 8199, 65536, 150001])
def test_loss_is_summed_in_fp64(hidden, layers, n):
    from paper_1810_08142_amd import mlp
    net = mlp.Net(8, hidden, layers)
    theta = np.zeros(mlp.init_params(8, hidden, layers, 1).size, dtype=np.float32)
    theta[-1] = 0.3
    net.set_params(theta)
    X = draw_matrix((n, 8), 31).astype(np.float32)
    for Y in (draw_matrix(n, 32).astype(np.float32), np.full(n, -0.123456, dtype=np.float32)):
        res = (theta[-1] - Y).astype(np.float64)
        ref = np.mean(res * res)
        loss, _ = net.gradient(dev(X), dev(Y))
        assert abs(loss - ref) <= (2.0**-24 + 1e-10) * ref


def test_weight_gradient_sums_are_short_chains_in_deep_networks():
    """With zero weights and a bias that saturates tanh, the gradient of the last hidden
    layer's weights is the sum over the rows of known FP32 terms dy * w.  Added up m at a time,
    terms of random sign are off by 0.30 sqrt(m) 2^-24 of their root sum of squares (0.42 2^-24
    of the running sum per addition); m = 256 rows here, and 15% for the spread over 256
    columns and the sums of the chains.  Ten layers of 256 leave one range of rows per tile,
    of which a wave takes 2048."""
    from paper_1810_08142_amd import mlp
    d_in, h, layers, n = 8, 256, 10, 8192
    net = mlp.Net(d_in, h, layers)
    theta = np.zeros(mlp.init_params(d_in, h, layers, 1).size, dtype=np.float32)
    last = d_in * h + h + (layers - 2) * (h * h + h)  # the last hidden layer's weights
    w = draw_matrix(h, 41).astype(np.float32)
    theta[last - h:last] = 20.0  # the layer before: tanh = 1
    theta[-h - 1:-1] = w
    net.set_params(theta)
    Y = draw_matrix(n, 42).astype(np.float32)
    _, g = net.gradient(dev(draw_matrix((n, d_in), 43).astype(np.float32)), dev(Y))
    dy = np.float32(2) * -Y / np.float32(n)
    terms = (dy[:, None] * w[None, :]).astype(np.float64)
    err = host(g)[last:last + h * h].reshape(h, h) - terms.sum(0)
    rel = err / np.sqrt((terms**2).sum(0))
    assert np.sqrt(np.mean(rel**2)) <= 1.15 * 0.30 * 256**0.5 * 2.0**-24
