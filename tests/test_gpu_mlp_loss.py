"""The loss of a batch against its 64-bit value.

With zero weights the network's output is its output bias, so the FP32 residuals are known
exactly.  Their squares and sums are formed in FP64 (error at most n 2^-53) and rounded once:
2^-24 of the loss."""
import numpy as np
import pytest

from gpu_util import dev
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
