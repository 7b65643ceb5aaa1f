"""The ladder where its unpack goes from four to sixteen columns per workgroup: one block pair
with 93 and 97 groups of sixteen columns (FP64) and with 156 and 160 (FP32 and split bf16), and
several block pairs of few and of many groups.

Tolerances: FP64 1e-11 of the largest value (at most 2e3 terms of random sign, summation order);
the others element by element within 2e-4 of the ladder of the absolute values (two rounding
stages of 3 * 2^-18 a product, FP32 accumulation)."""
import numpy as np
import pytest

from gpu_util import dev, host, rel_max
from oracle import native
from paper_1810_08142_amd.synthetic import draw_pair_symmetric, draw_system

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("o,v,naux", [(54, 16, 5), (55, 16, 5), (70, 16, 5), (71, 15, 5), (1, 130, 5), (9, 70, 5),
                                      (20, 33, 5)])
def test_ladder_across_unpack_forms(o, v, naux, precision):
    import torch
    from paper_1810_08142_amd import ppl
    s = draw_system(o, v, naux, seed=850 + v)
    tau = draw_pair_symmetric(o, v, 851 + o)
    R = torch.zeros((o, o, v, v), dtype=torch.float64, device="cuda")
    ppl.ppl(dev(s.B_vv), dev(tau), R, precision=precision)
    got, ref = host(R), native.ppl(s.B_vv, tau)
    if precision == "fp64":
        assert rel_max(got, ref) <= 1e-11
    else:
        assert np.all(np.abs(got - ref) <= 2e-4 * native.ppl(np.abs(s.B_vv), np.abs(tau)))
    assert np.array_equal(got, got.transpose(1, 0, 3, 2))
