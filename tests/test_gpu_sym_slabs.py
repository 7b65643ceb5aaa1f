"""The exchange-symmetric ladder at sizes whose later slabs, with fewer summed slots, would
be split further than the first (host check: test_slab_splits.py), default slabs.

Tolerances: FP64 differs from the oracle by summation order only, 1e-11 of the largest value
(at most 3e4 terms of random sign: 3e4^0.5 * 2^-53 = 2e-14 of a term's size, with room for
cancellation); the reduced precisions element by element within 2e-4 of the ladder of the
absolute values (two rounding stages of 3 * 2^-18 a product, FP32 accumulation), the ladder
here being the plain FP64 form, since the oracle takes minutes at these sizes."""
import numpy as np
import pytest

from gpu_util import dev, host, rel_max
from oracle import native
from paper_1810_08142_amd.synthetic import draw_pair_symmetric, draw_system

pytestmark = pytest.mark.gpu


def _inputs(o, v, naux):
    s = draw_system(o, v, naux, seed=820 + v)
    return np.ascontiguousarray(s.B_vv), draw_pair_symmetric(o, v, 821 + v, 0.01)


def _run(f, B, T, **kw):
    import torch
    R = torch.zeros(T.shape, dtype=torch.float64, device="cuda")
    f(dev(B), dev(T), R, **kw)
    return host(R)


@pytest.mark.parametrize("o,v,naux", [(9, 97, 24), (8, 112, 20), (10, 112, 20), (7, 128, 17), (12, 160, 9)])
def test_fp64_matches_oracle(o, v, naux):
    from paper_1810_08142_amd import ppl
    print(f"ppl_sym fp64 o={o} v={v} naux={naux}", flush=True)
    B, T = _inputs(o, v, naux)
    got = _run(ppl.ppl_sym, B, T)
    assert rel_max(got, native.ppl(B, T)) <= 1e-11
    assert np.array_equal(got, _run(ppl.ppl_sym, B, T))


@pytest.mark.parametrize("precision,o,v,naux", [("fp32", 25, 177, 9), ("fp32", 16, 230, 9), ("bf16x3", 4, 290, 9),
                                                 ("bf16x3", 44, 261, 9)])
def test_reduced_precision_matches_the_plain_ladder(precision, o, v, naux):
    from paper_1810_08142_amd import ppl
    print(f"ppl_sym {precision} o={o} v={v} naux={naux}", flush=True)
    B, T = _inputs(o, v, naux)
    got = _run(ppl.ppl_sym, B, T, precision=precision)
    err = np.abs(got - _run(ppl.ppl, B, T))
    assert np.all(err <= 2e-4 * _run(ppl.ppl, np.abs(B), np.abs(T)))
    assert np.array_equal(got, got.transpose(1, 0, 3, 2))
