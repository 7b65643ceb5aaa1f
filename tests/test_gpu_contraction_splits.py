"""FP64 contractions on the 128 x 128 tiles loaded straight to LDS, split over the summed
index: at least 128 rows and columns, at least 32 chunks of 16 summed indices per split and a
tile for every CU, with the last split shorter than the others.

At o=17 v=144 the occupied-pair product (289 x 289, the summed pair in two levels, both
operands contiguous along it) takes 40 splits of its 1296 chunks, the virtual-virtual product
of the residual (144 x 144, three summed levels, the second operand contiguous along its
columns) 79 of 2601.  At o=8 v=130 naux=2064 the integrals (ia|jb) (1040 x 1040, both operands
contiguous along their rows) take 4 of 129.

Tolerance: FP64 results differ from the oracle's by summation order only, 1e-11 of the largest
value (at most 5e4 terms of random sign: 5e4^0.5 * 2^-53 = 2.5e-14 of a term's size, with room
for cancellation)."""
import numpy as np
import pytest

from gpu_util import dev, host, rel_max
from oracle import ccsd as oc
from paper_1810_08142_amd.synthetic import draw_matrix, draw_pair_symmetric, draw_system

pytestmark = pytest.mark.gpu


def test_residual_with_split_pair_products():
    from paper_1810_08142_amd import ccsd
    o, v, naux = 17, 144, 33
    s = draw_system(o, v, naux, seed=830, scale=0.2)
    t1 = draw_matrix((o, v), 831, 0.05)
    t2 = draw_pair_symmetric(o, v, 832, 0.05)
    om1, om2 = ccsd.residual(dev(s.B), dev(s.eps), o, dev(t1), dev(t2))
    r1, r2 = oc.residual(s.B, s.eps, o, t1, t2)
    assert rel_max(host(om1), r1) <= 1e-11
    assert rel_max(host(om2), r2) <= 1e-11


def test_mp2_with_split_integrals():
    from paper_1810_08142_amd import ccsd
    o, v, naux = 8, 130, 2064
    s = draw_system(o, v, naux, seed=840, scale=0.2)
    t2 = ccsd.mp2_guess(dev(s.B), dev(s.eps), o)[0]
    ref = oc.mp2(s.B, s.eps, o)[1]
    assert rel_max(host(t2), ref) <= 1e-11
