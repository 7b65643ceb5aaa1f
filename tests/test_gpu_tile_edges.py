"""Ladder, contraction, (T) and solver kernels at the edges of their tiles and at the sizes
where one kernel takes over from another, against the oracle.

Tolerances: FP64 results differ from the oracle's by summation order only, 1e-11 of the
largest value (the sums have at most 1e5 terms of random sign: 1e5^0.5 * 2^-53 = 4e-14 of a
term's size, with room for cancellation); (T) 1e-10 of the energy; split-bf16 and FP32
ladders element by element within 2e-4 of the ladder of the absolute values (two rounding
stages of 3 * 2^-18 a product, FP32 accumulation)."""
import numpy as np
import pytest

from gpu_util import dev, host, rel_max
from oracle import ccsd as oc
from oracle import native
from paper_1810_08142_amd.synthetic import draw_matrix, draw_pair_symmetric, draw_system

pytestmark = pytest.mark.gpu


def _ladder(o, v, naux, precision, seed):
    import torch
    from paper_1810_08142_amd import ppl
    s = draw_system(o, v, naux, seed=seed)
    tau = draw_pair_symmetric(o, v, seed + 1)
    R = torch.zeros((o, o, v, v), dtype=torch.float64, device="cuda")
    ppl.ppl(dev(s.B_vv), dev(tau), R, precision=precision)
    return host(R), s.B_vv, tau


def _check(o, v, naux, precision, seed):
    got, B, tau = _ladder(o, v, naux, precision, seed)
    ref = native.ppl(B, tau)
    if precision == "fp64":
        assert rel_max(got, ref) <= 1e-11
    else:
        assert np.all(np.abs(got - ref) <= 2e-4 * native.ppl(np.abs(B), np.abs(tau)))


# Q steps of 32 in the split build and stages of 8 in the others: one, two, odd counts, remainders
@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("naux", [1, 8, 31, 32, 33, 64, 65, 97, 160])
def test_ladder_auxiliary_remainders(naux, precision):
    _check(3, 34, naux, precision, 700 + naux)


# every column strip of the contractions and the wide split tiles (po and pm columns)
@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("o", [1, 2, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 17, 19, 22])
def test_ladder_column_widths(o, precision):
    _check(o, 20, 40, precision, 720 + o)


# the build's small tiles up to v = 64 (ten block pairs) and large ones beyond; the unpack's
# groups of four columns up to 255 groups of sixteen and sixteen columns beyond
@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("o,v,naux", [(2, 16, 9), (2, 17, 9), (2, 63, 24), (2, 64, 24), (2, 65, 24), (2, 81, 24),
                                      (51, 20, 9), (53, 20, 9)])
def test_ladder_small_and_large_tiles(o, v, naux, precision):
    _check(o, v, naux, precision, 740 + v)


# contractions of latency-bound, middle and large tiles, even extents (loaded straight to
# LDS) and odd ones
@pytest.mark.parametrize("o,v,naux", [(3, 33, 16), (8, 40, 48), (7, 41, 33), (12, 48, 32), (4, 66, 50)])
def test_residual_across_contraction_kernels(o, v, naux):
    from paper_1810_08142_amd import ccsd
    s = draw_system(o, v, naux, seed=760 + v, scale=0.2)
    t1 = draw_matrix((o, v), 761, 0.05)
    t2 = draw_pair_symmetric(o, v, 762, 0.05)
    om1, om2 = ccsd.residual(dev(s.B), dev(s.eps), o, dev(t1), dev(t2))
    r1, r2 = oc.residual(s.B, s.eps, o, t1, t2)
    assert rel_max(host(om1), r1) <= 1e-11
    assert rel_max(host(om2), r2) <= 1e-11


# v + o = 16 m, 16 m + 1, + 4, + 15 (steps of the last chunk), 35 triplets (more than a batch)
@pytest.mark.parametrize("o,v", [(3, 13), (3, 14), (5, 15), (5, 26), (5, 27), (6, 31)])
def test_triples_summed_index_and_batches(o, v):
    from paper_1810_08142_amd import ccsd
    s = draw_system(o, v, 20, seed=780 + v, scale=0.3)
    t1 = draw_matrix((o, v), 781, 0.05)
    t2 = draw_pair_symmetric(o, v, 782, 0.05)
    ref = oc.triples(s.B, s.eps, o, t1, t2)
    got = ccsd.triples(dev(s.B), dev(s.eps), o, dev(t1), dev(t2))
    assert abs(got - ref) <= 1e-10 * abs(ref)


# inner products of short and of long vectors (2^15 elements), the longest history
@pytest.mark.parametrize("o,v,naux,diis", [(3, 20, 40, 16), (5, 40, 60, 6), (5, 40, 60, 16)])
def test_solve_with_short_and_long_vectors(o, v, naux, diis):
    from paper_1810_08142_amd import ccsd
    s = draw_system(o, v, naux, seed=790)
    t1, t2, rep = ccsd.solve(dev(s.B), dev(s.eps), o, max_iter=100, tol=1e-10, tol_energy=1e-10, diis_size=diis)
    ref = oc.solve(s.B, s.eps, o, max_iter=100, tol=1e-10, tol_energy=1e-10)
    assert rep.converged and ref.converged
    assert abs(rep.e_corr - ref.e_corr) <= 1e-10
    assert np.abs(host(t2) - ref.t2).max() <= 1e-9
    assert np.abs(host(t1) - ref.t1).max() <= 1e-9
