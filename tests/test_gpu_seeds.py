"""Hankel seeds at small arguments: waves that are all below 1/2, all below 2, or mixed take
series of different lengths; each is held to 40-digit values.

Bound: the terms dropped are below 1e-17 of H; the sums of some ten terms of decaying size round to a
few 1e-16; the logarithm adds one ulp: 2e-15 of |H|, which the longer series keep too.
"""
import mpmath as mp
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

RANGES = [(1e-9, 1e-6), (1e-4, 0.01), (0.01, 0.4999999), (0.45, 0.55), (0.5, 1.0), (1.0, 1.9999999),
          (1.9, 2.1), (0.3, 4.1), (3.9, 6.1), (0.01, 30.0)]


@pytest.mark.parametrize("lo,hi", RANGES)
def test_seeds(lo, hi):
    from paper_1207_4461_amd import qbx

    z = np.exp(np.random.default_rng(1).uniform(np.log(lo), np.log(hi), 64))
    z[0], z[-1] = lo, hi
    h = [t.cpu().numpy() for t in qbx.hankel01(torch.from_numpy(z).cuda())]
    with mp.workdps(40):
        for n in (0, 1):
            ref = [mp.hankel1(n, mp.mpf(float(x))) for x in z]
            err = [float(abs(mp.mpc(v.real, v.imag) - r) / abs(r)) for v, r in zip(h[n], ref)]
            assert max(err) < 2e-15


def test_seeds_at_the_ends_of_the_range():
    """z = 0, subnormal and negative: the logarithm's limits, as the library's has them."""
    from paper_1207_4461_amd import qbx

    z = np.array([0.0, 5e-324, 1e-310, 2.3e-308, -1e-310, -0.3, -1.5, -3.9, float("nan"), 0.7])
    h0, h1 = (t.cpu().numpy() for t in qbx.hankel01(torch.from_numpy(z).cuda()))
    assert h0[0].real == 1.0 and h0[0].imag == -np.inf and h1[0].real == 0.0
    for i in (1, 2, 3, 9):
        ref = mp.hankel1(0, mp.mpf(float(z[i])))
        assert abs(h0[i].imag - float(ref.imag)) < 2e-15 * abs(ref)
    assert np.isnan(h0[4:9].imag).all() and np.isnan(h1[4:9].imag).all()
    for i in (5, 6, 7):   # the series of J are even and odd; Y has no real value
        assert abs(h0[i].real - float(mp.besselj(0, float(z[i])))) < 4e-15
        assert abs(h1[i].real - float(mp.besselj(1, float(z[i])))) < 4e-15
    assert np.isnan(h0[8].real) and np.isnan(h1[8].real)
