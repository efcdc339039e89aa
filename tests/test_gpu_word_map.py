"""The fused iteration's grid map (Philox words straight to bins) at the
smallest, odd and largest bin counts, and the Gaussian's exponential where it
underflows, against the FP64 oracle.

Bars: rounding order only, 1e-12, as for the other FP64 iterations.  A narrow
Gaussian amplifies the rounding of x (2e-16 here): z = (x - c)/(sigma sqrt 2)
moves by 2e-13 for sigma = 1e-3, sum z^2 < 745 where exp does not underflow, so
over up to six dimensions the exponent moves by less than 2 sqrt(6 745) 2e-13
= 2.7e-11 and a squared weight by twice that: 1e-10.
"""
import math

import numpy as np
import pytest

from oracle import vegas as ov
from oracle.integrands import gauss
from synth.batch import GAUSS

pytestmark = pytest.mark.gpu


def grid(dim, nb, seed):
    w = np.random.default_rng(seed).uniform(0.2, 1.0, (dim, nb))
    e = np.concatenate([np.zeros((dim, 1)), np.cumsum(w, axis=1)], axis=1)
    e /= e[:, -1:]
    e[:, -1] = 1.0
    return e


@pytest.mark.parametrize("sigma,bar", [(0.2, 1e-12), (1e-3, 1e-10)])
@pytest.mark.parametrize("dim,nb", [(1, 2), (2, 3), (3, 49), (4, 64), (2, 255), (6, 256)])
def test_bins_and_sums(vgx, dim, nb, sigma, bar):
    n = 30_011
    print(f"word map dim={dim} nb={nb} sigma={sigma}", flush=True)
    v = vgx.vegas_create(GAUSS, dim, nb, 1.5, 21, 4, vgx.F64,
                         np.concatenate([np.full(dim, 0.5), np.full(dim, sigma)]))
    try:
        e = grid(dim, nb, nb)
        vgx.vegas_set_grid(v, e)
        r = vgx.vegas_iterate(v, n, 3)
        h = vgx.vegas_get_hist(v, dim, nb)
        ref = ov.iteration(lambda x: gauss(x, 0.5, sigma), e, 21, 4, 3, n)
        assert r["s1"] == pytest.approx(ref["s1"], rel=bar, abs=1e-300)
        assert r["s2"] == pytest.approx(ref["s2"], rel=bar, abs=1e-300)
        assert np.allclose(h, ref["hist"], rtol=bar, atol=1e-300)
    finally:
        vgx.vegas_destroy(v)


@pytest.mark.parametrize("centre", [math.nan, math.inf, -math.inf])
def test_centres_that_are_not_finite(vgx, centre):
    v = vgx.vegas_create(GAUSS, 2, 16, 1.5, 1, 0, vgx.F64, np.array([0.5, centre, 0.2, 0.2]))
    try:
        if math.isnan(centre):  # a NaN estimate is reported as such
            with pytest.raises(vgx.VgxError, match="mean=nan"):
                vgx.vegas_iterate(v, 1000, 0)
        else:
            assert vgx.vegas_iterate(v, 1000, 0)["s1"] == 0.0
    finally:
        vgx.vegas_destroy(v)
