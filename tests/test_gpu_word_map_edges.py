"""The fused iteration where its map reads the edges (many dimensions and
bins, the FP64 Gaussian from ten dimensions on) and just where it reads the
bins' table: the samples of vegas_sample, summed, for both parities.  Bars:
FP64 sums 1e-12; FP32 integrands 1e-6 of the sum (each weight is rounded alike
on both sides but for the last bits of FP32 functions, 2^-23 relative each)."""
import math

import numpy as np
import pytest

from synth.batch import GAUSS, GENZ_OSC, GENZ_PEAK

pytestmark = pytest.mark.gpu

SHAPES = [(8, 95), (8, 96), (8, 97), (9, 85), (9, 86), (10, 2), (10, 51), (10, 83), (10, 84), (11, 7), (11, 76),
          (12, 64), (12, 69), (12, 70), (12, 255), (12, 256)]


@pytest.mark.parametrize("kind", [GAUSS, GENZ_OSC, GENZ_PEAK])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_sums_of_the_samples(vgx, kind, prec):
    import torch
    n = 40_013
    for dim, nb in SHAPES:
        print(f"word map edges kind={kind} {prec} dim={dim} nb={nb}", flush=True)
        par = np.concatenate([[0.3], np.full(dim, 0.4)]) if kind == GENZ_OSC else np.concatenate([np.full(dim, 0.5), np.full(dim, 0.4)])
        v = vgx.vegas_create(kind, dim, nb, 1.5, 6, 3, vgx.F64 if prec == "f64" else vgx.F32, par)
        try:
            w = np.random.default_rng(nb).uniform(0.3, 1.0, (dim, nb))
            e = np.concatenate([np.zeros((dim, 1)), np.cumsum(w, axis=1)], axis=1)
            e /= e[:, -1:]
            vgx.vegas_set_grid(v, e)
            g = torch.empty(n, dtype=torch.float64, device="cuda")
            vgx.vegas_sample(v, 0, n, 1, g=g)
            r = vgx.vegas_iterate(v, n, 1)
            g = g.cpu().numpy()
            bar = 1e-12 if prec == "f64" else 1e-6
            mag = math.fsum(np.abs(g))
            assert abs(r["s1"] - math.fsum(g)) <= bar * mag
            assert r["s2"] == pytest.approx(math.fsum(g * g), rel=2 * bar)
            h = vgx.vegas_get_hist(v, dim, nb)
            assert np.allclose(h.sum(axis=1), r["s2"], rtol=1e-12)
        finally:
            vgx.vegas_destroy(v)
