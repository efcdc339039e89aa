"""The fused iteration's coordinates are those of vegas_sample bit for bit,
for odd bin counts too: a Gaussian of width 1e-9 at 0.5 turns half a unit in
the last place of x (5.5e-17) into 5e-8 of its weight, and the sums agree to
the bar of FP64 sums (1e-12: both sides evaluate the same exponent, their
exponentials and Jacobians are good to a few units in the last place)."""
import math

import numpy as np
import pytest

from synth.batch import GAUSS

pytestmark = pytest.mark.gpu

S = 1e-9


def narrow_grid(dim, nb):
    """The middle bin spans three widths on either side of 0.5."""
    m = nb // 2
    lo = (0.5 - 3 * S) * np.arange(m + 1) / max(m, 1)
    hi = 1.0 - (0.5 - 3 * S) * np.arange(nb - m)[::-1] / max(nb - m - 1, 1)
    return np.tile(np.concatenate([lo, hi]), (dim, 1))


@pytest.mark.parametrize("path", ["iterate", "batch"])
@pytest.mark.parametrize("dim,nb", [(1, 3), (2, 3), (1, 4), (1, 49), (4, 5), (5, 3), (1, 255), (1, 256)])
def test_same_coordinates(vgx, dim, nb, path):
    import torch
    n = 50_021
    print(f"odd word map dim={dim} nb={nb} {path}", flush=True)
    v = vgx.vegas_create(GAUSS, dim, nb, 1.5, 5, 2, vgx.F64, np.concatenate([np.full(dim, 0.5), np.full(dim, S)]))
    try:
        vgx.vegas_set_grid(v, narrow_grid(dim, nb))
        g = torch.empty(n, dtype=torch.float64, device="cuda")
        vgx.vegas_sample(v, 0, n, 3, g=g)
        if path == "iterate":
            r = vgx.vegas_iterate(v, n, 3)
        else:
            b = vgx.batch_create([v], [n], 4096, 256)
            try:
                r = vgx.batch_iterate(b, 3, 1)[0]
            finally:
                vgx.batch_destroy(b)
        g = g.cpu().numpy()
        assert np.count_nonzero(g) >= 10
        assert r["s1"] == pytest.approx(math.fsum(g), rel=1e-12)
        assert r["s2"] == pytest.approx(math.fsum(g * g), rel=1e-12)
    finally:
        vgx.vegas_destroy(v)
