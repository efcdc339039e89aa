"""A batch's LDS histograms at each number of columns per bin (1 to 16, by the
histogram's size) against the single-integral path: the same samples added in
another order, hence the bar for FP64 sums (1e-12)."""
import numpy as np
import pytest

from synth.batch import GAUSS

pytestmark = pytest.mark.gpu

SHAPES = [(12, 256), (12, 200), (12, 100), (6, 100), (5, 64), (3, 7), (1, 2)]  # 1, 2, 4, 8, 16, 16, 16 columns


@pytest.mark.parametrize("block", [64, 256])
def test_columns_match_single_path(vgx, block):
    n = 20_011
    print(f"batch columns block={block}", flush=True)

    def make(k, dim, nb):
        return vgx.vegas_create(GAUSS, dim, nb, 1.5, 8, k, vgx.F64,
                                np.concatenate([np.full(dim, 0.45), np.full(dim, 0.3)]))
    A = [make(k, *s) for k, s in enumerate(SHAPES)]
    B = [make(k, *s) for k, s in enumerate(SHAPES)]
    try:
        b = vgx.batch_create(A, [n] * len(SHAPES), 4096, block)
        try:
            rb = vgx.batch_iterate(b, 0, len(SHAPES))
        finally:
            vgx.batch_destroy(b)
        for k, (dim, nb) in enumerate(SHAPES):
            rs = vgx.vegas_iterate(B[k], n, 0)
            assert rb[k]["s1"] == pytest.approx(rs["s1"], rel=1e-12)
            assert rb[k]["s2"] == pytest.approx(rs["s2"], rel=1e-12)
            assert np.allclose(vgx.vegas_get_hist(A[k], dim, nb), vgx.vegas_get_hist(B[k], dim, nb), rtol=1e-12, atol=0)
    finally:
        for c in A + B:
            vgx.vegas_destroy(c)
