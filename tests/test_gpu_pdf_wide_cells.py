"""Grids of wide cells: a batch that fills the chip gives what small batches
give, to twice the FP64 bar of the interpolation (1e-13 of the value or of the
largest node here, 1)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

N, SMALL = 20_011, 16_383


@pytest.mark.parametrize("knots", [[1e-250, 1e-249, 1e-248, 1e250, 1e251], [1e-9, 1e-3, 0.7, 0.9, 1.0]])
def test_wide_cells(vgx, knots):
    import torch
    k = np.array(knots)
    rng = np.random.default_rng(4)
    xf = [rng.uniform(0.1, 1.0, (2, 5, 5))]
    lo, hi = np.log(k[0]), np.log(k[-1])
    x, q2 = (torch.tensor(np.clip(np.exp(rng.uniform(lo, hi, N)), k[0], k[-1]), device="cuda") for _ in "xq")
    print(f"wide cells {knots}", flush=True)
    ctx = vgx.pdf_create(k, [k], xf)
    try:
        got, ref = (torch.empty((2, N), dtype=torch.float64, device="cuda") for _ in "gr")
        vgx.pdf_interp(ctx, x, q2, got)
        for a in range(0, N, SMALL):
            o = torch.empty((2, min(SMALL, N - a)), dtype=torch.float64, device="cuda")
            vgx.pdf_interp(ctx, x[a:a + SMALL].clone(), q2[a:a + SMALL].clone(), o)
            ref[:, a:a + SMALL] = o
    finally:
        vgx.pdf_destroy(ctx)
    got, ref = got.cpu().numpy(), ref.cpu().numpy()
    assert np.isfinite(ref).all()
    assert (np.abs(got - ref) <= 2e-13 * np.maximum(np.abs(ref), 1.0)).all()
