"""Large multi-member calls (nodes in an LDS box) against small ones (nodes
from memory): the same weights, products and summation order, so the outputs
are equal bit for bit, for neighbouring points (a box), scattered ones (too
large a box), points outside the grid and workgroups without a point inside."""
import numpy as np
import pytest

from test_gpu_pdf_shapes import random_grid

pytestmark = pytest.mark.gpu


def points(grid, n, kind, rng):
    x0, x1 = grid.x_knots[0], grid.x_knots[-1]
    qs = np.concatenate(grid.q2_knots)
    if kind == "table":
        x, q2 = np.exp(np.linspace(np.log(x0), np.log(x1), n)), np.full(n, np.sqrt(qs[0] * qs[1]))
        x[0], x[-1] = x0, x1
    else:
        x = np.clip(np.exp(rng.uniform(np.log(x0), np.log(x1), n)), x0, x1)
        q2 = np.clip(np.exp(rng.uniform(np.log(qs[0]), np.log(qs[-1]), n)), qs[0], qs[-1])
    q2[300:600] = 0.1 * qs[0]  # a whole workgroup outside, and parts of two more
    x[1000] = 2.0 * x1
    return x, q2


@pytest.mark.parametrize("out", ["f64", "f32"])
@pytest.mark.parametrize("kind", ["table", "random"])
@pytest.mark.parametrize("n_flav,n_x,nqs", [(1, 2, [2]), (3, 90, [2, 9]), (11, 196, [5, 12]), (13, 40, [30])])
def test_box_equals_gather(vgx, n_flav, n_x, nqs, kind, out):
    import torch
    members, n = 331, 1451  # 331 x 1451 values: beyond the box's threshold in both types
    print(f"members box n_flav={n_flav} n_x={n_x} {kind} {out}", flush=True)
    rng = np.random.default_rng(n_flav)
    grid = random_grid(n_flav, n_x, nqs, 3)
    if n_x > 50:  # keep the knots' span moderate
        grid.x_knots = np.exp(np.linspace(np.log(1e-7), np.log(0.9), n_x))
    x, q2 = points(grid, n, kind, rng)
    sets = [[v * (1.0 + 0.01 * m) for v in grid.xf] for m in range(members)]
    dt = torch.float64 if out == "f64" else torch.float32
    ctx = vgx.pdf_create_set(grid.x_knots, grid.q2_knots, sets)
    try:
        xt, qt = torch.from_numpy(x).cuda(), torch.from_numpy(q2).cuda()
        big = torch.empty((members, n_flav, n), dtype=dt, device="cuda")
        vgx.pdf_interp_members(ctx, xt, qt, big)
        assert vgx.pdf_out_of_range(ctx) == 301
        for a in range(0, n, 300):
            b = min(a + 300, n)
            part = torch.empty((members, n_flav, b - a), dtype=dt, device="cuda")
            vgx.pdf_interp_members(ctx, xt[a:b].clone(), qt[a:b].clone(), part)
            assert torch.equal(torch.nan_to_num(part, nan=-1e30), torch.nan_to_num(big[:, :, a:b], nan=-1e30))
        bad = torch.isnan(big).all(0).all(0).cpu().numpy()
        assert bad.sum() == 301 and bad[300:600].all() and bad[1000]
    finally:
        vgx.pdf_destroy(ctx)
