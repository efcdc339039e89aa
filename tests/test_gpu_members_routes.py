"""Multi-member calls on both sides of the lines where the kernel with the LDS
box is taken (values, points, members, flavours, how full the last workgroup
is): bit for bit the outputs of the same points in parts of 250, which are read
from memory."""
import numpy as np
import pytest

from test_gpu_pdf_members_box import points
from test_gpu_pdf_shapes import random_grid

pytestmark = pytest.mark.gpu

# flavours, members, points: a box for FP64 (11 flavours, from 700 points and 150000 values), for FP32 (from 5
# flavours, 4 members, 1000 points and 600000 values, workgroups nine tenths full), and just not
SHAPES = [(11, 215, 1001), (11, 149, 1001), (11, 86, 1749), (11, 400, 1501), (11, 400, 1537), (11, 4, 151_001),
          (11, 3, 200_001), (5, 420, 1451), (4, 420, 1451), (13, 410, 1500), (11, 601, 1002), (16, 600, 1024)]


@pytest.mark.parametrize("out", ["f64", "f32"])
@pytest.mark.parametrize("n_flav,members,n", SHAPES)
def test_routes_agree(vgx, n_flav, members, n, out):
    import torch
    print(f"members routes n_flav={n_flav} {members}x{n} {out}", flush=True)
    rng = np.random.default_rng(n_flav)
    grid = random_grid(n_flav, 60, [4, 9], 3)
    grid.x_knots = np.exp(np.linspace(np.log(1e-7), np.log(0.9), 60))
    x, q2 = points(grid, n, "table", rng)
    ctx = vgx.pdf_create_set(grid.x_knots, grid.q2_knots, [[v * (1.0 + 0.01 * m) for v in grid.xf] for m in range(members)])
    dt = torch.float64 if out == "f64" else torch.float32
    try:
        xt, qt = torch.from_numpy(x).cuda(), torch.from_numpy(q2).cuda()
        big = torch.empty((members, n_flav, n), dtype=dt, device="cuda")
        vgx.pdf_interp_members(ctx, xt, qt, big)
        step = 250 if n < 2000 else 37_000 if members == 4 else 49_000
        for a in range(0, n, step):
            b = min(a + step, n)
            part = torch.empty((members, n_flav, b - a), dtype=dt, device="cuda")
            vgx.pdf_interp_members(ctx, xt[a:b].clone(), qt[a:b].clone(), part)
            assert torch.equal(torch.nan_to_num(part, nan=-1e30), torch.nan_to_num(big[:, :, a:b], nan=-1e30))
        assert int(torch.isnan(big[0, 0]).sum()) == 301
    finally:
        vgx.pdf_destroy(ctx)
