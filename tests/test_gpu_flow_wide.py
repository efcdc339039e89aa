"""Sampling and density of large batches (twelve waves per workgroup; eight
where the LDS does not hold twelve waves' columns, d = 11) against small ones:
a sample does not depend on the batch, so the outputs are equal bit for bit."""
import numpy as np
import pytest

from flow_model import H, K, L, random_theta

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", [2, 3, 8, 11])
@pytest.mark.parametrize("n", [131_073, 200_011])
def test_large_batches_equal_small_ones(vgx, dim, n):
    import torch
    print(f"flow wide dim={dim} n={n}", flush=True)
    f = vgx.flow_create(dim, random_theta(dim, 5), L, K, H)

    def new(m):
        return (torch.full((dim, m), -1.0, dtype=torch.float64, device="cuda"),
                torch.full((m,), -1.0, dtype=torch.float64, device="cuda"))
    try:
        y, lq = new(n)
        vgx.flow_sample(f, n, 11, 2, 1, y, lq)
        u, lu = new(n)
        vgx.flow_density(f, y, lu, u=u)
        m = 100_000
        ys, lqs = new(m)
        vgx.flow_sample(f, m, 11, 2, 1, ys, lqs)
        assert torch.equal(y[:, :m], ys) and torch.equal(lq[:m], lqs)
        for a in range(0, n, m):
            b = min(a + m, n)
            us, lus = new(b - a)
            vgx.flow_density(f, y[:, a:b].contiguous(), lus, u=us)
            assert torch.equal(u[:, a:b], us) and torch.equal(lu[a:b], lus)
        assert np.isfinite(lq.cpu().numpy()).all()
    finally:
        vgx.flow_destroy(f)
