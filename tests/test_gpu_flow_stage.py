"""The fused backward's weight gradients at every number of transformed
coordinates it takes (|B| = 1 to 4: both row lengths of its LDS stages) and at
sample counts around its tiles and groups, against the BF16-operand model,
with the bars of test_gpu_flow (each parameter tensor 1e-2 in relative L2
norm, the loss 1e-3)."""
import numpy as np
import pytest

from flow_model import H, K, L, random_theta, weights_bf16
from oracle.integrands import gauss
from test_gpu_flow import check_gradient_against_model, make_flow

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,n", [(2, 4097), (3, 4095), (5, 4097), (6, 8192 + 31), (7, 4096 + 129), (8, 4099)])
def test_gradient_matches_model(vgx, dim, n):
    import torch
    print(f"flow stage dim={dim} n={n}", flush=True)
    th = random_theta(dim, 60 + dim, out_scale=0.05)
    y = np.random.default_rng(dim).uniform(size=(n, dim))
    g = gauss(y, 0.5, 0.25) + 0.05
    f = make_flow(vgx, dim, th)
    try:
        loss, grad = vgx.flow_loss_grad(f, torch.tensor(y.T.copy(), device="cuda"), torch.tensor(g, device="cuda"),
                                        vgx.flow_num_params(dim, L, K, H))
    finally:
        vgx.flow_destroy(f)
    check_gradient_against_model(grad, loss, weights_bf16(th, dim), y, g, dim)
