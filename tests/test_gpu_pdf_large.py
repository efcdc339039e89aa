"""GPU PDF interpolation of large batches (the kernels with the grid in LDS)
against the oracle, and against the same queries in batches small enough
for the gathering kernel.

Bars: against the oracle those of the small batches (FP64 1e-13, FP32 1e-5,
relative or of the largest stencil node).  Against the gathering kernel,
twice the FP64 bar (each side may be off by one), plus one FP32 rounding
where the output is FP32: both sum the same FP32 nodes in FP64."""
import numpy as np
import pytest

from oracle import pdf as opdf
from synth import nonuniform_pdf_grid, synthetic_pdf_grid
from tests.test_gpu_pdf import check, stencil_scale
from tests.test_gpu_pdf_shapes import random_grid

pytestmark = pytest.mark.gpu

SMALL = 16_383   # the largest batch of the gathering kernel


def grid_of(kind):
    if kind == "even":
        return synthetic_pdf_grid()
    if kind == "uneven":
        return nonuniform_pdf_grid()
    n_flav, n_x, nqs = kind
    return random_grid(n_flav, n_x, nqs, 7)


def queries(grid, n, seed, outside):
    """Log-uniform points of the grid, with its knots, thresholds and corners;
    with `outside` also points around it and values that are no points."""
    rng = np.random.default_rng(seed)
    x0, x1 = grid.x_knots[0], grid.x_knots[-1]
    qs = np.concatenate(grid.q2_knots)
    x = np.clip(np.exp(rng.uniform(np.log(x0), np.log(x1), n)), x0, x1)
    q2 = np.clip(np.exp(rng.uniform(np.log(qs[0]), np.log(qs[-1]), n)), qs[0], qs[-1])
    k = rng.permutation(n)[:n // 8]
    x[k] = rng.choice(grid.x_knots, k.size)
    k = rng.permutation(n)[:n // 8]
    q2[k] = rng.choice(qs, k.size)
    x[:4], q2[:4] = [x0, x0, x1, x1], [qs[0], qs[-1], qs[0], qs[-1]]
    if outside:
        odd = [np.nan, np.inf, -np.inf, 0.0, -1.0, 5e-324, 1e300]
        for a, lo, hi in ((x, x0, x1), (q2, qs[0], qs[-1])):
            k = rng.permutation(n)[:64]
            a[k] = rng.choice(odd + [lo * (1 - 1e-15), hi * (1 + 1e-15), lo / 3, hi * 3], k.size)
    return x, q2


def interp(vgx, ctx, x, q2, n_flav, dt):
    import torch
    out = torch.full((n_flav, x.numel()), -7.0, dtype=dt, device="cuda")
    vgx.pdf_interp(ctx, x, q2, out)
    return out, vgx.pdf_out_of_range(ctx)


CASES = [("even", SMALL + 1, 0), ("uneven", SMALL + 2, 1), ("uneven", 100_003, 2), ("even", 999_999, 0),
         ("even", 1_000_000, 1), ("uneven", 1_000_003, 0), ("even", 1_000_001, 2),
         ((1, 4, [4]), 1_000_001, 0), ((2, 6, [2, 3]), 1_000_001, 0), ((3, 9, [2, 2, 4]), 40_001, 1),
         ((5, 20, [3, 9]), 70_001, 2), ((13, 40, [5, 30, 6]), 1_000_001, 0), ((16, 9, [6, 4]), 1_000_001, 2)]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_large_batches_match_small_ones_and_the_oracle(vgx, case, dtype):
    import torch
    kind, n, mode = CASES[case]
    print(f"pdf large {kind} n={n} mode={mode} {dtype}", flush=True)
    grid = grid_of(kind)
    x, q2 = queries(grid, n, 100 + case, outside=True)
    ctx = vgx.pdf_create(grid.x_knots, grid.q2_knots, grid.xf)
    dt = torch.float64 if dtype == "f64" else torch.float32
    try:
        vgx.pdf_set_extrapolation(ctx, mode)
        xt, qt = torch.tensor(x, device="cuda"), torch.tensor(q2, device="cuda")
        got, lost = interp(vgx, ctx, xt, qt, grid.n_flav, dt)
        ref, lost_ref = torch.empty_like(got), 0
        for lo in range(0, n, SMALL):
            o, k = interp(vgx, ctx, xt[lo:lo + SMALL].clone(), qt[lo:lo + SMALL].clone(), grid.n_flav, dt)
            ref[:, lo:lo + SMALL] = o
            lost_ref += k
    finally:
        vgx.pdf_destroy(ctx)
    got, ref = got.double().cpu().numpy(), ref.double().cpu().numpy()
    assert lost == lost_ref
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    qs = np.concatenate(grid.q2_knots)
    cx, cq = np.clip(x, grid.x_knots[0], grid.x_knots[-1]), np.clip(q2, qs[0], qs[-1])
    keep = np.isfinite(cx) & np.isfinite(cq)
    scale = np.zeros(n)
    scale[keep] = stencil_scale(grid, cx[keep], cq[keep])
    fine = ~np.isnan(ref) & keep
    bar = (2e-13 + (2.0 ** -23 if dtype == "f32" else 0.0)) * np.abs(ref) + 2e-13 * scale
    with np.errstate(invalid="ignore"):  # the continuation's infinities, the same in both batches
        off = fine & (got != ref) & ~(np.abs(got - ref) <= bar)
    assert not off.any(), f"{off.sum()} off, first at {np.argwhere(off)[:3]}"
    inside = np.flatnonzero((x >= grid.x_knots[0]) & (x <= grid.x_knots[-1]) & (q2 >= qs[0]) & (q2 <= qs[-1]))
    s = np.concatenate([inside[:50], np.random.default_rng(1).choice(inside, 4000, replace=False), inside[-50:]])
    ok, r = check(got[:, s], opdf.interp(grid, x[s], q2[s]), scale[s], 1e-13 if dtype == "f64" else 1e-5)
    assert ok.all(), f"worst r_i {r[~ok].max():.3e}"


@pytest.mark.parametrize("n", [SMALL + 1, 1_000_000])
def test_node_values_exact_in_large_batches(vgx, c1_grid, n):
    """On knots of both axes the node values come back bit for bit, the
    vanishing ones at the last x knot included."""
    import torch
    s, qs = 2, c1_grid.q2_knots[2]
    i, j = np.arange(n) % 196, (np.arange(n) // 196) % len(qs)
    ctx = vgx.pdf_create(c1_grid.x_knots, c1_grid.q2_knots, c1_grid.xf)
    try:
        x, q2 = torch.tensor(c1_grid.x_knots[i], device="cuda"), torch.tensor(qs[j], device="cuda")
        got, lost = interp(vgx, ctx, x, q2, 11, torch.float64)
    finally:
        vgx.pdf_destroy(ctx)
    assert lost == 0
    assert np.array_equal(got.cpu().numpy(), c1_grid.xf[s][:, j, i])


def test_outputs_over_the_queries(vgx, c1_grid):
    """Queries in the first row of the outputs are read before they are overwritten."""
    import torch
    n = 1_000_003
    ctx = vgx.pdf_create(c1_grid.x_knots, c1_grid.q2_knots, c1_grid.xf)
    try:
        x, q2 = (torch.tensor(a, device="cuda") for a in queries(c1_grid, n, 5, outside=False))
        ref, _ = interp(vgx, ctx, x, q2, 11, torch.float64)
        out = torch.empty((11, n), dtype=torch.float64, device="cuda")
        out[0] = x
        vgx.pdf_interp(ctx, out[0], q2, out)
        scale = stencil_scale(c1_grid, x.cpu().numpy(), q2.cpu().numpy())
        ok, _ = check(out.cpu().numpy(), ref.cpu().numpy(), scale, 2e-13)
        assert ok.all()
    finally:
        vgx.pdf_destroy(ctx)
