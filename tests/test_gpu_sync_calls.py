"""Calls that the header marks "sync" leave nothing of their stream's work
undone when they return: the stream is idle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

DIM, NB = 8, 256  # a histogram of 2048 columns: the reduction runs on beyond the record's workgroup


@pytest.fixture
def ctx(vgx):
    import torch
    st = torch.cuda.Stream()
    v = vgx.vegas_create(vgx.GAUSS, DIM, NB, 1.5, 3, 0, vgx.F64,
                         np.concatenate([np.full(DIM, 0.5), np.full(DIM, 0.3)]), stream=st)
    yield v, st
    vgx.vegas_destroy(v)


def test_vegas_calls(vgx, ctx):
    import torch
    v, st = ctx
    busy = []

    def check(name, f):
        for _ in range(20):
            f()
            busy.append(name) if not st.query() else None

    edges = np.tile(np.arange(NB + 1) / NB, (DIM, 1))
    y = torch.rand(DIM, 200_000, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    check("vegas_iterate", lambda: vgx.vegas_iterate(v, 200_000, 0))
    check("vegas_set_grid", lambda: vgx.vegas_set_grid(v, edges))
    check("vegas_iterate_points", lambda: vgx.vegas_iterate_points(v, y, None))
    vgx.vegas_iterate(v, 200_000, 0)
    check("vegas_results", lambda: (vgx.vegas_refine(v), vgx.vegas_results(v)))
    check("vegas_get_grid", lambda: (vgx.vegas_refine(v), vgx.vegas_get_grid(v, DIM, NB)))
    assert not busy, f"work left after {sorted(set(busy))}"


def test_flow_vegas_iterate(vgx, ctx):
    v, st = ctx
    rng = np.random.default_rng(2)
    parts = [rng.standard_normal(size) * (np.sqrt(2 / fan) if kind == "w" else 0.1)
             for kind, fan, size in vgx.flow_param_layout(DIM)]
    f = vgx.flow_create(DIM, np.concatenate(parts).astype(np.float32), stream=st)
    try:
        for it in range(20):
            vgx.flow_vegas_iterate(f, v, 50_000, 1, 2, it, allow_fallback=True)
            assert st.query()
    finally:
        vgx.flow_destroy(f)
