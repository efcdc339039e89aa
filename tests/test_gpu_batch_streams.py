"""A batch on a stream of its own takes its contexts where their streams leave
them: whatever is still queued there (iterations, refinements, a record not
yet completed) comes first.  The reference makes the same calls on one
stream, so every sum agrees bit for bit; workgroups of one wave, since
several waves add to a workgroup's histogram in no fixed order."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

DIM, NB, N = 3, 20, 4001
LONG = 20_000_000  # the context's stream is milliseconds behind when the batch is called


def run(vgx, order, own, batch):
    """a: a long queued iteration, s: a synchronous one, r: a refinement, b: the batch."""
    v = vgx.vegas_create(vgx.GAUSS, DIM, NB, 1.5, 9, 1, vgx.F64, np.array([0.4, 0.5, 0.6, 0.2, 0.1, 0.3]), stream=own)
    b = vgx.batch_create([v], [N], 1024, 64, stream=batch)
    got = []
    try:
        for it, c in enumerate(order):
            if c == "a":
                vgx.vegas_iterate_async(v, LONG, it)
            elif c == "s":
                got.append(vgx.vegas_iterate(v, N, it))
            elif c == "r":
                vgx.vegas_refine(v)
            else:
                got.append(vgx.batch_iterate(b, it, 1)[0])
        return got, vgx.vegas_results(v), vgx.vegas_result(v), vgx.vegas_get_grid(v, DIM, NB)
    finally:
        vgx.batch_destroy(b)
        vgx.vegas_destroy(v)


@pytest.mark.parametrize("order", ["arb", "abrb", "ab", "srb", "ararb", "barb"])
def test_batch_follows_the_contexts_stream(vgx, order):
    import torch
    print(f"batch streams {order}", flush=True)
    one = torch.cuda.Stream()
    got, rec, res, grid = run(vgx, order, torch.cuda.Stream(), torch.cuda.Stream())
    got1, rec1, res1, grid1 = run(vgx, order, one, one)
    assert got == got1 and rec == rec1 and res == res1
    assert np.array_equal(grid, grid1)


def test_batch_refines_after_the_samples_are_drawn(vgx):
    """vegas_sample reads the grid on the context's stream; a batch refines it on another."""
    import torch
    own, batch = torch.cuda.Stream(), torch.cuda.Stream()
    v = vgx.vegas_create(vgx.GAUSS, DIM, NB, 1.5, 9, 1, vgx.F64, np.array([0.4, 0.5, 0.6, 0.2, 0.1, 0.3]), stream=own)
    b = vgx.batch_create([v], [N], 1024, 64, stream=batch)
    try:
        want, got = (torch.empty(LONG, dtype=torch.float64, device="cuda") for _ in "wg")
        torch.cuda.synchronize()
        vgx.vegas_sample(v, 0, LONG, 7, g=want)
        torch.cuda.synchronize()
        vgx.vegas_sample(v, 0, LONG, 7, g=got)
        vgx.batch_iterate(b, 0, 1)
        torch.cuda.synchronize()
        assert torch.equal(got, want)
    finally:
        vgx.batch_destroy(b)
        vgx.vegas_destroy(v)
