"""The host's copies of the records: any order of synchronous, queued and
batched iterations, refinements and resets gives the records that one fresh
context per order computes synchronously, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

DIM, NB = 3, 20
PARAMS = np.array([0.4, 0.5, 0.6, 0.2, 0.1, 0.3])


def make(vgx, stream=None):
    return vgx.vegas_create(vgx.GAUSS, DIM, NB, 1.5, 9, 1, vgx.F64, PARAMS, stream=stream)


ORDERS = ["sss", "asa", "ssaar", "sRss", "aaRsa", "sgsas", "r", "sbs", "absa"]


@pytest.mark.parametrize("side_stream", [False, True])
@pytest.mark.parametrize("order", ORDERS)
def test_records_of_any_order(vgx, order, side_stream):
    """s: synchronous, a: queued, b: batched (on its own stream with side_stream), each followed by a
    refinement; R: reset the results, r: read them, g: set the grid to itself."""
    import torch
    print(f"records {order} side_stream={side_stream}", flush=True)
    n, it = 4001, 0
    v, ref = make(vgx), make(vgx)
    st = torch.cuda.Stream() if side_stream else None
    b = vgx.batch_create([v], [n], 1024, 256, stream=st) if "b" in order else None
    want = []
    try:
        for c in order:
            if c in "sab":
                w = vgx.vegas_iterate(ref, n, it)
                if c == "s":
                    got = vgx.vegas_iterate(v, n, it)
                    assert got == w
                elif c == "a":
                    vgx.vegas_iterate_async(v, n, it)
                if c == "b":
                    torch.cuda.synchronize()  # the queued refinement runs on another stream than the batch
                    got = vgx.batch_iterate(b, it, 1)[0]
                    assert np.isclose(got["s1"], w["s1"], rtol=1e-13, atol=0)
                    vgx.vegas_set_grid(ref, vgx.vegas_get_grid(v, DIM, NB))  # the batch sums in another order
                    want.append(got)
                else:
                    vgx.vegas_refine(v)
                    vgx.vegas_refine(ref)
                    want.append(w)
                it += 1
            elif c == "R":
                vgx.vegas_reset_results(v)
                assert vgx.vegas_results(v) == [] and vgx.vegas_result(v)["n_used"] == 0
                want = []
            elif c == "g":
                vgx.vegas_set_grid(v, vgx.vegas_get_grid(v, DIM, NB))
            else:
                assert vgx.vegas_results(v) == want
            if c != "a":
                assert vgx.vegas_result(v)["n_used"] == len(want)
        assert vgx.vegas_results(v) == want
        r = vgx.vegas_result(v)
        if want:
            inv = sum(1 / k["var"] for k in want)
            assert np.isclose(r["mean"], sum(k["mean"] / k["var"] for k in want) / inv, rtol=1e-13, atol=0)
            assert np.isclose(r["sigma"], inv ** -0.5, rtol=1e-13, atol=0)
        assert np.array_equal(vgx.vegas_get_grid(v, DIM, NB), vgx.vegas_get_grid(ref, DIM, NB))
    finally:
        if b is not None:
            vgx.batch_destroy(b)
        vgx.vegas_destroy(v)
        vgx.vegas_destroy(ref)
