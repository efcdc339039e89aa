"""RAMBO at the edges of its arithmetic: every kind of mass list (massless
particles among massive ones, sums close to the threshold) and tiny and huge
energies, against the oracle with the bars of `tests/test_gpu_rambo.py`
(1e-9: events whose massless momenta are nearly aligned are boosted by a large
factor, whatever the arithmetic)."""
import numpy as np
import pytest

from oracle import rambo as orb
from tests.test_gpu_rambo import run_gpu

pytestmark = pytest.mark.gpu

CASES = [([0.0] * n, 91.2) for n in (2, 5, 10)] + [
    ([173.0, 0.0], 1500.0), ([0.0, 4.7, 0.0, 0.0, 173.0], 1500.0), ([10.0] * 9 + [0.0], 101.0),
    ([80.4, 80.4, 91.2], 1e7), ([1e-9, 0.0, 0.0], 10.0), ([1e-60, 2e-60, 0.0], 1e-58)]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_matches_oracle(vgx, case):
    masses, rs = CASES[case]
    n = 2003
    print(f"rambo masses={masses} sqrt_s={rs}", flush=True)
    k, w = run_gpu(vgx, masses, rs, 17 + case, 2, 1, 5, n)
    kr, wr = orb.generate(17 + case, 2, 1, 5, n, masses, rs)
    assert np.max(np.abs(k - kr)) <= 1e-9 * rs
    assert np.allclose(w, wr, rtol=1e-9, atol=0)
