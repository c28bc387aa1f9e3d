"""The Ritz step's zero threshold far outside the spectrum, on the register kernel and the wider one:
the number of values above it is known exactly (none, or all of them), however far the scaled
threshold lies from the scaled matrix."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q", [1, 2, 9, 17, 48, 64, 90, 112, 120])
def test_threshold_far_outside_the_spectrum(q):
    from paper_2304_00337_amd.api import Solver
    rng = np.random.default_rng(q)
    z = rng.standard_normal((3 * q, q)) + 1j * rng.standard_normal((3 * q, q))
    g = z.conj().T @ z
    w = rng.standard_normal((3 * q, q)) + 1j * rng.standard_normal((3 * q, q))
    h = w.conj().T @ w   # positive definite: every value lies above zero and below 2^20
    with Solver(8, 8, 1.0, 1.0, np.ones(64), nev=2, nthrow=1, autotune=0) as s:
        ref = s.ritz_small(g, h, q)[0]
        assert len(ref) == q
        for scale, thr, found in ((2.0 ** -460, 0.5, 0), (2.0 ** -900, 0.5, 0), (1.0, 1e300, 0), (1.0, 2.0 ** 200, 0),
                                  (2.0 ** -460, -0.5, q), (2.0 ** -900, -0.5, q), (1.0, 2.0 ** 21, 0)):
            th, _ = s.ritz_small(g, h * scale, q, zero_thr=thr)
            assert len(th) == found, (scale, thr, len(th))
