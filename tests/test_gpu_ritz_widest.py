"""The widest bases the Ritz step takes (512 columns): their index arrays, reflector and p need the
most LDS of any launch of the wide kernel.

Reference: numpy in FP64 with the bound of the sizes below it, 64 q u cond(G) max|theta|."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q", [505, 511, 512])
def test_widest(q):
    from paper_2304_00337_amd.api import Solver
    rng = np.random.default_rng(q)
    z = rng.standard_normal((3 * q, q)) + 1j * rng.standard_normal((3 * q, q))
    g = z.conj().T @ z
    lam = np.sort(rng.uniform(1.0, 50.0, q))
    c = np.linalg.cholesky(g)
    v, _ = np.linalg.qr(rng.standard_normal((q, q)) + 1j * rng.standard_normal((q, q)))
    h = c @ (v * lam) @ v.conj().T @ c.conj().T
    h = 0.5 * (h + h.conj().T)
    with Solver(8, 8, 1.0, 1.0, np.ones(64), nev=2, nthrow=1, autotune=0) as s:
        th, y = s.ritz_small(g, h, 40)
    tol = 64 * q * 2.0 ** -53 * np.linalg.cond(g)
    assert len(th) == 40
    assert np.abs(th - lam[:40]).max() <= tol * 50.0
    assert np.abs(y.conj().T @ g @ y - np.eye(40)).max() <= tol
    assert np.abs(y.conj().T @ h @ y - np.diag(th)).max() <= tol * 50.0
