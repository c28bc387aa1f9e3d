"""The Ritz step's dense problem at the edges of its register kernels (thread grids of 16, 32, 48,
64, 96 and 112 columns; the wider kernel beyond) and in the forms that take branches of their own:
columns already reduced, dropped columns, repeated eigenvalues, a zero threshold, matrices scaled
far from one.

References: spectra known by construction or numpy in FP64.  The reduction is backward stable, so
a value is off by at most a small multiple of q u cond(G) max|theta| (u = 2^-53): the bound used is
64 q u cond(G) max|theta|; orthonormality and diagonality likewise, relative to one and max|theta|."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


@pytest.fixture(scope="module")
def solver():
    from paper_2304_00337_amd.api import Solver
    with Solver(8, 8, 1.0, 1.0, np.ones(64), nev=2, nthrow=1, autotune=0) as s:
        yield s


def _pencil(rng, q, lam):
    """G and H = G^{1/2} ... with the given spectrum, and cond(G)."""
    z = rng.standard_normal((3 * q + 4, q)) + 1j * rng.standard_normal((3 * q + 4, q))
    g = z.conj().T @ z
    c = np.linalg.cholesky(g)
    v, _ = np.linalg.qr(rng.standard_normal((q, q)) + 1j * rng.standard_normal((q, q)))
    h = c @ (v * lam) @ v.conj().T @ c.conj().T
    return g, 0.5 * (h + h.conj().T), np.linalg.cond(g)


def _check(th, y, g, h, lam, cond):
    q, top = len(g), np.abs(lam).max()
    tol = 64 * q * U * cond
    assert len(th) == y.shape[1]
    assert np.abs(th - lam[:len(th)]).max() <= tol * top
    assert np.abs(y.conj().T @ g @ y - np.eye(len(th))).max() <= tol
    assert np.abs(y.conj().T @ h @ y - np.diag(th)).max() <= tol * top


@pytest.mark.parametrize("q", [1, 2, 3, 4, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 95, 96, 97, 111, 112, 113])
def test_sizes(solver, q):
    rng = np.random.default_rng(q)
    lam = np.sort(np.concatenate([rng.uniform(0.5, 200.0, q - q // 3), 10.0 ** rng.uniform(2.5, 5.0, q // 3)]))
    g, h, cond = _pencil(rng, q, lam)
    for want in sorted({1, (q + 1) // 2, q}):
        th, y = solver.ritz_small(g, h, want)
        assert len(th) == want
        _check(th, y, g, h, lam, cond)


@pytest.mark.parametrize("q", [6, 30, 48, 64, 90, 108])
def test_forms(solver, q):
    rng = np.random.default_rng(1000 + q)
    want = (q + 1) // 2
    # diagonal pencils: every column is reduced already
    d = rng.uniform(0.5, 3.0, q)
    lam = np.sort(rng.uniform(1.0, 50.0, q))
    th, y = solver.ritz_small(np.diag(d).astype(complex), np.diag(d * lam).astype(complex), want)
    _check(th, y, np.diag(d), np.diag(d * lam), lam, d.max() / d.min())
    # repeated eigenvalues at both ends of the wanted range
    lam = np.sort(rng.uniform(1.0, 50.0, q))
    lam[:2] = lam[0]
    lam[max(2, want - 2):want + 1] = lam[max(2, want - 2)]
    lam = np.sort(lam)
    g, h, cond = _pencil(rng, q, lam)
    th, y = solver.ritz_small(g, h, want)
    _check(th, y, g, h, lam, cond)
    # values below the zero threshold are skipped (indefinite H)
    lam = np.sort(np.concatenate([rng.uniform(-5.0, 1e-3, 2), rng.uniform(1.0, 50.0, q - 2)]))
    g, h, cond = _pencil(rng, q, lam)
    th, y = solver.ritz_small(g, h, want, zero_thr=0.5)
    assert np.abs(th - lam[2:2 + len(th)]).max() <= 64 * q * U * cond * 50.0 and len(th) == min(want, q - 2)
    # H scaled far from one
    g, h, cond = _pencil(rng, q, lam)
    for s in (2.0 ** -460, 2.0 ** 460):
        th, y = solver.ritz_small(g, h * s, want)
        assert np.abs(th / s - lam[:want]).max() <= 64 * q * U * cond * 50.0
    # a copy of a column is dropped: the pencil of the others remains
    g, h, cond = _pencil(rng, q - 1, np.sort(rng.uniform(1.0, 50.0, q - 1)))
    e = np.insert(np.eye(q - 1), q // 2, np.eye(q - 1)[0] * 3.0, axis=1)
    th, y = solver.ritz_small(e.T @ g @ e, e.T @ h @ e, q)
    ref = np.linalg.eigvalsh(np.linalg.solve(c := np.linalg.cholesky(g), np.linalg.solve(c, h).conj().T))
    assert len(th) == q - 1
    assert np.abs(th - ref).max() <= 64 * q * U * cond * 50.0


def test_no_valid_direction(solver):
    """A zero or non-finite G spans nothing: no values, no hang."""
    for bad in (np.zeros((20, 20)), np.full((20, 20), np.nan), np.full((70, 70), np.inf)):
        th, _ = solver.ritz_small(bad.astype(complex), np.eye(len(bad), dtype=complex), 5)
        assert len(th) == 0
