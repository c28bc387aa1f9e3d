"""The Rayleigh-Ritz products at the edges of their one-launch kernel: column counts around every
multiple of its 16-column tiles (and of the waves' task plans), one past its widest (96 columns),
and meshes whose slices of 16 nodes are partly filled, odd, narrower than one slice, or two nodes
wide, with Bloch phases on both seams.

Reference: the oracle's sparse matrices in FP64.  Each entry is a sum over N edges or cells with
the rounding of a few operations per term, so its error is of order sqrt(N) u times the two
columns' norms (u = 2^-53); the bound used is 8 u sqrt(N) sqrt(G_ii G_jj) (H alike, with the norm
of A in place of M's: 8 / (h1 h2) max(kappa) |s|^2)."""
import numpy as np
import pytest

from oracle import fem

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


@pytest.mark.parametrize("n,m", [(16, 16), (17, 9), (33, 5), (15, 31), (2, 40), (48, 21)])
def test_products_at_tile_edges(n, m):
    from paper_2304_00337_amd import Solver, to_device_block
    rng = np.random.default_rng(100 * n + m)
    a, b, k = 1.0, 0.7, (0.9, -1.7)
    eps = rng.uniform(1.0, 12.0, n * m)
    d = fem.Discretization(n, m, a, b, eps, *k)
    top = 8.0 * (1.0 / eps).max() * n * m / (a * b)
    with Solver(n, m, a, b, eps, nev=33, nthrow=0, levels=1, mu=5.0, autotune=0) as s:
        s.set_k(*k)
        for q in (1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 79, 80, 81, 95, 96, 97):
            S = rng.standard_normal((d.n_edges, q)) + 1j * rng.standard_normal((d.n_edges, q))
            G, H = s.rr_products(to_device_block(S))
            norm = np.linalg.norm(S, axis=0)
            tol = 8 * U * np.sqrt(d.n_edges) * np.outer(norm, norm)
            mass = max(d.M.diagonal().real) * 1.5
            assert (np.abs(G - S.conj().T @ (d.M @ S)) <= tol * mass).all(), q
            assert (np.abs(H - S.conj().T @ (d.A @ S)) <= tol * top).all(), q
            if q <= 96:   # (the wider kernel forms both triangles of its diagonal tiles)
                assert np.array_equal(G, G.conj().T) and np.array_equal(H, H.conj().T), q
