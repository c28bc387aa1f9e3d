"""The coarsest level's direct solvers where the block steps of their inversion can go wrong:
matrices smaller than one block of 32 unknowns, exactly one, one more than a multiple, and
sizes whose edge and nodal matrices take different step counts.

Reference: the level's own operators probed with unit vectors and solved in FP64 by numpy.  An
inverse applied to b carries an error of about u cond(K) |x| per elimination step growth; the
bound used is 8 n u cond(K) (n unknowns, u = 2^-53), relative to the column's largest entry."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,k", [(2, 2, (0.9, 0.4)), (4, 4, (0.9, 0.4)), (3, 11, (0.3, -1.1)), (8, 8, (0.0, 0.0)),
                                   (5, 13, (2.0, 1.0)), (9, 15, (0.7, 0.2)), (15, 15, (1.3, 0.0))])
def test_coarse_solvers_at_block_edges(n, m, k):
    import torch

    from paper_2304_00337_amd.api import Solver, from_device_block, to_device_block
    rng = np.random.default_rng(n * 100 + m)
    eps = rng.uniform(1.0, 9.0, n * m)
    with Solver(n, m, 1.0, 0.8, eps, nev=1, nthrow=0, levels=1, mu=5.0, autotune=0) as s:
        s.set_k(*k)
        for op, solve, size in (("K", "COARSE_EDGE", 2 * n * m), ("P", "COARSE_NODAL", n * m)):
            eye = to_device_block(np.eye(size, dtype=complex))
            mat = from_device_block(s.apply(op, eye, out=torch.empty_like(eye)))
            if op == "P" and k == (0.0, 0.0):   # constants: the kernel, lifted by the diagonal's size
                mat = mat + np.real(mat[0, 0]) / size
            b = rng.standard_normal((size, 3)) + 1j * rng.standard_normal((size, 3))
            x = to_device_block(b)
            got = from_device_block(s.apply(solve, x, out=torch.empty_like(x)))
            ref = np.linalg.solve(mat, b)
            tol = 8 * size * 2.0 ** -53 * np.linalg.cond(mat)
            err = np.abs(got - ref).max(axis=0) / np.abs(ref).max(axis=0)
            assert err.max() <= tol, (op, err.max(), tol)
