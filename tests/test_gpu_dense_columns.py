"""Direct solves of several columns: a workgroup takes one, two or four of them by the matrix's size and
the column count, and a column's result is the one it has alone, bit for bit.  Sizes on both sides of
that rule, with column counts that leave a remainder."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,cols,dtype", [(2, 2, 5, "float64"), (8, 8, 33, "float64"), (16, 16, 35, "float64"),
                                            (30, 30, 3, "float64"), (30, 30, 19, "float64"), (30, 30, 35, "float64"),
                                            (30, 30, 34, "float32"), (31, 33, 33, "float32"), (18, 20, 47, "float32")])
def test_columns_as_alone(n, m, cols, dtype):
    import torch

    from paper_2304_00337_amd.api import Solver
    rng = np.random.default_rng(n * 100 + cols)
    with Solver(n, m, 1.0, 0.8, rng.uniform(1.0, 9.0, n * m), nev=1, nthrow=0, levels=1, mu=5.0, autotune=0) as s:
        s.set_k(0.9, 0.4)
        for op, size in (("COARSE_EDGE", 2 * n * m), ("COARSE_NODAL", n * m)):
            x = torch.from_numpy(rng.standard_normal((cols, 2, size))).to(getattr(torch, dtype)).cuda()
            got = s.apply(op, x, out=torch.zeros_like(x))
            for c in {0, 1, cols // 2, cols - 2, cols - 1}:
                one = x[c:c + 1].clone()
                assert torch.equal(s.apply(op, one, out=torch.zeros_like(one))[0], got[c]), (op, c)


def test_columns_of_several_slots():
    """Problems of one engine, whose launches carry several slots' columns of a wide coarsest matrix,
    against each problem alone."""
    import synth

    from paper_2304_00337_amd.api import Batch, Solver, to_device_block
    n, nev, nthrow = 62, 9, 4   # coarsest level 31 x 31, 13 columns a slot
    rng = np.random.default_rng(3)
    probs = []
    for i in range(3):
        probs.append(dict(n=n, m=n, a=1.0, b=1.0, eps=rng.uniform(1.0, 9.0, n * n), nev=nev, nthrow=nthrow,
                          ks=np.array([[0.9, 0.4 + 0.3 * i]]),
                          start=to_device_block(synth.start_block(2 * n * n, nev + nthrow, i))))
    with Batch(precision="fp64", tol=1e-8, max_iter=300) as batch:
        res = batch.run(probs)
    for p, r in zip(probs, res):
        with Solver(n, n, 1.0, 1.0, p["eps"], nev=nev, nthrow=nthrow, tol=1e-8, max_iter=300) as s:
            alone = s.solve_k(*p["ks"][0], start=p["start"])
        assert alone["converged"] and np.array_equal(np.ravel(r["evals"]), alone["evals"])
