"""The fused coarse cycles at the shapes where their work split can go wrong: one and two lanes per
coarse node (36 x 32 and 60 x 36 have more nodes than the two-lane workgroups hold in FP64, in
FP32), a level of a single coarse node in one direction, odd coarsest levels, and dense solves of
less than one group of 64 rows and of more groups than LDS takes at a time.

Reference: the same cycle with every level launched by itself, whose kernels are tested against the
operators; both perform the same operations in the same order, so the results are equal."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,levels", [(36, 32, 0), (36, 32, 2), (60, 36, 0), (64, 32, 3), (8, 4, 2), (4, 20, 2)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_fused_cycles_equal_per_level_cycles(n, m, levels, precision):
    import torch

    from paper_2304_00337_amd.api import Solver, from_device_block, to_device_block
    rng = np.random.default_rng(n * 100 + m)
    eps = rng.uniform(1.0, 9.0, n * m)
    dt = torch.float32 if precision == "mixed" else torch.float64
    out = []
    for fuse in (0, 1):
        with Solver(n, m, 1.0, 0.8, eps, nev=1, nthrow=0, levels=levels, coarsest_min=2, mu=5.0, autotune=0,
                    precision=precision, coarse_fuse=fuse) as s:
            s.set_k(0.9, -0.7)
            if fuse:
                assert s.info()["fused_edge_level"] >= 0 and s.info()["fused_nodal_level"] >= 0
            res = []
            for op, size in (("EDGE_VCYCLE", 2 * n * m), ("NODAL_VCYCLE", n * m)):
                b = np.random.default_rng(size).standard_normal((size, 3, 2)) @ [1, 1j]
                x = to_device_block(b, dtype=dt)
                res.append(from_device_block(s.apply(op, x, out=torch.empty_like(x))))
            out.append(res)
    for ref, got in zip(*out):
        assert np.isfinite(ref).all() and np.abs(ref).max() > 0
        assert np.array_equal(got, ref)


@pytest.mark.parametrize("n,m", [(20, 12), (32, 32), (4, 4)])
@pytest.mark.parametrize("cycles", [1, 2, 3])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_fused_nodal_solve_equals_cycles_one_by_one(n, m, cycles, precision):
    import torch

    from paper_2304_00337_amd.api import Solver, from_device_block, to_device_block
    eps = np.random.default_rng(n).uniform(1.0, 9.0, n * m)
    b = np.random.default_rng(m).standard_normal((2 * n * m, 3, 2)) @ [1, 1j]
    out = []
    for fuse in (0, 1):
        with Solver(n, m, 1.0, 0.8, eps, nev=1, nthrow=0, coarsest_min=2, mu=5.0, autotune=0, precision=precision,
                    coarse_fuse=fuse, nodal_cycles=cycles) as s:
            s.set_k(0.9, -0.7)
            assert s.info()["fused_nodal_level"] == (0 if fuse else -1)
            x = to_device_block(b)
            out.append(from_device_block(s.apply("PROJECT", x, out=torch.empty_like(x))))
    assert np.isfinite(out[0]).all() and np.array_equal(out[0], out[1])
