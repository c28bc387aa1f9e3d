"""The tiled sweeps where their split can go wrong: grids smaller than a tile's halo, exactly a tile,
one block more, ragged in either direction, several periods to a box, one and two sweeps a level
(from zero and not, with and without the folded transfers), and columns that do not start on a pair
of values.

Reference: the colours launched one by one (tested against the operators); the same operations in the
same order, so the results are equal."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = [(4, 4), (6, 10), (32, 32), (34, 30), (40, 66), (96, 64), (8, 100)]


def _rand(rows, cols):
    return np.random.default_rng(rows).standard_normal((rows, cols, 2)) @ [1, 1j]


@pytest.mark.parametrize("n,m", SIZES)
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_sweeps_equal_colour_passes(n, m, precision):
    import torch

    from paper_2304_00337_amd.api import Solver, from_device_block, to_device_block
    eps = np.random.default_rng(n * 100 + m).uniform(1.0, 9.0, n * m)
    dt = torch.float32 if precision == "mixed" else torch.float64
    for nu in (1, 2):
        out = []
        for tiled in (0, 1, 2):
            with Solver(n, m, 1.0, 0.8, eps, nev=1, nthrow=0, levels=0, coarsest_min=2, mu=5.0, autotune=0,
                        precision=precision, coarse_fuse=0, tiled_sweeps=tiled, nu_pre=nu, nu_post=nu) as s:
                s.set_k(0.9, -0.7)
                res = []
                for op, size, t in (("EDGE_VCYCLE", 2 * n * m, dt), ("NODAL_VCYCLE", n * m, dt),
                                    ("PROJECT", 2 * n * m, torch.float64)):
                    x = to_device_block(_rand(size, 3), dtype=t)
                    res.append(from_device_block(s.apply(op, x, out=torch.empty_like(x))))
                out.append(res)
        for got in out[1:]:
            for a, b in zip(out[0], got):
                assert np.isfinite(a).all() and np.array_equal(a, b)


@pytest.mark.parametrize("op,comps", [("NODAL_SWEEP", 1), ("NODAL_SWEEP_BACK", 1), ("EDGE_SWEEP", 2), ("EDGE_SWEEP_BACK", 2)])
@pytest.mark.parametrize("fp32", [False, True])
def test_sweeps_of_columns_off_a_pair(op, comps, fp32):
    import torch

    from paper_2304_00337_amd.api import Solver, to_device_block
    n, m = 34, 30
    eps = np.random.default_rng(7).uniform(1.0, 9.0, n * m)
    dt = torch.float32 if fp32 else torch.float64

    def shifted(x, by):   # the same block, `by` values past an allocation's start
        buf = torch.empty(x.numel() + by, dtype=x.dtype, device=x.device)
        v = buf[by:].view(x.shape)
        v.copy_(x)
        return v

    with Solver(n, m, 1.0, 0.8, eps, nev=1, nthrow=0, levels=0, coarsest_min=2, mu=5.0, autotune=0,
                precision="mixed" if fp32 else "fp64") as s:
        s.set_k(0.9, -0.7)
        x = to_device_block(_rand(comps * n * m, 3), dtype=dt)
        y = to_device_block(_rand(comps * n * m, 4)[:, 1:], dtype=dt)
        ref = s.apply(op, x, y=y, out=torch.empty_like(x))
        for bx, by in ((1, 0), (0, 1), (1, 1)):
            got = s.apply(op, shifted(x, bx), y=shifted(y, by), out=shifted(x, bx))
            assert torch.equal(got, ref)
