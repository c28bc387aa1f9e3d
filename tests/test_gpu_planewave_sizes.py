"""The projection's plane-wave component where its reductions change form: one workgroup (32 x 32) and
two for the dot product, 256 partials of the right-hand side (512 x 512: summed by the kernel that uses
them) and more (a launch of their own).

The component is solved exactly, so w^* L^* M (projected block) vanishes up to rounding: the block's
entries carry a few u of their size (u = 2^-53) and L^* M sums twelve of them per node, which is at most
256 u times the sum of the moduli of L^* M of the given block."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m", [(32, 32), (36, 32), (512, 512), (512, 576)])
def test_plane_wave_component_is_removed(n, m):
    import torch

    from paper_2304_00337_amd.api import Solver, from_device_block, to_device_block
    k = (0.9, -0.7)
    u = np.random.default_rng(n + m).standard_normal((2 * n * m, 3, 2)) @ [1, 1j]
    with Solver(n, m, 1.0, 0.8, np.full(n * m, 2.0), nev=1, nthrow=0, mu=5.0, autotune=0, precision="fp64") as s:
        s.set_k(*k)
        x = to_device_block(u)
        b0 = torch.empty((3, 2, n * m), dtype=torch.float64, device="cuda")
        b1 = torch.empty_like(b0)
        s.apply("LHM", x, out=b0)
        s.apply("LHM", s.apply("PROJECT", x, out=torch.empty_like(x)), out=b1)
        b0, b1 = from_device_block(b0), from_device_block(b1)
    j = np.arange(n * m)
    w = np.exp(1j * (k[0] * 1.0 / n * (j % n) + k[1] * 0.8 / m * (j // n)))
    assert np.all(np.abs(w.conj() @ b1) <= 256 * 2.0 ** -53 * np.abs(b0).sum(axis=0))
