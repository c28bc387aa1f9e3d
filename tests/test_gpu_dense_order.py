"""FP32 nodal direct solves add their terms one after the other, the real and imaginary part of a term each
as a r b r + a i b i rounded per operation: bit for bit what numpy gives in float32.  Sizes around the groups of eight
terms that the kernel loads ahead, and of the 64 rows of a wave.

The inverse's entries come from the solve itself: on a unit vector it returns a column, exactly."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m", [(2, 2), (2, 4), (3, 3), (5, 3), (4, 4), (17, 2), (5, 5), (7, 7), (8, 8), (13, 5), (15, 15)])
def test_terms_in_order(n, m):
    import torch

    from paper_2304_00337_amd.api import Solver
    rng = np.random.default_rng(100 * n + m)
    nn = n * m
    with Solver(n, m, 1.0, 0.8, rng.uniform(1.0, 9.0, nn), nev=1, nthrow=0, levels=1, mu=5.0, autotune=0) as s:
        s.set_k(0.9, 0.4)
        eye = torch.zeros((nn, 2, nn), dtype=torch.float32, device="cuda")
        eye[torch.arange(nn), 0, torch.arange(nn)] = 1.0
        inv = s.apply("COARSE_NODAL", eye, out=torch.empty_like(eye)).cpu().numpy()   # [l, :, i]: entry (i, l)
        b = rng.standard_normal((3, 2, nn)).astype(np.float32)
        x = torch.from_numpy(b).cuda()
        got = s.apply("COARSE_NODAL", x, out=torch.empty_like(x)).cpu().numpy()
    ref = np.zeros_like(b)
    for l in range(nn):   # (i, l) is the conjugate of (l, i), whose parts are ar and ai
        ar, ai = inv[l, 0], -inv[l, 1]
        for c in range(3):
            br, bi = b[c, 0, l], b[c, 1, l]
            ref[c, 0] += ar * br + ai * bi
            ref[c, 1] += ar * bi + -ai * br
    assert np.array_equal(got, ref)
