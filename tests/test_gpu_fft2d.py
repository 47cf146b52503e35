"""The Fourier path's own transforms (rows, columns with the filter, rows)
against the FP64 CPU oracle, at the edges of their lengths: the smallest, every
last step (2, 4, 8 points), powers of two on both sides of the two column
kernels, chirps that fill their points, odd numbers of rows, and the longest.

White noise in every field, so every mode counts; 1e-12 as for the other
tests of the path (a transform adds a few eps log2 n, a chirp twice that)."""
import numpy as np
import pytest

from oracle import coeffs as oc
from oracle import expm_modes as em
from oracle import lrsw
from oracle import rexii_modes as rm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [
    (16, 16), (17, 16), (16, 33), (32, 64), (31, 128), (256, 19), (512, 16), (16, 512), (513, 21), (23, 513),
    (1024, 17), (17, 1024), (1023, 18), (18, 1023), (2048, 19), (19, 2048), (2047, 16), (16, 2047), (1025, 22),
    (22, 1025), (4096, 16), (16, 4096),
])
def test_own_transforms_match_oracle(nx, ny):
    import torch
    from paper_2008_11607_amd import rexii
    rexii.load()
    op = lrsw.LRSW(nx, ny, fc=10.0)
    t = 40.3 / lrsw.rho(op)
    ref = oc.api_coeffs(t, lrsw.rho(op), h=0.5, tol=1e-10)
    f = np.random.default_rng(nx + 7 * ny).standard_normal((3, ny, nx))
    print(f"own transforms {nx}x{ny}", flush=True)
    fd = torch.from_numpy(f).cuda()
    u, rep = rexii.apply_fourier(fd, t, fc=10.0, tol=1e-10)
    assert torch.equal(fd.cpu(), torch.from_numpy(f))
    r = rm.rexii_spectral(op, f, t, ref["z"], ref["w"])
    assert em.rel_l2(u.cpu().numpy(), r) <= 1e-12
    # a single value that is not finite is reported wherever it lies
    for at in ((0, 0, 0), (2, ny - 1, nx - 1), (1, ny // 2, nx // 2)):
        bad = fd.clone()
        bad[at] = float("inf")
        with pytest.raises(rexii.RexiiError) as e:
            rexii.apply_fourier(bad, t, fc=10.0)
        assert e.value.status == -2
