"""Pole sums of the Fourier path by near and far terms (grids with many
distinct frequencies and many poles) against the FP64 CPU oracle.

Every mode carries energy, so each box of theta = t omega is met, the first
one (theta = 0 for f_c = 0) and the ends included.  Tolerance as for the
direct sums, 1e-12: theta^2 is rounded once (theta eps / 2 < 2e-13 of the
result for theta <= 1500) and the sums add a few eps kappa."""
import numpy as np
import pytest

from oracle import coeffs as oc
from oracle import expm_modes as em
from oracle import lrsw
from oracle import rexii_modes as rm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,trho,fc,h", [
    (301, 299, 1300.0, 10.0, 0.5),
    (299, 301, 1500.0, 0.0, 0.5),    # theta = 0
    (320, 321, 900.0, 10.0, 0.2),    # narrow strip: many near terms
    (401, 399, 1500.0, 900.0, 1.0),  # theta in the upper boxes only
    (640, 640, 1000.0, 20.0, 0.1),   # square, even: the unordered table
])
def test_boxed_pole_sums_match_oracle(nx, ny, trho, fc, h):
    import torch
    from paper_2008_11607_amd import rexii
    rexii.load()
    op = lrsw.LRSW(nx, ny, fc=fc)
    t = trho / lrsw.rho(op)
    f = np.random.default_rng(nx).standard_normal((3, ny, nx))
    print(f"boxed pole sums {nx}x{ny} trho={trho} h={h}", flush=True)
    u, rep = rexii.apply_fourier(torch.from_numpy(f).cuda(), t, fc=fc, h=h, tol=1e-10)
    # t rho / h is a whole number here: its rounding decides the last term of
    # the sum, so the poles are those of the M that was taken
    z, w = oc.poles_weights(rep["M"], h)
    assert rep["P"] == len(z)
    assert rep["total_iters"] * rep["solves"] > 4e7   # many sums: the boxes pay
    r = rm.rexii_spectral(op, f, t, z, w)
    assert em.rel_l2(u.cpu().numpy(), r) <= 1e-12
