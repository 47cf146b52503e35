"""A workspace sized for a time step holds the shorter ones too: the scratch of
the pole sums does not grow with t where boxes take the place of split sums."""
import pytest
import torch

from oracle import expm_modes as em
from oracle import lrsw
from paper_2008_11607_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,top", [(93, 2139, 400.0), (1875, 18, 8000.0), (2289, 51, 700.0), (67, 2166, 1400.0),
                                       (64, 64, 2000.0)])
def test_workspace_of_a_longer_step(nx, ny, top):
    from paper_2008_11607_amd import rexii
    rexii.load()
    op = lrsw.LRSW(nx, ny, fc=10.0)
    rho = lrsw.rho(op)
    fh = inputs.gaussian_bumps(nx, ny, nbumps=2, seed=3, velocity=True)
    f = torch.from_numpy(fh).cuda()
    sizes = [(tr, rexii.fourier_workspace_size(nx, ny, tr / rho)) for tr in [top * 1.25 ** -i for i in range(16)]]
    least = sizes[0][1]
    for tr, need in sizes:
        ws = torch.empty(least, dtype=torch.uint8, device="cuda")
        u, _ = rexii.apply_fourier(f, tr / rho, workspace=ws)
        if need > least or tr == top:   # the rounding of theta: 1e-16 t rho, and of the transforms
            assert em.rel_l2(u.cpu().numpy(), em.expm_closed_real(op, fh, tr / rho)) <= 1e-10
    assert nx == 64 or max(s for _, s in sizes[1:]) > sizes[0][1]
