"""Which calls run their inner steps on the chip (a launch takes a slot up to
256 steps further; the streamed passes launch 16 steps at a time) and that
their results meet the bars of the two precisions against the exact
exponential."""
import pytest
import torch

from oracle import expm_modes as em
from oracle import lrsw
from paper_2008_11607_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rx():
    from paper_2008_11607_amd import rexii
    rexii.load()
    return rexii


# few rows, few slots, few points: the mailboxes of the fastest shape do not
# fit into the slots' spare vectors, those of another do
@pytest.mark.parametrize("precision,nx,ny,trho", [
    ("fp64", 291, 11, 5.0), ("mixed", 289, 6, 5.0), ("mixed", 7, 8, 20.0), ("fp64", 144, 32, 20.0),
    ("mixed", 149, 75, 20.0), ("mixed", 133, 128, 2.0), ("fp64", 95, 37, 20.0), ("mixed", 173, 106, 5.0),
    ("fp64", 4, 5, 20.0)])
def test_short_grids_run_on_the_chip(rx, precision, nx, ny, trho):
    op = lrsw.LRSW(nx, ny, fc=10.0)
    fh, t = inputs.gaussian_bumps(nx, ny, nbumps=2, seed=nx + ny), trho / lrsw.rho(op)
    bar = 1e-10 if precision == "fp64" else 1e-6
    u, rep = rx.apply(torch.from_numpy(fh).cuda(), t, precision=precision, tol=bar, profile=1)
    assert rep["kernel_launches"] < 16 and rep["not_converged"] == 0
    assert em.rel_l2(u.cpu().numpy(), em.expm_closed_real(op, fh, t)) <= bar
