"""Workspace of the shared-Krylov path: the small problem's share is bounded
for any time step (host code, no GPU)."""
import ctypes

import pytest


@pytest.mark.parametrize("h", [0.1, 0.5, 1.5])
@pytest.mark.parametrize("nx,ny,nrhs", [(16, 16, 1), (64, 48, 3)])
@pytest.mark.parametrize("t", [1e-3, 1.0, 100.0, 2e3, 1e5, 1e9, 1e15, 1e300])
def test_basis_size_is_bounded(nx, ny, nrhs, t, h):
    from paper_2008_11607_amd import rexii as rx
    lib = rx.load()
    op, o, lo, hi = rx.make_op(nx, ny), rx.make_opts(h=h), ctypes.c_size_t(), ctypes.c_size_t()
    assert lib.rexii_multishift_workspace_size(ctypes.byref(op), nrhs, ctypes.byref(o), ctypes.byref(lo)) == 0
    assert lib.rexii_multishift_basis_size(ctypes.byref(op), nrhs, t, ctypes.byref(o), ctypes.byref(hi)) == 0
    # the least, at most 50000 vectors, 2 GiB of recurrences and 4.2M poles of 48 bytes, mailboxes
    vectors = 50000 * nrhs * 3 * nx * ny * 8
    assert lo.value < hi.value <= lo.value + vectors + (2 << 30) + (1 << 28) + (64 << 20)
