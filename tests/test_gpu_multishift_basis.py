"""Shared-Krylov calls with every size of workspace: the least (each step runs
twice, the small problem on the host), room for the small problem and some
vectors (their sum, then repeated steps), and the full size (a sum only).  All
repeat the same recurrence, so results agree to the rounding of the final sum
and of the small problem (1e-12 allowed against 1e-16 per term and at most a
few hundred terms)."""
import ctypes

import numpy as np
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


def _call(rx, f, t, fc, H, nbytes, **opts):
    lib = rx.load()
    nrhs, ny, nx = f.shape[0], f.shape[2], f.shape[3]
    op, o, rep = rx.make_op(nx, ny, fc=fc, Hfield=H), rx.make_opts(**opts), rx.Report()
    u = torch.full_like(f, float("nan"))
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None
    st = lib.rexii_apply_multishift(ctypes.byref(op), nrhs, ctypes.c_void_p(f.data_ptr()), ctypes.c_void_p(u.data_ptr()),
                                    float(t), ctypes.byref(o), ctypes.c_void_p(ws.data_ptr()) if nbytes else None,
                                    nbytes, rx._stream(), ctypes.byref(rep))
    assert st == 0, rx.last_error()
    torch.cuda.synchronize()
    return u, rep.as_dict()


def _sizes(rx, nx, ny, nrhs, t, fc, H, **opts):
    lib = rx.load()
    op, o = rx.make_op(nx, ny, fc=fc, Hfield=H), rx.make_opts(**opts)
    lo, hi = ctypes.c_size_t(), ctypes.c_size_t()
    assert lib.rexii_multishift_workspace_size(ctypes.byref(op), nrhs, ctypes.byref(o), ctypes.byref(lo)) == 0
    assert lib.rexii_multishift_basis_size(ctypes.byref(op), nrhs, float(t), ctypes.byref(o), ctypes.byref(hi)) == 0
    return lo.value, hi.value


@pytest.mark.parametrize("nx,ny,nrhs,depth", [(64, 64, 1, False), (33, 21, 2, True), (130, 66, 3, False),
                                              (5, 4, 1, False), (96, 72, 2, True), (256, 192, 1, True)])
def test_workspace_sizes_agree(rx, nx, ny, nrhs, depth):
    fc = 10.0
    H = torch.from_numpy(inputs.variable_depth(nx, ny)).cuda() if depth else None
    fh = [inputs.gaussian_bumps(nx, ny, nbumps=3, seed=60 + r, velocity=r % 2 == 0) for r in range(nrhs)]
    f = torch.from_numpy(np.stack(fh)).cuda()
    t = 60.0 / rx.rho(nx, ny, fc=fc, Hfield=H)
    lo, hi = _sizes(rx, nx, ny, nrhs, t, fc, H)
    ref, r0 = _call(rx, f, t, fc, H, 0)
    vec = nrhs * 3 * nx * ny * 8
    scratch = hi - lo   # about: small-problem scratch and vectors
    for nb in (lo, lo + scratch // 2 // 256 * 256, hi - 40 * vec if hi - 40 * vec > lo else lo + 256, hi, hi + 10 * vec):
        u, rep = _call(rx, f, t, fc, H, nb)
        assert rep["solves"] == r0["solves"]
        err = float((u - ref).norm() / ref.norm())
        assert err <= 1e-12, (nb, err)
    if not depth:
        op = lrsw.LRSW(nx, ny, fc=fc)
        for r in range(nrhs):
            assert em.rel_l2(u[r].cpu().numpy(), em.expm_closed_real(op, fh[r], t)) <= 1e-10


def test_zero_state_and_cap(rx):
    """A zero state stays zero beside a live one; a cap below the dimension
    needed is reported and u is written from it."""
    f = torch.zeros(2, 3, 40, 48, dtype=torch.float64, device="cuda")
    f[1] = torch.from_numpy(inputs.gaussian_bumps(48, 40, nbumps=2, seed=3)).cuda()
    t = 50.0 / rx.rho(48, 40, fc=10.0)
    u, _ = rx.apply_multishift(f, t, fc=10.0)
    assert float(u[0].abs().max()) == 0.0 and float(u[1].abs().max()) > 0.0
    with pytest.raises(rx.RexiiError) as e:
        rx.apply_multishift(f[1].clone(), t, fc=10.0, max_iter=20)
    assert e.value.status == -3


@pytest.mark.parametrize("nx,ny,nrhs,depth", [(4, 4, 1, False), (7, 5, 3, True), (512, 6, 1, True), (511, 33, 2, False),
                                              (65, 63, 9, True), (128, 128, 1, False), (200, 300, 17, False),
                                              (513, 40, 1, True), (512, 512, 1, True)])
def test_steps_on_the_chip_match_launched_steps(rx, nx, ny, nrhs, depth):
    """One block a state, one XCD a state, blocks across XCDs, more states than
    fit at once, a row past the widest block: against the least workspace,
    whose steps are one launch each.  Both are the same recurrence in FP64."""
    fc = 10.0
    H = torch.from_numpy(inputs.variable_depth(nx, ny)).cuda() if depth else None
    f = torch.stack([torch.from_numpy(inputs.gaussian_bumps(nx, ny, nbumps=2, seed=80 + r, velocity=True))
                     for r in range(nrhs)]).cuda()
    t = 30.0 / rx.rho(nx, ny, fc=fc, Hfield=H)
    lo, hi = _sizes(rx, nx, ny, nrhs, t, fc, H)
    a, ra = _call(rx, f, t, fc, H, lo)
    b, rb = _call(rx, f, t, fc, H, hi)
    assert ra["solves"] == rb["solves"]
    assert float((a - b).norm() / a.norm()) <= 1e-12
    c, _ = _call(rx, f, t, fc, H, hi)
    assert bool((b == c).all())
