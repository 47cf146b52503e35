"""The small problem of the shared-Krylov path in several launches (its scratch
is bounded: 64 pairs of poles take 16 bytes a row and pair)."""
import ctypes

import pytest
import torch

from paper_2008_11607_amd import inputs

pytestmark = pytest.mark.gpu


def test_small_problem_in_several_launches():
    """t rho 12000: about 16000 rows and 24000 pairs, 6 GiB at once.  Against the
    least workspace, where the host solves it: the same recurrences, 1e-16 a
    row and 1.6e4 rows, and as much again from the poles' phases: 1e-11."""
    from paper_2008_11607_amd import rexii as rx
    lib = rx.load()
    nx = ny = 64
    f = torch.from_numpy(inputs.gaussian_bumps(nx, ny, nbumps=3, seed=4)).cuda()
    t = 12000.0 / rx.rho(nx, ny)
    op, o, nb = rx.make_op(nx, ny), rx.make_opts(), ctypes.c_size_t()
    assert lib.rexii_multishift_workspace_size(ctypes.byref(op), 1, ctypes.byref(o), ctypes.byref(nb)) == 0
    ws, u, rep = torch.empty(nb.value, dtype=torch.uint8, device="cuda"), torch.empty_like(f), rx.Report()
    assert lib.rexii_apply_multishift(ctypes.byref(op), 1, ctypes.c_void_p(f.data_ptr()), ctypes.c_void_p(u.data_ptr()),
                                      float(t), ctypes.byref(o), ctypes.c_void_p(ws.data_ptr()), nb.value, rx._stream(),
                                      ctypes.byref(rep)) == 0
    v, r2 = rx.apply_multishift(f, t)
    assert r2["solves"] == rep.solves > 5000
    assert float((u - v).norm() / u.norm()) <= 1e-11


def test_no_room_for_the_vectors():
    """Where PyTorch's allocator has no room for the kept vectors (4 GB here,
    2 GB allowed) the call runs in the least workspace."""
    from paper_2008_11607_amd import rexii as rx
    nx = ny = 512
    f = torch.from_numpy(inputs.gaussian_bumps(nx, ny, nbumps=3, seed=4)).cuda()
    t = 400.0 / rx.rho(nx, ny)
    u, _ = rx.apply_multishift(f, t)
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (2 << 30)) / total)
    try:
        v, _ = rx.apply_multishift(f, t)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert float((u - v).norm() / u.norm()) <= 1e-12   # a few hundred terms of 1e-16


@pytest.mark.parametrize("trho", [4e9, 1e12, 1e200])
def test_time_step_past_every_integer(trho):
    """The step at which a check falls due is past an int: the cap on m ends
    pass 1, and the pole count is refused as by the other entry points."""
    from paper_2008_11607_amd import rexii as rx
    f = torch.from_numpy(inputs.gaussian_bumps(32, 24, nbumps=3, seed=4)).cuda()
    with pytest.raises(rx.RexiiError) as e:
        rx.apply_multishift(f, trho / rx.rho(32, 24), max_iter=96)
    assert e.value.status == -1 and "too large" in str(e.value)


def test_no_step_reads_no_depth():
    from paper_2008_11607_amd import rexii as rx
    f = torch.from_numpy(inputs.gaussian_bumps(32, 24, nbumps=3, seed=4)).cuda()
    H = torch.full((24, 32), float("nan"), dtype=torch.float64, device="cuda")
    u, _ = rx.apply_multishift(f, 0.0, Hfield=H)
    assert bool((u == f).all())
