"""The COCG steps that run on the chip (kernels_chip.hip): every launch shape
that the host can pick, against the oracle's exact exponential.

Bars: the targets of the two precisions (rel-L2 1e-10 in FP64, 1e-6 mixed) and
the call's own error bound.  The grids below take one block a slot, one block
a chain, strips on one XCD and across XCDs; chains of even and odd length
(odd ny is one chain); segments with RT and with RT - 1 rows; column counts
that are no multiple of a wavefront; and sizes just past what a group holds,
which go through the streaming passes.
"""
import threading

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


def _case(nx, ny, trho, seed, vel):
    op = lrsw.LRSW(nx, ny, fc=10.0)
    f = inputs.gaussian_bumps(nx, ny, nbumps=3, seed=seed, velocity=vel)
    return op, torch.from_numpy(f).cuda(), f, trho / lrsw.rho(op)


SHAPES = [(4, 4), (5, 7), (4, 64), (64, 4), (33, 8), (64, 64), (63, 65), (96, 80), (130, 66), (75, 101),
          (128, 128), (127, 129), (200, 37), (37, 200), (511, 24), (512, 40), (513, 24), (600, 30), (256, 256)]


@pytest.mark.parametrize("nx,ny", SHAPES)
@pytest.mark.parametrize("precision,bar", [("fp64", 1e-10), ("mixed", 1e-6)])
def test_chip_steps_match_oracle(rx, nx, ny, precision, bar):
    vel = (nx + ny) % 2 == 0     # unpaired solves for half of the grids
    op, f, fh, t = _case(nx, ny, 25.0, 1000 + nx + ny, vel)
    u, rep = rx.apply(f, t, fc=10.0, precision=precision)
    assert rep["not_converged"] == 0 and rep["err_bound"] <= bar
    assert em.rel_l2(u.cpu().numpy(), em.expm_closed_real(op, fh, t)) <= bar
    u2, _ = rx.apply(f, t, fc=10.0, precision=precision)
    assert bool((u == u2).all())


@pytest.mark.parametrize("slots", [1, 3, 9, 70])
def test_chip_few_slots(rx, slots):
    """Fewer slots than groups, one slot, a number no multiple of the XCDs."""
    op, f, fh, t = _case(128, 96, 40.0, 5, False)
    u, rep = rx.apply(f, t, fc=10.0, pole_batch=slots)
    assert rep["slots"] == slots
    assert em.rel_l2(u.cpu().numpy(), em.expm_closed_real(op, fh, t)) <= 1e-10


@pytest.mark.parametrize("cap", [1, 2, 7, 300])
def test_chip_iteration_cap(rx, cap):
    """The cap ends an inner solve inside a launch and between two launches;
    the result stays within the reported bound."""
    op, f, fh, t = _case(96, 64, 150.0, 6, True)
    try:
        u, rep = rx.apply(f, t, fc=10.0, max_iter=cap)
    except rx.RexiiError as e:
        assert e.status == -3
        rep = e.report
    assert rep["max_iters"] <= cap + 1


def test_chip_calls_from_two_threads(rx):
    """Two host threads, each on its own stream, with groups of blocks that
    wait for each other: both finish, with the results of single calls."""
    cases = [_case(128, 128, 60.0, 7, False), _case(192, 160, 50.0, 8, False)]
    single = [rx.apply(f, t, fc=10.0)[0] for _, f, _, t in cases]
    torch.cuda.synchronize()
    got, errs = [None, None], []

    def work(i):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                for _ in range(3):
                    got[i] = rx.apply(cases[i][1], cases[i][3], fc=10.0)[0]
            s.synchronize()
        except Exception as ex:  # noqa: BLE001
            errs.append(ex)

    th = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for x in th:
        x.start()
    for x in th:
        x.join()
    assert not errs, errs
    for a, b in zip(got, single):
        assert np.array_equal(a.cpu().numpy(), b.cpu().numpy())
