"""A depth field formed on the caller's stream just before a shared-Krylov call
is read there, after the work that forms it."""
import numpy as np
import pytest
import torch

from paper_2008_11607_amd import inputs

pytestmark = pytest.mark.gpu


def test_depth_field_formed_on_a_side_stream():
    from paper_2008_11607_amd import rexii
    rexii.load()
    nx, ny = 96, 72
    Hd = torch.from_numpy(inputs.variable_depth(nx, ny)).cuda()
    f = torch.from_numpy(inputs.gaussian_bumps(nx, ny, nbumps=2, seed=5)).cuda()
    t = 40.0 / rexii.rho(nx, ny, Hfield=Hd)
    ref, _ = rexii.apply_multishift(f, t, Hfield=Hd)
    slow = torch.randn(4096, 4096, dtype=torch.float64, device="cuda")
    for _ in range(3):
        H = torch.full_like(Hd, float("nan"))
        torch.cuda.synchronize()
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for _ in range(4):            # milliseconds of work before the field is there
                slow2 = slow @ slow
            H.copy_(Hd)
            u, _ = rexii.apply_multishift(f, t, Hfield=H)
        s.synchronize()
        assert np.isfinite(float(slow2[0, 0]))
        assert bool((u == ref).all())
