"""Calls on several threads and streams whose groups of blocks each take a
whole XCD or the whole chip: they take turns, none waits for CUs that another
one holds."""
import threading
import time

import pytest
import torch

from paper_2008_11607_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kinds", [("mixed", "mixed"), ("mixed", "lanczos"), ("lanczos", "lanczos"),
                                   ("fp64", "mixed", "lanczos", "lanczos")])
def test_calls_share_the_chip(kinds):
    from paper_2008_11607_amd import rexii
    rexii.load()
    f = [torch.from_numpy(inputs.gaussian_bumps(512, 512, nbumps=2, seed=9 + i)).cuda() for i in range(len(kinds))]

    def call(kind, x):
        if kind == "lanczos":
            return rexii.apply_multishift(x, 0.3)[0]
        return rexii.apply(x, 0.02, precision=kind, tol=1e-6 if kind == "mixed" else 1e-10)[0]

    single = [call(k, x) for k, x in zip(kinds, f)]
    torch.cuda.synchronize()
    t0 = time.time()
    for k, x in zip(kinds, f):
        call(k, x)
    torch.cuda.synchronize()
    alone = time.time() - t0
    got, errs, rounds = [None] * len(kinds), [], 4

    def work(i):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                for _ in range(rounds):
                    got[i] = call(kinds[i], f[i])
            s.synchronize()
        except Exception as ex:  # noqa: BLE001
            errs.append(ex)

    th = [threading.Thread(target=work, args=(i,)) for i in range(len(kinds))]
    t0 = time.time()
    for x in th:
        x.start()
    for x in th:
        x.join()
    took = time.time() - t0
    assert not errs, errs
    for a, b in zip(got, single):
        assert bool((a == b).all())
    # one after the other, and hand-overs; a group that does not fill waits
    # for tens of milliseconds or more each time
    assert took <= 3.0 * rounds * alone + 0.5, (took, alone)
