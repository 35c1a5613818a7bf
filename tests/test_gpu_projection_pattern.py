"""FGMRES's speculative second projection in each of its turns: launched behind the first after a step that needed one
and taken, launched and skipped on the device, and launched by the host after a step that needed none.

The steps that needed a second projection are read off the solver's count over solves of 1, 2, .. steps (a solve is
bitwise reproducible, so each repeats the shorter one's steps).  The estimate, built from the coefficients of both
projections, is the true residual within rounding (eps times the condition of the projected basis, far below 1e-4).
"""
import numpy as np
import pytest
import torch

import paper_2603_14040_amd as tph
import workloads as wl

pytestmark = pytest.mark.gpu


# 192: 73 blocks of 2048 entries, the projection adds up the dot products itself; 304, 352: more than 128 blocks
@pytest.mark.parametrize("n", [192, 304, 352])
def test_taken_skipped_and_late(n):
    pr = wl.sinker(n, eta_in=10.0)
    c = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (pr.eta_b, pr.eta_p, pr.rho_b)]
    needed, before = "", 0
    for steps in range(1, 11):
        with tph.Solver(n, n, precision=tph.MIXED, rtol=1e-13, max_iters=steps, restart=20, accel="fgmres",
                        uzawa_steps=1) as s:
            s.set_coefficients(*c, pr.gx, pr.gy)
            info = s.solve()[3]
            count = s.second_projections
        needed += str(count - before)
        before = count
        assert info.iters == steps and 1e-7 < info.res_energy < 1.0
        assert info.res_estimate == pytest.approx(info.res_energy, rel=1e-4)
    print(f"[pattern {n}] {needed}", flush=True)
    assert set(needed) == {"0", "1"}
    assert "11" in needed and "10" in needed and "01" in needed
