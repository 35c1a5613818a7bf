"""FGMRES's two projections over the ways they are launched.

The projection adds up the dot products itself on grids of up to 128 blocks of 2048 entries (sizes on both
sides of 64 and 128), and after a step that needed a second projection the next one's is launched before the
host knows.  The estimate is built from the coefficients of both; it is the true residual of the solution only
if every coefficient and every skipped or repeated pass is right (a wrong one changes it by O(1); rounding
separates them by about eps times the condition of the projected basis, far below 1e-4).
"""
import numpy as np
import pytest
import torch

import paper_2603_14040_amd as tph
import workloads as wl

pytestmark = pytest.mark.gpu


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("n", [16, 48, 192, 208, 288, 304])
@pytest.mark.parametrize("contrast", [1.0, 1e3])
@pytest.mark.parametrize("iters", [2, 7, 16])
def test_estimate_with_second_projections(n, contrast, iters):
    pr = wl.sinker(n, eta_in=contrast)
    with tph.Solver(n, n, precision=tph.MIXED, rtol=1e-13, max_iters=iters, restart=20, accel="fgmres") as s:
        s.set_coefficients(T(pr.eta_b), T(pr.eta_p), T(pr.rho_b), pr.gx, pr.gy)
        a = s.solve()
        b = s.solve()
    print(f"[second {n}] contrast={contrast} true={a[3].res_energy:.6e} estimate={a[3].res_estimate:.6e}", flush=True)
    assert all(torch.equal(u, v) for u, v in zip(a[:3], b[:3]))
    assert 0 < a[3].iters <= iters and 0.0 < a[3].res_energy < 1.0     # an easy problem ends before, at the rounding floor
    if a[3].res_energy > 1e-7:
        assert a[3].res_estimate == pytest.approx(a[3].res_energy, rel=1e-4)
