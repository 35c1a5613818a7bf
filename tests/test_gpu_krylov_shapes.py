"""Krylov reductions over every way they split their vectors over workgroups.

FGMRES and GCR carry a residual estimate built from nothing but the dot
products and norms of their basis; the true residual is recomputed from b - A x
at the end.  The two agree only if every reduction is right, whatever number of
vectors shares a workgroup (1, 4 or 8, by the vectors' length) and however the
basis size divides by it.  Rounding separates them by about eps times the
condition of the projected basis, far below the 1e-4 asked for; a lost vector,
block or tail of a vector changes them by O(1).
"""
import numpy as np
import pytest
import torch

import paper_2603_14040_amd as tph
import workloads as wl

pytestmark = pytest.mark.gpu


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# 48: one vector per workgroup; 384: four; 640: eight (short, middle and long vectors)
@pytest.mark.parametrize("n", [48, 384, 640])
@pytest.mark.parametrize("accel", ["fgmres", "gcr"])
@pytest.mark.parametrize("iters", [1, 4, 8, 9, 17])
def test_estimate_is_the_true_residual(n, accel, iters):
    pr = wl.sinker(n, eta_in=10.0)
    with tph.Solver(n, n, precision=tph.FP64, rtol=1e-14, max_iters=iters, restart=20, accel=accel) as s:
        s.set_coefficients(T(pr.eta_b), T(pr.eta_p), T(pr.rho_b), pr.gx, pr.gy)
        *_, info = s.solve()
    print(f"[{accel} {n}] iters={info.iters} true={info.res_energy:.6e} estimate={info.res_estimate:.6e}", flush=True)
    assert info.iters == iters and 0.0 < info.res_energy < 1.0
    # at the end of the first cycle; below 1e-9 of the start GCR's recurrence has no digits left
    if info.res_energy > 1e-7:
        assert info.res_estimate == pytest.approx(info.res_energy, rel=1e-4)
