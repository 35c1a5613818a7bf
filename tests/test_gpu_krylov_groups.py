"""The dot products and projections of long and middle vectors over every way the basis divides into groups.

The residual estimate of FGMRES and GCR is built from dot products and norms alone; the true residual is recomputed
from b - A x at the end.  A vector that a group loses, takes twice or sums partly changes the estimate by O(1);
rounding separates the two by about eps times the condition of the projected basis, far below the 1e-4 asked for.
One Uzawa step an iteration keeps the residual where the estimate has digits.  GCR's goes up to nine vectors only:
it takes |w|^2 - |h|^2 down to 1e-6 |w|^2 for the norm of a projected vector, which leaves 1e-10 in each step's part
of |r|^2 and 1e-4 of |r| while that is above 3e-3.
"""
import numpy as np
import pytest
import torch

import paper_2603_14040_amd as tph
import workloads as wl

pytestmark = pytest.mark.gpu


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# 320: up to four vectors a workgroup; 640: up to eight; 1216: up to eight, more than eight entries a thread.
# iters vectors at the last step: one group of each size, two and three of equal and of different sizes.
@pytest.mark.parametrize("n", [320, 640, 1216])
@pytest.mark.parametrize("accel", ["fgmres", "gcr"])
def test_estimate_is_the_true_residual_for_every_basis_size(n, accel):
    pr = wl.sinker(n, eta_in=10.0)
    c = T(pr.eta_b), T(pr.eta_p), T(pr.rho_b)
    for iters in (1, 2, 3, 5, 6, 7, 8, 9) + ((11, 15, 17, 18) if accel == "fgmres" else ()):
        with tph.Solver(n, n, precision=tph.FP64, rtol=1e-13, max_iters=iters, restart=20, accel=accel, uzawa_steps=1) as s:
            s.set_coefficients(*c, pr.gx, pr.gy)
            *_, info = s.solve()
        print(f"[{accel} {n}] iters={info.iters} true={info.res_energy:.6e} estimate={info.res_estimate:.6e}", flush=True)
        assert info.iters == iters and (1e-7 if accel == "fgmres" else 3e-3) < info.res_energy < 1.0
        assert info.res_estimate == pytest.approx(info.res_energy, rel=1e-4)
