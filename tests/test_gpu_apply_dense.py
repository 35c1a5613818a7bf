"""tph_apply between the caller's arrays: block edges, walls, garbage, overlap.

The oracle's assembled operator times the state, row by row, for sides below, at
and above the 64 x 4 block and its ring; entries outside the unknowns are NaN on
input (ignored) and zero on output.  Each row is a sum of at most 15 products
of eps-accurate factors, so it is exact to 32 eps of its absolute terms, which
1e-13 of the largest row bounds for viscosities within two decades.
"""
import numpy as np
import pytest
import torch

import paper_2603_14040_amd as tph
import workloads as wl
from oracle import stokes as st

pytestmark = pytest.mark.gpu


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def state(nx, ny):
    vx, vy, p = wl.random_state(nx, ny, 5)
    keep = np.zeros((3, ny + 2, nx + 2), bool)
    keep[0, 1:ny + 1, 1:nx] = keep[1, 1:ny, 1:nx + 1] = keep[2, 1:ny + 1, 1:nx + 1] = True
    return [np.where(k, v, np.nan) for k, v in zip(keep, (vx, vy, p))], keep


@pytest.mark.parametrize("nx,ny", [(2, 2), (3, 2), (5, 7), (62, 3), (63, 4), (64, 5), (65, 6), (126, 2), (130, 9)])
@pytest.mark.parametrize("bc", [(0, 0, 0, 0), (1, 0, 1, 1)])
def test_apply_matches_the_assembled_operator(nx, ny, bc):
    eb, ep, rb = wl.random_fields(nx, ny, 3)
    x, keep = state(nx, ny)
    g = st.Grid(nx, ny, 1.3, 0.8, bc)
    A = st.assemble(g, eb, ep)
    ref = A @ st.to_vector(g, *[np.nan_to_num(v) for v in x])
    with tph.Solver(nx, ny, lx=1.3, ly=0.8, bc=bc, levels=1 if nx * ny < 2000 else 0) as s:
        s.set_coefficients(T(eb), T(ep), T(rb))
        out = [t.cpu().numpy() for t in s.apply(*[T(v) for v in x])]
        # an output in the place of an input
        vx, vy, p = [T(v) for v in x]
        ptr = lambda t: s._p(t, "t")  # noqa: E731
        ay, ap = torch.empty_like(vx), torch.empty_like(vx)
        assert s._lib.tph_apply(s._h, ptr(vx), ptr(vy), ptr(p), ptr(vx), ptr(ay), ptr(ap)) == 0
        same = [vx.cpu().numpy(), ay.cpu().numpy(), ap.cpu().numpy()]
    for o, q, k in zip(out, same, keep):
        assert np.all(o[~k] == 0) and np.all(q[~k] == 0)
    tol = 1e-13 * np.abs(ref).max()
    assert np.abs(st.to_vector(g, *out) - ref).max() <= tol
    assert np.abs(st.to_vector(g, *same) - ref).max() <= tol
