"""The dense inverse of the coarsest operator, at the edges of the panels of its elimination.

A hierarchy of one level is the dense solve alone.  Sizes: less than a panel of 32 unknowns, one less and one
exactly, one and two panels with a remainder, a multiple of 32, the sizes about 136 that one workgroup can
hold, and the largest coarsest grid of the default hierarchies (15 x 15).  Condition numbers are below 1e6
(viscosity within two decades, at most 15 cells a side), so both solves agree to 1e6 eps with a margin of ten.
"""
import numpy as np
import pytest
import torch

import paper_2603_14040_amd as tph
from oracle import multigrid as mg
from oracle import stokes as st

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,unknowns", [(4, 4, 24), (4, 5, 31), (3, 7, 32), (5, 8, 67), (2, 22, 64), (8, 8, 112), (7, 11, 136),
                                            (6, 13, 137), (13, 9, 212), (15, 15, 420)])
def test_dense_solve_matches_the_oracle(nx, ny, unknowns):
    assert 2 * nx * ny - nx - ny == unknowns
    rng = np.random.default_rng(unknowns)
    shape = (ny + 2, nx + 2)
    eb, ep, rb = 10.0 ** rng.uniform(0, 2, shape), 10.0 ** rng.uniform(0, 2, shape), rng.random(shape)
    g = st.Grid(nx, ny)
    prm = mg.MGParams(levels=1, nu_pre=[1], nu_post=[1], alpha=1.0)
    rx, ry, rp = (rng.standard_normal(shape) for _ in range(3))
    ox, oy, _ = mg.precondition(mg.build_hierarchy(g, eb, ep, prm), prm, rx, ry, rp)
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    with tph.Solver(nx, ny, levels=1, precision=tph.FP64, alpha=1.0, uzawa_steps=1, restart=1) as s:
        s.set_coefficients(T(eb), T(ep), T(rb))
        gx, gy, _ = s.precondition(T(rx), T(ry), T(rp))
    gx, gy = gx.cpu().numpy(), gy.cpu().numpy()
    a, b = gx[1:ny + 1, 1:nx], gy[1:ny, 1:nx + 1]
    assert np.linalg.norm(a - ox[1:ny + 1, 1:nx]) < 1e-9 * np.linalg.norm(ox[1:ny + 1, 1:nx])
    assert np.linalg.norm(b - oy[1:ny, 1:nx + 1]) < 1e-9 * np.linalg.norm(oy[1:ny, 1:nx + 1])
