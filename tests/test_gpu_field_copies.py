"""Fields between the caller's dense arrays and the solver's pitched ones, bit for bit.

Widths below, at and above the 64 columns of a workgroup, heights about its 16 rows, long and flat grids:
the viscosities of level 0 come back as they went in, and a solution read back gives the residual that the
solve reported for its own.
"""
import pytest
import torch

import paper_2603_14040_amd as tph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(2, 2), (62, 14), (63, 15), (64, 13), (8, 510), (1030, 6), (192, 132)])
def test_fields_come_back_as_they_went_in(nx, ny):
    g = torch.Generator(device="cuda")
    g.manual_seed(nx)
    eb, ep, rb = (0.5 + torch.rand((ny + 2, nx + 2), generator=g, device="cuda", dtype=torch.float64) for _ in range(3))
    levels = 1 if nx * ny <= 2048 else 2 if nx * ny <= 8192 else 3       # at most 4096 unknowns on the coarsest level
    with tph.Solver(nx, ny, levels=levels, precision=tph.FP64, rtol=1e-6, max_iters=40) as s:
        s.set_coefficients(eb, ep, rb)
        gb, gp = s.level_viscosity(0)
        assert torch.equal(gb[:ny + 1, :nx + 1], eb[:ny + 1, :nx + 1])
        assert torch.equal(gp[1:ny + 1, 1:nx + 1], ep[1:ny + 1, 1:nx + 1])
        vx, vy, p, info = s.solve()
        # the pressure's mean is taken out after the reported residual: a rounding of the residual of the start
        assert abs(s.energy_residual(vx, vy, p) - info.res_energy) < 1e-12
