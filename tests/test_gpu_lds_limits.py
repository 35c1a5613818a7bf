"""Dynamic LDS beyond 64 KB belongs to a kernel, not to a handle: handles of several sizes alive at once, and the
largest used after a smaller one was made."""
import numpy as np
import pytest
import torch

import paper_2603_14040_amd as tph
from oracle import markers as mk
from oracle import stokes as st

pytestmark = pytest.mark.gpu

DEV = "cuda"


def test_marker_handles_of_falling_need():
    # 2053 (73.9 KB), 2300 (82.8 KB), 1958 (70.5 KB) and 1861 (67.0 KB) buckets of 512 cells, then one below 64 KB
    sides = [(1024, 1024), (1084, 1084), (1000, 1000), (975, 975), (120, 90)]
    handles = [(nx, ny, tph.Markers(nx, ny, capacity=30001)) for nx, ny in sides]
    rng = np.random.default_rng(1)
    n = 30001
    x, y, f = rng.random(n), rng.random(n), rng.uniform(0.5, 1.5, n)
    T = lambda a: torch.from_numpy(a).to(DEV)  # noqa: E731
    for nx, ny, m in handles:
        print(f"[case] lds {nx}x{ny}", flush=True)
        got = m.to_grid("basic", T(x), T(y), [T(f)], fill=-3.0)[0].cpu().numpy()[:ny + 1, :nx + 1]
        ref = mk.markers_to_grid(st.Grid(nx, ny), "basic", x, y, f, fill=-3.0)[:ny + 1, :nx + 1]
        # averages of values in [0.5, 1.5]; a weight's error is eps times the position in cells, and the smallest
        # weight that a node hangs on alone is 1e-8 or more: markers that near a cell's edge are few in 30001
        assert np.array_equal(got == -3.0, ref == -3.0)
        assert np.abs(got - ref).max() < 1e-6
    for *_, m in handles:
        m.close()


@pytest.mark.parametrize("precision", [tph.FP64, tph.MIXED])
def test_largest_coarse_tail(precision):
    """The tails that need the most LDS (96 x 16 cells in FP64, 88 x 40 in FP32, beside smaller ones) against the
    level-by-level kernels, which use none."""
    shapes = [(96, 16), (40, 88), (32, 32)]
    solvers = [tph.Solver(nx, ny, precision=precision, rtol=1e-10, max_iters=200, levels=4) for nx, ny in shapes]
    for (nx, ny), s in zip(shapes, solvers):
        assert "coarse_tail" in [s.level_plan(k)[0] for k in range(s.levels)]
        g = torch.Generator(device=DEV)
        g.manual_seed(nx)
        c = [torch.exp(torch.randn((ny + 2, nx + 2), generator=g, device=DEV, dtype=torch.float64)) for _ in range(3)]
        s.set_coefficients(*c)
        a = s.solve()
        with tph.Solver(nx, ny, precision=precision, rtol=1e-10, max_iters=200, levels=4, fused=False) as u:
            u.set_coefficients(*c)
            b = u.solve()
        assert a[3].status == b[3].status == "TPH_OK"
        for p, q in zip(a[:3], b[:3]):
            # both stop at a relative residual of 1e-10; the operator's condition on so few cells is below 1e5
            assert (p - q).abs().max().item() < 1e-5 * q.abs().max().item()
    for s in solvers:
        s.close()
