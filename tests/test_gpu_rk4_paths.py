"""RK4 of many markers and of few: one kernel keeps a cell's nodes between the stages and takes short cuts inside the
node range, the other does neither.  A marker's path does not depend on the others, so both give the same bits."""
import pytest
import torch

import paper_2603_14040_amd as tph

pytestmark = pytest.mark.gpu

F64 = torch.float64


@pytest.mark.parametrize("nx,ny", [(10, 7), (300, 211)])
@pytest.mark.parametrize("cells_a_step", [0.3, 5.0, 200.0])
def test_same_bits(nx, ny, cells_a_step):
    n = 60001                                # one more than the few
    g = torch.Generator(device="cuda")
    g.manual_seed(nx)
    x, y = (torch.rand(n, generator=g, device="cuda", dtype=F64) for _ in range(2))
    x[: n // 4] = torch.round(x[: n // 4] * 2 * nx) / (2 * nx)      # on node lines and between them
    y[n // 8: n // 3] = torch.round(y[n // 8: n // 3] * 2 * ny) / (2 * ny)
    x[:7] = torch.tensor([0.0, 1.0, -0.5, 1.5, float("nan"), float("inf"), 0.5], device="cuda", dtype=F64)
    y[:7] = torch.tensor([1.0, 0.0, 0.5, 2.0, 0.5, 0.5, float("nan")], device="cuda", dtype=F64)
    v = [torch.randn((ny + 2, nx + 2), generator=g, device="cuda", dtype=F64) for _ in range(2)]
    dt = cells_a_step / max(nx, ny)
    m = tph.Markers(nx, ny, capacity=n)
    a, b = x.clone(), y.clone()
    m.advect_rk4(a, b, *v, dt)
    parts = []
    for lo, hi in ((0, 30001), (30001, n)):
        p, q = x[lo:hi].clone(), y[lo:hi].clone()
        m.advect_rk4(p, q, *v, dt)
        parts.append((p, q))
    m.close()
    for many, few in zip((a, b), (torch.cat(t) for t in zip(*parts))):
        assert torch.equal(many.isnan(), few.isnan()) and many.isnan().sum().item() <= 2
        assert torch.equal(many.nan_to_num(), few.nan_to_num())
