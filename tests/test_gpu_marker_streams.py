"""Markers on a stream of their own, the caller's stream busy: each waits for the other where it has to."""
import pytest
import torch

import paper_2603_14040_amd as tph

pytestmark = pytest.mark.gpu


def test_to_grid_behind_a_busy_stream(monkeypatch):
    nx, ny, n = 40, 30, 12000
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    x, y, f = (torch.rand(n, generator=g, device="cuda", dtype=torch.float64) for _ in range(3))
    same = tph.Markers(nx, ny, capacity=n)
    want = same.to_grid("basic", x, y, [f, 2.0 * f], fill=-1.0)
    side = tph.Markers(nx, ny, capacity=n, stream=torch.cuda.Stream())
    torch.cuda.synchronize()
    zeros = torch.zeros

    def late(*args, **kw):
        torch.cuda._sleep(20_000_000)                # some 10 ms on the caller's stream before the zeros
        return zeros(*args, **kw)

    monkeypatch.setattr(torch, "zeros", late)
    got = side.to_grid("basic", x, y, (a for a in (f, 2.0 * f)), fill=-1.0)     # any iterable of fields
    monkeypatch.undo()
    # read on the caller's stream, which waits for the markers' one
    assert all(torch.equal(a, b) for a, b in zip(got, want))
    same.close()
    side.close()
