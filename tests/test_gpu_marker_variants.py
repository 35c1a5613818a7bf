"""Marker -> grid through every kernel that the counts choose: node averages with one and two cell rows a wave and
each size of a staged piece, buckets sorted by four waves and by eight, two-level binning with each tile size."""
import numpy as np
import pytest
import torch

import paper_2603_14040_amd as tph
from oracle import markers as mk
from oracle import stokes as st

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,n,crowd", [
    # one row a wave (up to 300000 cells), pieces of 128, 192, 256 and 320 markers: by the mean of 16 cells
    (150, 100, 60000, 0), (150, 100, 120000, 0), (150, 100, 180000, 0), (150, 100, 240000, 0),
    # two rows a wave, the same
    (600, 510, 1200000, 0), (600, 510, 2150000, 0), (600, 510, 3370000, 0), (600, 510, 4900000, 0),
    (547, 547, 300000, 0), (546, 547, 300000, 0),           # the cell counts on both sides of the line
    # more than 4096 markers a bucket (79 of 32 cells): sorted by eight waves, in one piece and in two
    (60, 40, 400000, 0), (60, 40, 400000, 30000),
    # two passes, the second and the third tile size
    (2300, 2050, 2 ** 18 + 3, 0), (2300, 2050, 2 ** 22 + 5, 0),
])
def test_to_grid_against_the_oracle(nx, ny, n, crowd):
    g = st.Grid(nx, ny, nx / 1024.0, ny / 1024.0)            # spacings a power of two, as in the binning's tests
    rng = np.random.default_rng(nx + n)
    x, y, f = rng.uniform(0, g.lx, n), rng.uniform(0, g.ly, n), rng.uniform(0.5, 1.5, n)
    x[:crowd] = (nx // 2 + rng.random(crowd)) * g.dx         # in one cell
    y[:crowd] = (ny // 2 + rng.random(crowd)) * g.dy
    perm = rng.permutation(n)
    x, y = x[perm], y[perm]
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    m = tph.Markers(nx, ny, g.lx, g.ly, capacity=n)
    for kind in ("basic", "cell") if n < 1000000 else ("basic",):
        print(f"[case] variants {nx}x{ny} n={n} crowd={crowd} {kind}", flush=True)
        got = m.to_grid(kind, T(x), T(y), [T(f)], fill=-3.0)[0].cpu().numpy()
        ref = mk.markers_to_grid(g, kind, x, y, f, fill=-3.0)
        lo = 1 if kind == "cell" else 0
        got, ref = got[lo:ny + 1, lo:nx + 1], ref[lo:ny + 1, lo:nx + 1]
        assert np.array_equal(got == -3.0, ref == -3.0)
        # positive values and weights: sums of N terms agree to N eps, N at most 31000 in these cases
        assert np.abs(got - ref).max() < 1e-11
    m.close()
