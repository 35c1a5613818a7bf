"""Marker -> grid at the edges of the binning: one marker, tiles of each size with and without a remainder,
buckets of each width, one pass and two, buckets sorted in pieces, markers in cell order and shuffled."""
import numpy as np
import pytest
import torch

import paper_2603_14040_amd as tph
from oracle import markers as mk
from oracle import stokes as st

pytestmark = pytest.mark.gpu

DEV = "cuda"


@pytest.mark.parametrize("nx,ny,n,order", [
    (1, 1, 1, "cells"),                       # one marker, one bucket
    (62, 7, 1023, "random"),                  # one column block of nodes, one tile less a marker
    (63, 8, 1025, "cells"),                   # the next of each
    (300, 136, 2 ** 18, "random"),            # 32-cell buckets, the most markers of the smallest tile
    (200, 205, 2 ** 18 + 1, "random"),        # the next larger tile
    (640, 400, 2 ** 22 + 4097, "cells"),      # the largest tile, with a remainder
    (1030, 1020, 300001, "random"),           # 512-cell buckets, two rows a wave
    (2000, 1301, 70001, "random"),            # the widest buckets, in one pass
    (2300, 2050, 70001, "cells"),             # two passes
    (90, 64, 50000, "crowded"),               # a bucket in pieces
    (2300, 2050, 50000, "crowded"),           # the same behind two passes
])
def test_to_grid_at_the_edges_of_the_binning(nx, ny, n, order):
    g = st.Grid(nx, ny, nx / 1024.0, ny / 1024.0)   # spacings a power of two: weights agree to a few eps, small ones too
    rng = np.random.default_rng(nx + n)
    if order == "crowded":                    # half of them in two neighbouring cells
        xm, ym = rng.uniform(0, g.lx, n), rng.uniform(0, g.ly, n)
        half = n // 2
        xm[:half] = (nx // 2 + 2.0 * rng.random(half)) * g.dx
        ym[:half] = (ny // 2 + rng.random(half)) * g.dy
        perm = rng.permutation(n)
        xm, ym = xm[perm], ym[perm]
    elif order == "cells":                    # by cell, moved by up to three
        c = np.sort(rng.integers(0, nx * ny, n))
        xm = np.clip((c % nx + rng.random(n)) * g.dx + rng.uniform(-3, 3, n) * g.dx, 0, g.lx)
        ym = np.clip((c // nx + rng.random(n)) * g.dy + rng.uniform(-3, 3, n) * g.dy, 0, g.ly)
    else:
        xm, ym = rng.uniform(0, g.lx, n), rng.uniform(0, g.ly, n)
    f = rng.uniform(0.5, 1.5, n)
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)  # noqa: E731
    m = tph.Markers(nx, ny, g.lx, g.ly, capacity=n, device=DEV)
    for kind in ("basic", "cell"):
        print(f"[case] binning {nx}x{ny} n={n} {order} {kind}", flush=True)
        got = m.to_grid(kind, T(xm), T(ym), [T(f)], fill=-3.0)[0].cpu().numpy()
        again = m.to_grid(kind, T(xm), T(ym), [T(f)], fill=-3.0)[0].cpu().numpy()
        assert np.array_equal(got, again)
        ref = mk.markers_to_grid(g, kind, xm, ym, f, fill=-3.0)
        lo = 1 if kind == "cell" else 0
        got, ref = got[lo:ny + 1, lo:nx + 1], ref[lo:ny + 1, lo:nx + 1]
        assert np.array_equal(got == -3.0, ref == -3.0)
        # positive values and weights: sums of N terms agree to N eps, N at most 25000 in these cases
        assert np.abs(got - ref).max() < 1e-11
    m.close()
