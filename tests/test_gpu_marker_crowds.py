"""Marker -> grid where some cells hold far more markers than the others: the sums of a run of sixteen cells on both
sides of the 512 markers from which each cell is summed by all lanes, and over pieces of every size.

The reference adds up in extended precision.  Spacings are powers of two, so a marker's parts of its cell are exact
but for 1 - r; with positive values a node's average is off by the roundings of its longest chain of sums: at most
512 in the walked runs, N / 16 + 4 in the others, and four more over the cells.
"""
import numpy as np
import pytest
import torch

import paper_2603_14040_amd as tph
from oracle import markers as mk
from oracle import stokes as st

pytestmark = pytest.mark.gpu


def reference(g, kind, x, y, f):
    x0, y0, jmin, jmax, imin, imax = mk.node_grid(g, kind)
    X, Y = x.astype(np.longdouble), y.astype(np.longdouble)
    j, i = np.floor((x - x0) / g.dx).astype(int), np.floor((y - y0) / g.dy).astype(int)
    rx, ry = (X - (x0 + j * g.dx)) / g.dx, (Y - (y0 + i * g.dy)) / g.dy
    num, den = np.zeros((g.ny + 2, g.nx + 2), np.longdouble), np.zeros((g.ny + 2, g.nx + 2), np.longdouble)
    for a, b, w in ((0, 0, (1 - rx) * (1 - ry)), (0, 1, rx * (1 - ry)), (1, 0, (1 - rx) * ry), (1, 1, rx * ry)):
        ok = (i + a >= imin) & (i + a <= imax) & (j + b >= jmin) & (j + b <= jmax)
        np.add.at(num, (i[ok] + a, j[ok] + b), (w * f)[ok])
        np.add.at(den, (i[ok] + a, j[ok] + b), w[ok])
    return np.where(den > 0, num / np.where(den > 0, den, 1), -3.0)


@pytest.mark.parametrize("nx,ny,base,crowds", [
    (40, 9, 32, {}),                                            # every run has 512 markers
    (40, 9, 32, {17: 33, 90: 33}),                              # some have one more
    (70, 5, 3, {0: 700, 15: 1, 62: 900, 63: 513, 69: 20000}),   # ends of runs and of column blocks
    (70, 40, 0, {5: 600, 8: 17, 6: 15, 1000: 16, 1001: 600, 2799: 641}),   # empty cells between
    (140, 66, 9, {777: 5000, 778: 5000, 779: 1, 917: 3000}),    # longer pieces
    (600, 520, 1, {100: 4000, 5000: 600, 170123: 2500}),        # two rows a wave
    (600, 520, 0, {k: 400 for k in range(160000, 160060)}),
])
def test_sums_of_crowded_cells(nx, ny, base, crowds):
    g = st.Grid(nx, ny, nx / 1024.0, ny / 1024.0)
    rng = np.random.default_rng(nx + base)
    count = np.full(nx * ny, base)
    for c, k in crowds.items():
        count[c] = k
    cell = rng.permutation(np.repeat(np.arange(nx * ny), count))
    u = rng.integers(1, 2 ** 30, (2, cell.size)) * 2.0 ** -30   # no marker on an edge
    x, y, f = (cell % nx + u[0]) * g.dx, (cell // nx + u[1]) * g.dy, rng.uniform(0.5, 1.5, cell.size)
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    m = tph.Markers(nx, ny, g.lx, g.ly, capacity=cell.size)
    longest = max(512, max(list(crowds.values()) + [0]) / 16 + 4) + 4
    for kind in ("basic", "cell"):
        print(f"[case] crowds {nx}x{ny} {kind} n={cell.size}", flush=True)
        got = m.to_grid(kind, T(x), T(y), [T(f)], fill=-3.0)[0].cpu().numpy()
        again = m.to_grid(kind, T(x), T(y), [T(f)], fill=-3.0)[0].cpu().numpy()
        assert np.array_equal(got, again)
        lo = 1 if kind == "cell" else 0
        got, ref = got[lo:ny + 1, lo:nx + 1], reference(g, kind, x, y, f)[lo:ny + 1, lo:nx + 1]
        # the chain's roundings in numerator and denominator, and a few of a weight and the division
        assert np.abs(got / ref - 1).max() < (2 * longest + 10) * 2.0 ** -53
    m.close()
