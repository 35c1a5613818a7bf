"""Grid -> marker between nodes of very different size: the error is relative to the result, not to the larger node.

Spacings are powers of two and markers lie on a lattice of 2^-20 cells, so the parts rx, ry, 1 - rx, 1 - ry of a
cell and the products of two of them are exact.  What is left is four products and three sums of positive
terms (fewer with fused operations): seven roundings, 7 * 2^-53 < 8e-16 of the result.
"""
import numpy as np
import pytest
import torch

import paper_2603_14040_amd as tph
from oracle import markers as mk
from oracle import stokes as st

pytestmark = pytest.mark.gpu

T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731


def _markers(nx, ny, g):
    """Lattice positions: corners, middles and a hair beside every node line, the clamped half cells included."""
    u = np.array([0.0, 2.0 ** -20, 0.25, 0.5, 0.75, 1.0 - 2.0 ** -20])
    xs = np.append((np.arange(nx)[:, None] + u).ravel(), nx) * g.dx
    ys = np.append((np.arange(ny)[:, None] + u).ravel(), ny) * g.dy
    return (a.ravel() for a in np.meshgrid(xs, ys))


@pytest.mark.parametrize("kind", ["basic", "cell", "vx", "vy"])
@pytest.mark.parametrize("ratio", [1.0, 1e2, 1e6, 1e12])
def test_error_is_relative_to_the_result(kind, ratio):
    nx, ny = 9, 7
    g = st.Grid(nx, ny, nx / 16.0, ny / 16.0)
    xm, ym = _markers(nx, ny, g)
    rng = np.random.default_rng(5)
    grid = rng.uniform(1.0, 2.0, (ny + 2, nx + 2)) * np.where(rng.random((ny + 2, nx + 2)) < 0.5, 1.0, ratio)
    with_long = mk.grid_to_markers(g, kind, grid.astype(np.longdouble), xm.astype(np.longdouble),
                                   ym.astype(np.longdouble))
    m = tph.Markers(nx, ny, g.lx, g.ly, capacity=xm.size)
    got = m.from_grid(kind, T(xm), T(ym), T(grid)).cpu().numpy()
    m.close()
    assert with_long.dtype == np.longdouble
    assert np.abs(got / with_long - 1).max() < 8e-16


@pytest.mark.parametrize("kind", ["basic", "cell"])
def test_a_marker_on_a_node_has_its_value(kind):
    """Beyond the outermost nodes (the clamped half cells of the cell centres) too."""
    nx, ny = 6, 5
    g = st.Grid(nx, ny, nx / 8.0, ny / 8.0)
    rng = np.random.default_rng(6)
    grid = 10.0 ** rng.uniform(-9, 9, (ny + 2, nx + 2))
    h = 0.0 if kind == "basic" else 0.5
    lo = 0 if kind == "basic" else 1
    j, i = (a.ravel() for a in np.meshgrid(np.arange(lo, nx + 1), np.arange(lo, ny + 1)))
    xs, ys, want = [(j - h) * g.dx], [(i - h) * g.dy], [grid[i, j]]
    if kind == "cell":                       # the outer edges of the box: the nearest centre's value
        for e, f in ((0, 0), (nx, ny), (0, ny), (nx, 0)):
            xs.append(np.array([e * g.dx]))
            ys.append(np.array([f * g.dy]))
            want.append(np.array([grid[ny if f else 1, nx if e else 1]]))
    m = tph.Markers(nx, ny, g.lx, g.ly, capacity=256)
    got = m.from_grid(kind, T(np.concatenate(xs)), T(np.concatenate(ys)), T(grid)).cpu().numpy()
    m.close()
    assert np.array_equal(got, np.concatenate(want))


def test_infinite_and_huge_nodes():
    nx, ny = 4, 4
    grid = np.ones((ny + 2, nx + 2))
    grid[:, 2] = np.inf
    big = np.full((ny + 2, nx + 2), 2.0 ** 1023)       # their difference overflows
    big[:, 2] = -2.0 ** 1023
    x, y = np.array([1.5, 2.25]) / nx, np.array([1.25, 2.5]) / ny
    m = tph.Markers(nx, ny, capacity=16)
    assert np.isposinf(m.from_grid("basic", T(x), T(y), T(grid)).cpu().numpy()).all()
    assert np.array_equal(m.from_grid("basic", T(x), T(y), T(big)).cpu().numpy(), [0.0, -2.0 ** 1022])
    m.close()


@pytest.mark.parametrize("kind", ["basic", "cell", "vx", "vy"])
@pytest.mark.parametrize("nx,ny", [(10, 7), (30, 49)])
def test_no_weight_is_negative(kind, nx, ny):
    """Markers on node lines of a spacing that is no power of two: the scaled position rounds to either side of
    the line.  Node values are not left behind, whatever the neighbours (1 and 1e20 in turn)."""
    g = st.Grid(nx, ny)
    xs = np.arange(2 * nx + 1) * (0.5 * g.dx)
    ys = np.arange(2 * ny + 1) * (0.5 * g.dy)
    xm, ym = (a.ravel() for a in np.meshgrid(np.concatenate([xs, np.nextafter(xs, 0)]),
                                             np.concatenate([ys, np.nextafter(ys, 0)])))
    xm, ym = xm.clip(0, 1), ym.clip(0, 1)
    m = tph.Markers(nx, ny, capacity=xm.size)
    for flip in (0, 1):
        grid = np.where((np.add.outer(np.arange(ny + 2), np.arange(nx + 2)) + flip) % 2, 1e20, 1.0)
        got = m.from_grid(kind, T(xm), T(ym), T(grid)).cpu().numpy()
        # the weights add up to one but for the rounding of the two products and three sums
        assert got.min() > 1 - 1e-15 and got.max() < 1e20 * (1 + 1e-15)
    m.close()
