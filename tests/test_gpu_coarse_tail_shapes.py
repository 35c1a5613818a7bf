"""The single-workgroup coarse tail over its shapes.

One application of the preconditioner with the tail (coarse_level = l) against
the same cycle launched level by level (coarse_level = -2, checked against the
oracle elsewhere): every number of threads and cell pairs per thread, both
precisions and smoothers, ragged and elongated levels, coarsest systems whose
inverse is held in registers (up to 128 unknowns) and streamed, and hierarchies
of two to four tail levels.  Both run the same operations on the same levels;
only the sums of the dense coarsest product are ordered differently, so FP64
agrees to rounding (1e-12) and FP32 to the bound of the parity tests (2e-5).
"""
import pytest
import torch

import paper_2603_14040_amd as tph

pytestmark = pytest.mark.gpu

# (nx, ny, levels, tail level): pairs of the tail's top level, coarsest unknowns
CASES = [
    (16, 16, 2, 0),      # 128 pairs, 112 unknowns
    (32, 16, 2, 0),      # 256 pairs, 232 unknowns
    (36, 16, 2, 0),      # 288 pairs: 512 threads, part of them idle
    (32, 32, 3, 0),      # 512 pairs
    (36, 32, 2, 0),      # 576 pairs: two per thread
    (64, 32, 3, 0),      # 1024 pairs (FP32 only)
    (64, 48, 4, 0),      # 1536 pairs: four per thread (FP32 only)
    (128, 16, 2, 0),     # elongated (FP32 only)
    (8, 64, 3, 0),
    (4, 4, 2, 0),        # the smallest: 2 x 2 coarsest
    (48, 80, 4, 1),      # 24 x 40 tail under a finest level
    (104, 72, 4, 2),     # 26 x 18, coarsest 13 x 9 (212 unknowns)
]


def run(nx, ny, levels, prec, smoother, nu, bc, coarse_level):
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    R = lambda: torch.rand((ny + 2, nx + 2), generator=g, device="cuda", dtype=torch.float64)  # noqa: E731
    eb, ep, rb = 10.0 ** (2 * R()), 10.0 ** (2 * R()), R()
    eb[:, nx + 1] = ep[:, nx + 1] = eb[ny + 1] = ep[ny + 1] = float("nan")     # outside the ranges: ignored
    ep[0] = ep[:, 0] = float("nan")
    r = [R() - 0.5 for _ in range(3)]
    with tph.Solver(nx, ny, lx=1.0, ly=0.7, levels=levels, precision=prec, smoother=smoother, nu_pre=nu[0], nu_post=nu[1],
                    omega=0.8, bc=bc, uzawa_steps=1, restart=1, coarse_level=coarse_level) as s:
        s.set_coefficients(eb, ep, rb)
        return [t.clone() for t in s.precondition(*r)], s.level_plan(max(coarse_level, 0))[0]


@pytest.mark.parametrize("nx,ny,levels,lc", CASES)
@pytest.mark.parametrize("prec", [tph.FP64, tph.MIXED])
@pytest.mark.parametrize("smoother,nu,bc", [(tph.SMOOTH_GS, (1, 2), (0, 1, 0, 1)), (tph.SMOOTH_GS, (2, 0), (1, 1, 1, 1)),
                                            (tph.SMOOTH_JACOBI, (2, 1), (0, 0, 0, 0)), (tph.SMOOTH_GS, (0, 1), (1, 0, 1, 0))])
def test_tail_is_the_cycle_level_by_level(nx, ny, levels, lc, prec, smoother, nu, bc):
    if prec == tph.FP64 and (nx >> lc) * (ny >> lc) > 36 * 32:
        pytest.skip("does not fit one workgroup's LDS in FP64")
    got, kind = run(nx, ny, levels, prec, smoother, nu, bc, lc)
    assert kind == "coarse_tail"
    ref, _ = run(nx, ny, levels, prec, smoother, nu, bc, -2)
    tol = 1e-12 if prec == tph.FP64 else 2e-5
    for a, b in zip(got, ref):
        assert bool(torch.isfinite(a).all())
        assert float((a - b).norm()) <= tol * float(b.norm())
