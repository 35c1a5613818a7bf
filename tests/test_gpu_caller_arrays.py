"""Arrays that a caller of the C functions may pass by mistake or in earnest: host memory and arrays that end beyond
their allocation are refused with an error (nothing reads them), pinned memory and odd addresses are taken."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2603_14040_amd as tph
import workloads as wl
from paper_2603_14040_amd import _lib

pytestmark = pytest.mark.gpu

DEV = "cuda"
NX, NY = 48, 32
SHAPE = (NY + 2, NX + 2)


def P(t):
    return ctypes.c_void_p(t.ctypes.data if isinstance(t, np.ndarray) else t.data_ptr())


def fields(seed, n=3):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return [torch.rand(SHAPE, generator=g, device=DEV, dtype=torch.float64) + 0.5 for _ in range(n)]


def short():
    """A pinned array one row short, which its allocation does not reach beyond: 2^k entries, k whole."""
    t = torch.empty(1024, dtype=torch.float64, pin_memory=True)
    assert t.numel() < SHAPE[0] * SHAPE[1]
    return t


@pytest.fixture()
def solver():
    with tph.Solver(NX, NY) as s:
        s.set_coefficients(*fields(1))
        yield s


@pytest.mark.parametrize("bad", ["host", "short"])
def test_refused(solver, bad):
    lib, h = _lib.load(), solver._h
    host = np.ones(SHAPE)
    x = P(host) if bad == "host" else P(short())
    ok = fields(2, 6)
    d = [P(t) for t in ok]
    info = _lib.Info()
    calls = {
        "set_coefficients": [(0, 1, 2), lambda a: lib.tph_set_coefficients(h, a[0], a[1], a[2], 0.0, -1.0, None, None)],
        "body force": [(0, 1), lambda a: lib.tph_set_coefficients(h, d[2], d[3], d[4], 0.0, -1.0, a[0], a[1])],
        "apply": [range(6), lambda a: lib.tph_apply(h, *a[:6])],
        "level_viscosity": [(0, 1), lambda a: lib.tph_level_viscosity(h, 0, a[0], a[1])],
        "lithostatic": [(0, 1), lambda a: lib.tph_lithostatic_pressure(h, a[0], -1.0, a[1])],
        "precondition": [range(6), lambda a: lib.tph_precondition(h, *a[:6])],
        "solve": [(0, 1, 2), lambda a: lib.tph_solve(h, a[0], a[1], a[2], ctypes.byref(info))],
        "adjoint": [(0, 1, 2), lambda a: lib.tph_solve_adjoint(h, *a[:6], ctypes.byref(info))],
    }
    for name, (places, call) in calls.items():
        for k in places:
            print(f"[case] {bad} array {k} of {name}", flush=True)
            solver.set_coefficients(*fields(1))
            a = list(d)
            a[k] = x
            assert _lib.STATUS_NAMES[call(a)] == "TPH_ERR_HIP"
            assert "not device memory" in lib.tph_last_error().decode()
    torch.cuda.synchronize()
    assert (host == 1.0).all()
    # the solver goes on
    pr = wl.sinker(32)
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    with tph.Solver(32, 32) as s:
        s.set_coefficients(T(pr.eta_b), T(pr.eta_p), T(pr.rho_b), pr.gx, pr.gy)
        assert s.solve()[3].status == "TPH_OK"


@pytest.mark.parametrize("kind", ["pinned", "odd address"])
def test_taken(solver, kind):
    lib, h = _lib.load(), solver._h
    keep = []

    def other(t):
        if kind == "pinned":
            u = torch.empty(SHAPE, dtype=torch.float64, pin_memory=True)
            u.copy_(t)
            p = u.data_ptr()
        else:                                    # four bytes into a device array
            u = torch.zeros(t.numel() * 8 + 8, dtype=torch.uint8, device=DEV)
            u[4:4 + t.numel() * 8] = t.reshape(-1).view(torch.uint8)
            p = u.data_ptr() + 4
        keep.append((u, t.numel() * 8))
        return ctypes.c_void_p(p)

    def back(k):
        u, n = keep[k]
        return u.to(DEV) if kind == "pinned" else u[4:4 + n].clone().view(torch.float64).view(SHAPE)

    c, x = fields(3), fields(4)
    solver.set_coefficients(*c)
    want = solver.apply(*x)
    zero = torch.zeros(SHAPE, dtype=torch.float64, device=DEV)
    out = [other(zero) for _ in range(3)]
    args = [other(t) for t in c]
    torch.cuda.synchronize()
    assert lib.tph_set_coefficients(h, *args, 0.0, -1.0, None, None) == 0
    assert lib.tph_apply(h, *[other(t) for t in x], *out) == 0
    torch.cuda.synchronize()
    for k, w in enumerate(want):
        # the two routes round their sums of some twenty products differently: 20 * 2^-53 of terms that are up to
        # some ten times the largest result
        assert (back(k) - w).abs().max().item() < 1e-13 * w.abs().max().item()
