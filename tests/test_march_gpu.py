"""The marching form of the FP64 pass (column strips, one wave each), which the
library takes on larger grids, against the FP64 oracle: every boundary kind,
obstacles on the walls, beside the inlet and outlet and in strips of their own
(rows of solid cells alone keep their values), stretched widths, extents that
are no multiples of a strip or a segment, loop 2 to a tolerance.

Asserted: normwise relative difference <= 1e-10 per field, the parity bar of the
FP64 form (the kernels evaluate the equations in another operation order with
fused multiply-adds), and equal pass counts.  One or two short steps from a
seeded state: implicit TVD's limiter is discontinuous in the old iterate, so
longer runs of it are compared elsewhere, step by step.
"""
from __future__ import annotations

import numpy as np
import pytest

from paper_1802_04243_amd import workloads as W

pytestmark = pytest.mark.gpu
TOL = 1e-10


def _widths(n, seed):
    return np.random.default_rng(seed).uniform(0.018, 0.03, n)


def _problem(name):
    rng = np.random.default_rng(17)
    if name == "periodic":
        nx, ny = 1103, 389
        return W.Problem(nx=nx, ny=ny, periodic=True, dx=_widths(nx, 1), dy=_widths(ny, 2),
                         wall_u=(0.3, -0.2), wall_T=(1 + 0.1 * rng.uniform(size=nx),
                                                     1 - 0.1 * rng.uniform(size=nx)), gx=0.2, gy=-0.1)
    if name == "obstacles":
        nx, ny = 1700, 601
        obst = [(2, 100, 20, 140), (nx - 40, 300, nx - 3, 320), (300, 0, 340, 9),
                (500, ny - 5, 501, ny - 1), (640, 200, 899, 420), (1000, 250, 1000, 250),
                (1100, 300, 1130, 301)]
        return W.Problem(nx=nx, ny=ny, dx=_widths(nx, 3), dy=_widths(ny, 4), obstacles=obst,
                         u_in=1 + 0.05 * rng.uniform(size=ny), T_in=1 + 0.05 * rng.uniform(size=ny),
                         obstacle_T=1.1)
    nx, ny = 1601, 640  # slip-jump and adiabatic walls, slip-jump obstacles
    return W.Problem(nx=nx, ny=ny, dx=_widths(nx, 5), dy=_widths(ny, 6), wall_type=(2, 1),
                     wall_u=(0.5, 0.0), kn=0.01, obstacle_type=W.WALL_SLIP_JUMP,
                     obstacles=[(200, 0, 230, 20), (700, 300, 760, 340)], gx=0.1)


def _pair(p, seed):
    from oracle import oracle as O
    from paper_1802_04243_amd import sts
    g, o = sts.Solver(p), O.Oracle(p)
    f0 = W.initial_fields(p, seed, amp=1e-2)
    g.set_fields(*f0)
    o.set_fields(*f0)
    return g, o


def _compare(g, o, label):
    errs = [float(np.abs(a - b).max() / np.abs(b).max()) for a, b in zip(g.fields(), o.fields())]
    rg, ro = g.residuals(), o.residuals()
    print(f"{label}: " + " ".join(f"{n}={e:.1e}" for n, e in zip("uvpT", errs)), flush=True)
    assert max(errs) <= TOL, (label, errs)
    # the increments are differences of fields of size one, as in the 3-D parity
    # tests: relative to their own size down to the fields' rounding
    assert np.abs(rg[:4] - ro[:4]).max() <= 1e-8 * np.abs(ro[:4]).max() + 1e-14, (label, rg, ro)


@pytest.mark.parametrize("name", ["periodic", "obstacles", "slip"])
@pytest.mark.parametrize("scheme", list(W.SCHEMES))
def test_march_matches_the_oracle(name, scheme):
    p = _problem(name)
    dt = 0.2 * p.cfl_dt()
    print(f"case {name} {p.nx}x{p.ny} {scheme}", flush=True)
    g, o = _pair(p, 9)
    for _ in range(2):
        g.step(dt, 4, W.SCHEMES[scheme])
        o.step(dt, 4, W.SCHEMES[scheme])
    _compare(g, o, f"{name}/{scheme}")
    if scheme != "implicit_tvd":
        ng, no = (s.step_tol(dt, 30, 1e-7, W.SCHEMES[scheme]) for s in (g, o))
        assert ng == no, (ng, no)
        _compare(g, o, f"{name}/{scheme} to 1e-7 in {ng} passes")
    g.close()
