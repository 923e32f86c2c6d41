"""The FP64 pass in strips and in tiles, each forced on the same grids: the
fields, the residuals and the passes a tolerance step takes are equal, bit for
bit (the strips evaluate the tiles' expressions, so the tolerance is zero).
Grids of one narrow strip, of a last strip of one column, of four to seven rows
and with more than one segment; every boundary kind; obstacles that
leave rows of solid cells alone in a strip, at a wall, across a strip border and
across the periodic seam.  Solid cells keep the values a caller wrote to the
state's device arrays, in every later step and in either form.
"""
from __future__ import annotations


import numpy as np
import pytest

from paper_1802_04243_amd import workloads as W

pytestmark = pytest.mark.gpu
TILES, STRIPS = 1, 2


def _widths(n, seed):
    return np.random.default_rng(seed).uniform(0.018, 0.03, n)


def _problem(name):
    if name == "one_strip":  # fewer columns than a strip, walls two cells from each other's rules
        return W.Problem(nx=41, ny=9, dx=_widths(41, 1), dy=_widths(9, 2), obstacles=[(12, 3, 14, 4)])
    if name == "narrow_periodic":
        return W.Problem(nx=7, ny=300, periodic=True, dx=_widths(7, 3), dy=_widths(300, 4), gx=0.2,
                         wall_u=(0.3, -0.2), obstacles=[(0, 40, 6, 52), (5, 100, 5, 101)])
    if name.startswith("rows"):  # every row is next to a wall
        ny = int(name[4:])
        return W.Problem(nx=230, ny=ny, dx=_widths(230, 13), dy=_widths(ny, 14), wall_u=(0.2, 0.1),
                         periodic=ny % 2 == 1, gx=0.1, obstacles=[(70, 0, 140, 1)] if ny > 4 else [])
    if name == "last_column":  # 58 strips of 58 columns and one of one
        return W.Problem(nx=3365, ny=40, dx=_widths(3365, 11), dy=_widths(40, 12), obstacles=[(3350, 10, 3362, 12)])
    if name == "obstacles":  # at the inlet, at the bottom wall over whole strips, of one cell
        obst = [(2, 100, 20, 140), (300, 0, 480, 30), (500, 150, 501, 179), (640, 60, 899, 120),
                (1000, 90, 1000, 90), (1100, 40, 1130, 41)]
        return W.Problem(nx=1202, ny=180, dx=_widths(1202, 5), dy=_widths(180, 6), obstacles=obst,
                         obstacle_T=1.1)
    if name == "periodic":  # a block across the seam, one that touches the top wall
        return W.Problem(nx=349, ny=131, periodic=True, dx=_widths(349, 7), dy=_widths(131, 8), gx=0.1,
                         wall_type=(1, 0), obstacles=[(0, 30, 130, 70), (250, 30, 348, 70), (150, 100, 230, 130)])
    nx, ny = 1900, 160  # slip-jump walls and obstacles
    return W.Problem(nx=nx, ny=ny, dx=_widths(nx, 9), dy=_widths(ny, 10), wall_type=(2, 1),
                     wall_u=(0.5, 0.0), kn=0.01, obstacle_type=W.WALL_SLIP_JUMP,
                     obstacles=[(60, 0, 190, 20), (1300, 70, 1420, 90)], gx=0.1)


def _form(s, form):
    from paper_1802_04243_amd import sts
    return sts.lib().sts_internal_pass_form(s._h, form)


def _pair(p, seed):
    """A solver of each form with the same state."""
    from paper_1802_04243_amd import sts
    out = []
    for form in (TILES, STRIPS):
        s = sts.Solver(p)
        s.set_fields(*W.initial_fields(p, seed, amp=1e-2))
        n = _form(s, form)
        assert (n == 0) == (form == TILES), (form, n)
        out.append(s)
    return out


def _same(a, b, label):
    for f, x, y in zip("uvpT", a.fields(), b.fields()):
        assert np.array_equal(x, y, equal_nan=True), (label, f, int((x != y).sum()))
    assert np.array_equal(a.residuals(), b.residuals()), label


@pytest.mark.parametrize("name", ["one_strip", "narrow_periodic", "rows4", "rows5", "rows6", "rows7",
                                  "last_column", "obstacles", "periodic", "slip"])
@pytest.mark.parametrize("scheme", list(W.SCHEMES))
def test_strips_equal_tiles(name, scheme):
    p, k = _problem(name), W.SCHEMES[scheme]
    dt = 0.2 * p.cfl_dt()
    print(f"case {name} {p.nx}x{p.ny} {scheme}", flush=True)
    pair = _pair(p, 9)
    for n in (1, 2, 5):
        for s in pair:
            s.step(dt, n, k)
        _same(*pair, (n, "passes"))
    passes = [s.step_tol(dt, 6, 1e-9, k) for s in pair]
    assert passes[0] == passes[1]
    _same(*pair, "tolerance step")
    for s in pair:
        s.close()


@pytest.mark.parametrize("name", ["one_strip", "obstacles", "periodic"])
@pytest.mark.parametrize("scheme", list(W.SCHEMES))
def test_strips_equal_tiles_on_values_that_are_not_finite(name, scheme):
    """NaN, infinities, zero and negative temperatures and pressures: the same
    entries of every field become non-finite, and as many are reported."""
    from paper_1802_04243_amd import sts
    p, k = _problem(name), W.SCHEMES[scheme]
    rng = np.random.default_rng(8)
    pair = _pair(p, 9)
    for bad in (np.nan, np.inf, -np.inf, 0.0, -1.0):
        f = [a.copy() for a in W.initial_fields(p, 9, amp=1e-2)]
        for a in f:
            a.flat[rng.integers(0, a.size, 3)] = bad
        for s in pair:
            s.set_fields(*f)
        for n in (1, 1, 2):
            out = []
            for s in pair:
                s.step(0.2 * p.cfl_dt(), n, k)
                r = np.zeros(6)
                rc = sts.lib().sts_residuals(s._h, sts._ptr(r))
                out.append((rc, sts.lib().sts_last_error() if rc else b"", r))
            assert out[0][:2] == out[1][:2], (bad, n, out)
            assert np.array_equal(out[0][2], out[1][2], equal_nan=True), (bad, n, out)
            for q, x, y in zip("uvpT", *(s.fields() for s in pair)):
                assert np.array_equal(x, y, equal_nan=True), (bad, n, q)
    for s in pair:
        s.close()


class _Array:
    def __init__(self, ptr, shape, pitch):
        self.__cuda_array_interface__ = dict(shape=shape, strides=(8 * pitch, 8), typestr="<f8",
                                             data=(ptr, False), version=2)


@pytest.mark.parametrize("name", ["narrow_periodic", "obstacles", "periodic"])
@pytest.mark.parametrize("scheme", ["explicit_upwind", "implicit_tvd"])
def test_solid_cells_keep_what_a_caller_wrote(name, scheme):
    import torch
    p, k = _problem(name), W.SCHEMES[scheme]
    dt = 0.2 * p.cfl_dt()
    solid = np.zeros((p.ny, p.nx), bool)
    for i0, j0, i1, j1 in p.obstacles:
        solid[j0:j1 + 1, i0:i1 + 1] = True
    pair = _pair(p, 3)
    for s in pair:
        ptrs, origin, pitch = s.field_ptrs()
        for f, (ptr, shape) in enumerate(zip(ptrs, s.shapes())):
            t = torch.as_tensor(_Array(ptr + 8 * origin, shape, pitch), device="cuda")
            m = torch.tensor(np.pad(solid, [(0, a - b) for a, b in zip(shape, solid.shape)]), device="cuda")
            t[m] = 0.25 + 0.01 * f
        torch.cuda.synchronize()
        for n in (1, 1, 3):
            s.step(dt, n, k)
            T, q = s.fields()[3], s.fields()[2]
            assert (T[solid] == 0.28).all() and (q[solid] == 0.27).all(), n
        s.step_tol(dt, 3, 1e-12, k)
        assert (s.fields()[3][solid] == 0.28).all()
    _same(*pair, "after the edits")
    for s in pair:
        s.close()


def test_the_grids_of_the_oracle_tests_take_the_form_they_are_meant_for():
    """The strips' parity with the oracle is tested on grids that take strips,
    the replayed steps' on a grid that records them."""
    from paper_1802_04243_amd import sts
    import test_march_gpu as M
    for name in ("periodic", "obstacles", "slip"):
        s = sts.Solver(M._problem(name))
        assert _form(s, 0) > 0, name
        s.close()
    p, run = W.workload("channel_120x24")
    s = sts.Solver(p, use_torch=False)
    assert _form(s, 0) == 0
    s.set_fields(*W.initial_fields(p, 1))
    graphs = sts.lib().sts_internal_graphs
    for n, recorded in ((6, 1), (5, 3)):  # an odd number of passes: one from either buffer
        for _ in range(20):
            s.step(run["dt"], n, W.EXPLICIT)
        assert graphs(s._h) == recorded
    s.residuals()
    s.close()
