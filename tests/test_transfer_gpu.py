"""Setting and reading fields on the GPU against the oracle's boundary rules.

Dense host arrays are scattered and gathered by kernels that also impose the
boundary values, so what comes back is a copy, a constant or an exact zero:
every comparison is for equality.  Grids below and above one block of 256
columns and, for the read-back in several threads, above 4 MiB a field; fields
given and kept (None), at creation, after set_fields and after a step.  The
state gradient is the transpose of the same map, checked by the inner product
with integers (exact in FP64).
"""
from __future__ import annotations

import itertools

import numpy as np
import pytest

from paper_1802_04243_amd import workloads as W
from paper_1802_04243_amd import workloads3 as W3

pytestmark = pytest.mark.gpu


def _same(a, b):
    for x, y in zip(a, b):
        np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("periodic", [False, True])
@pytest.mark.parametrize("nx,ny", [(24, 9), (255, 31), (257, 40), (1100, 490)])
def test_fields_2d(nx, ny, periodic):
    from oracle import oracle as O
    from paper_1802_04243_amd import sts
    rng = np.random.default_rng(nx)
    p = W.Problem(nx=nx, ny=ny, periodic=periodic, obstacle_T=1.3, p_in=1.1,
                  u_in=rng.uniform(0.9, 1.1, ny), T_in=rng.uniform(0.9, 1.1, ny),
                  obstacles=[(nx // 3, 0, nx // 3 + 4, ny // 3), (nx - 7, ny // 2, nx - 4, ny // 2)])
    g, o = sts.Solver(p), O.Oracle(p)
    _same(g.fields(), o.fields())
    f = [rng.integers(1, 50, s).astype(float) for s in g.shapes()]
    g.set_fields(*f), o.set_fields(*f)
    first = g.fields()
    _same(first, o.fields())
    g.step(1e-9, 1, 0)  # the current buffer is the other one
    cur = g.fields()
    for a in (g, o):
        a.set_fields(*[2 * x for x in f])
        a.set_fields(None, f[1], None, f[3])
    _same(g.fields(), o.fields())
    assert not np.array_equal(cur[2], g.fields()[2])
    if periodic:
        return
    # <w, M f> = <M^T w, f> plus what M adds where it does not read f
    w = [rng.integers(1, 50, s).astype(float) for s in g.shapes()]
    g.adjoint_begin(1)
    g.adjoint_seed(*w)
    grad = g.adjoint_state_grad()
    g.set_fields(*[0 * x for x in f])
    fixed = g.fields()
    exact = sum(float((a * (b - c)).sum()) for a, b, c in zip(w, first, fixed))
    assert abs(sum(float((a * b).sum()) for a, b in zip(grad, f)) - exact) <= 1e-12 * abs(exact)


@pytest.mark.parametrize("n", [(37, 9, 6), (259, 5, 4), (160, 70, 50)])
def test_fields_3d(n):
    from oracle import oracle3 as O3
    from paper_1802_04243_amd import sts3
    rng = np.random.default_rng(n[0])
    d = tuple(rng.uniform(0.05, 0.08, m) for m in n)
    for per in itertools.product((False, True), repeat=3):
        bc = tuple(W3.PERIODIC if q else (W3.WALLS if e else W3.INLET_OUTLET) for e, q in enumerate(per))
        box = W3.Box3(d=d, bc=bc, p_in=1.1)
        g, o = sts3.Solver3(box), O3.Oracle3(box)
        f = [rng.integers(1, 50, s).astype(float) for s in box.shapes()]
        for a in (g, o):
            a.set_fields(*f)
        _same(g.fields(), o.fields())
        for a in (g, o):
            a.set_fields(None, 2 * f[1], f[2], None, 3 * f[4])
        _same(g.fields(), o.fields())
