"""3-D boxes of more planes than a quarter of the launch limit along z (the
constants' launch takes its groups along y there) against the FP64 oracle, with
walls and with every direction periodic.  Asserted: normwise relative
difference <= 1e-10 per field, the parity bar of the 3-D form."""
from __future__ import annotations

import numpy as np
import pytest

from paper_1802_04243_amd import workloads3 as W3

pytestmark = pytest.mark.gpu
TOL = 1e-10


@pytest.mark.parametrize("periodic", [False, True])
@pytest.mark.parametrize("scheme", [2, 1])
def test_long_box(periodic, scheme):
    from oracle import oracle3 as O3
    from paper_1802_04243_amd import sts3
    n = (5, 6, 16387)
    rng = np.random.default_rng(4)
    bc = (W3.PERIODIC,) * 3 if periodic else (W3.INLET_OUTLET, W3.WALLS, W3.WALLS)
    box = W3.Box3(d=tuple(rng.uniform(0.05, 0.08, m) for m in n), bc=bc, g=(0.1, 0.0, -0.1))
    print(f"case {n} periodic={periodic} scheme={scheme}", flush=True)
    g, o = sts3.Solver3(box), O3.Oracle3(box)
    for s in (g, o):
        s.set_fields(*W3.initial_fields3(box, 5, amp=1e-2))
        for _ in range(2):
            s.step(0.2 * box.cfl_dt(), 3, scheme)
    errs = [float(np.abs(a - b).max() / np.abs(b).max()) for a, b in zip(g.fields(), o.fields())]
    print(errs, flush=True)
    assert max(errs) <= TOL, errs
