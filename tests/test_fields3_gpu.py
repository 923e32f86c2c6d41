"""Reading 3-D fields of boxes on both sides of the size up to which they are
packed into pinned memory (1 MiB of all five), all of them and some: what comes
back is a copy, so the comparison with the oracle's is for equality."""
from __future__ import annotations

import numpy as np
import pytest

from paper_1802_04243_amd import workloads3 as W3

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(4, 4, 4), (30, 30, 28), (30, 30, 29)])
def test_fields(n):
    from oracle import oracle3 as O3
    from paper_1802_04243_amd import sts, sts3
    rng = np.random.default_rng(n[2])
    box = W3.Box3(d=tuple(np.full(m, 0.1) for m in n))
    total = 8 * sum(int(np.prod(s)) for s in box.shapes())
    assert (total <= 1 << 20) == (n != (30, 30, 29))
    g, o = sts3.Solver3(box), O3.Oracle3(box)
    for k in range(2):
        f = [rng.integers(1, 50, s).astype(float) for s in box.shapes()]
        for a in (g, o):
            a.set_fields(*f)
        want = o.fields()
        for x, y in zip(g.fields(), want):
            np.testing.assert_array_equal(x, y)
        for some in ((1, 4), (0,), ()):
            out = [np.full(s, np.pi) if q in some else None for q, s in enumerate(box.shapes())]
            p = (sts._D * 5)(*[sts._ptr(a) if a is not None else None for a in out])
            sts._check(sts3.lib3().sts3_fields(g._h, p))
            for q in some:
                np.testing.assert_array_equal(out[q], want[q])
