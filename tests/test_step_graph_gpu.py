"""Small grids launch a repeated step as a recorded graph: the fields and the
residuals are bitwise those of the plain launches (a solver with event timing
on takes them), in every step of a sequence that changes dt, the pass count,
the scheme and the state in between, with reads, tolerance steps and checkpoint
loads among the replays, and with two solvers on streams of their own."""
from __future__ import annotations

import numpy as np
import pytest

from paper_1802_04243_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scheme", [W.EXPLICIT | W.TVD, W.IMPLICIT | W.UPWIND,
                                    W.EXPLICIT | W.TVD | W.MIXED])
def test_replayed_steps_are_the_plain_steps(scheme):
    from paper_1802_04243_amd import sts
    p, run = W.workload("channel_120x24")
    plain, other, g = (sts.Solver(p, use_torch=False) for _ in range(3))
    plain.timing(True)
    for s, seed in ((plain, 1), (g, 1), (other, 2)):
        s.set_fields(*W.initial_fields(p, seed))
    dt = run["dt"]
    plan = [(dt, 6)] * 7 + [(dt, 5)] * 9 + [(0.5 * dt, 6)] * 4 + [(dt, 1)] * 4 + [(dt, 70)] * 4 + \
        [(dt * (1 + 0.01 * k), 4) for k in range(6)] + [(dt, 6)] * 5
    g.state_slots(1)
    plain.state_slots(1)
    for k, (d, n) in enumerate(plan):
        other.step(dt, 6, scheme)
        for s in (plain, g):
            if k == 3:
                s.state_save(0)
            if k == 12:
                s.state_load(0)
            if k == 18:
                s.step_tol(dt, 9, 1e-7, scheme)
            s.step(d, n, scheme)
        a, b = plain.residuals(), g.residuals()
        assert np.array_equal(a, b), (k, a, b)
        if k % 4 == 0:
            for x, y in zip(plain.fields(), g.fields()):
                assert np.array_equal(x, y), k
    for x, y in zip(plain.fields(), g.fields()):
        assert np.array_equal(x, y)
    for s in (plain, g, other):
        s.close()


def test_a_caller_that_records_the_stream_gets_plain_launches():
    import torch
    from paper_1802_04243_amd import sts
    p, run = W.workload("channel_120x24")
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        g, ref = sts.Solver(p), sts.Solver(p, use_torch=False)
        for s in (g, ref):
            s.set_fields(*W.initial_fields(p, 1))
            for _ in range(4):  # recorded by the library from the third on
                s.step(run["dt"], 6, W.EXPLICIT)
        st.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st):
            g.step(run["dt"], 6, W.EXPLICIT)
            g.step(run["dt"], 6, W.EXPLICIT)
        for _ in range(3):
            graph.replay()
            st.synchronize()
            for _ in range(2):
                ref.step(run["dt"], 6, W.EXPLICIT)
            assert np.array_equal(g.residuals(), ref.residuals())
            for x, y in zip(g.fields(), ref.fields()):
                assert np.array_equal(x, y)
        g.close()
        ref.close()
