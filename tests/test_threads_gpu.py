"""Contexts in threads of their own, small enough to record step graphs (on the
recording stream that they share): while some record, others allocate, copy,
wait and step.  Every thread's fields are bitwise those of the same steps taken
alone with plain launches."""
from __future__ import annotations

import threading

import numpy as np
import pytest

from paper_1802_04243_amd import workloads as W

pytestmark = pytest.mark.gpu


def _steps(s, p, run, seed, passes):
    s.set_fields(*W.initial_fields(p, seed))
    for k in range(40):
        s.step(run["dt"], passes, W.EXPLICIT | (W.TVD if seed % 2 else 0))
        if k % 7 == seed % 7:
            s.residuals()
    return s.fields()


def test_contexts_in_threads():
    from paper_1802_04243_amd import sts
    p, run = W.workload("channel_120x24")
    want, got, errors = {}, {}, []
    for seed in range(4):
        s = sts.Solver(p, use_torch=False)
        s.timing(True)
        want[seed] = _steps(s, p, run, seed, 4 + seed)
        s.close()

    def work(seed):
        try:
            for r in range(3):
                s = sts.Solver(p, use_torch=False)
                got[seed, r] = _steps(s, p, run, seed, 4 + seed)
                s.close()
        except Exception as e:  # noqa: BLE001 (reported below)
            errors.append((seed, e))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for (seed, r), f in got.items():
        for q, x, y in zip("uvpT", want[seed], f):
            assert np.array_equal(x, y), (seed, r, q)
