"""Coarse steps of several levels replayed from graphs: t_end is not part of a
graph.  Calls whose t_end changes take the same steps, to the bit, as calls on
a fresh context (which launches them one by one), and cost what calls with a
constant t_end cost.
"""
import math
import time

import numpy as np
import pytest

import cases

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ry():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_14631_amd import ry as R
    R.lib()
    return R


def test_changing_end(ry):
    prob = cases.amr_blob(level_min=3, level_max=5)
    h, ref = ry.Hydro(prob), ry.Hydro(prob)
    ref.set_timing(True)                      # no graphs
    dt = h.cfl_dt()
    ends = [math.inf] * 3 + [2.5, 1.3, 0.0, 3.0, 40.0, math.inf, 1.5]
    for n in ends:
        te = h.t + n * dt
        h.advance(4, t_end=te)
        ref.advance(4, t_end=te)
        assert h.t == ref.t
        if n < 4:
            assert h.t == te
        for lv in h.levels:
            np.testing.assert_array_equal(h.download(lv), ref.download(lv))
    h.close()
    ref.close()


def test_changing_end_costs_no_capture(ry):
    prob = cases.amr_blob(level_min=3, level_max=5)
    times = []
    for change in (0, 1):
        h = ry.Hydro(prob)
        best = np.inf
        for i in range(40):
            t = time.perf_counter()
            h.advance(4, t_end=1e9 + change * i)
            if i >= 8:
                best = min(best, time.perf_counter() - t)
        times.append(best)
        h.close()
    assert times[1] < 1.2 * times[0], times   # a capture: 1.35
