"""Chained steps enqueued past t_end: they leave the state alone and cost a
launch, not a pass over the state.
"""
import time

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ry():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_14631_amd import ry as R
    R.lib()
    return R


@pytest.mark.parametrize("tuning", [(1, 0, 4, 1, 1, 4), (1, 0, 4, 1, 4, 4), (4, 0, 4, 1, 1, 4), (1, 0, 4, 1, 8, 8),
                                    (1, 0, 4, 1, 4, 8)])
def test_steps_past_the_end(ry, tuning):
    prob = W.random_smooth(18, seed=5, mach=0.9)
    h, ref = ry.Hydro(prob), ry.Hydro(prob)
    for x in (h, ref):
        x.set_tuning(*tuning)
    for n in (4, 5, 6, 7):                    # every phase of the rotating slots at the end
        dt = ref.cfl_dt()
        te = ref.t + 1.5 * dt
        ref.advance(2, t_end=te)
        h.advance(2 + n, t_end=te)
        assert h.t == ref.t == te
        np.testing.assert_array_equal(h.download(prob.level_min), ref.download(prob.level_min))
        assert h.cfl_dt() == ref.cfl_dt()
        h.advance(1)
        ref.advance(1)
        np.testing.assert_array_equal(h.download(prob.level_min), ref.download(prob.level_min))
    h.close()
    ref.close()


def test_steps_past_the_end_are_cheap(ry):
    """A running step of 128^3 takes about 90 us and reads and writes 168 MB;
    a launch that ends at once a few us.  With the state read: a third."""
    prob = W.random_smooth(128, seed=5, mach=0.9)
    h = ry.Hydro(prob)
    h.advance(4)

    def per_step(n, **kw):
        best = np.inf
        for _ in range(3):
            t = time.perf_counter()
            h.advance(n, **kw)
            best = min(best, time.perf_counter() - t)
        return best / n

    running = per_step(40)
    past = per_step(400, t_end=h.t)
    h.close()
    assert past < 0.15 * running, (past, running)
