"""A batch box whose time step underflows to zero: its state then stays what it
is while the other boxes go on (all boxes share the state buffers' parity).
The queue-fed launch, with a time-step kernel between the steps, is the
reference, bit for bit.
"""
import dataclasses

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


def hot_box(n=16, v=1e40, cfl=0.4, gamma=1.2):
    """Gas expanding into a thinner one, cells so small that the first step is
    about the smallest double; the signal speed grows until half of that."""
    shape = (n, n, n)
    left = (np.arange(n) < n // 2)[None, None, :] & np.ones(shape, bool)
    rho = np.where(left, 1.0, 1e-3)
    p = np.where(left, 1.0, 1e-6) * v * v / gamma
    z = np.zeros(shape)
    dx = 0.6 * 4.94e-324 / cfl * (3 * v)
    return W.Problem("hot", 4, 4, shape, gamma, W.conserved(rho, z, z, z, p, gamma), boxlen=dx * n, cfl=cfl,
                     bc=(W.BC_OUTFLOW,) * 6)


def test_step_of_zero(ry):
    boxes = [dataclasses.replace(W.batch_box(60, 10, 0.8, 1.2, 1.2), cfl=0.4), hot_box(),
             dataclasses.replace(W.batch_box(61, 16, 0.8, 1.2, 1.2), cfl=0.4)]
    res = []
    for t in ((1, 1, 8, 1, 1, 4), (1, 0, 4, 1, 1, 4), (1, 0, 4, 1, 4, 4), (1, 0, 4, 1, 8, 8), None):
        h = ry.BatchHydro(boxes)
        if t:
            h.set_tuning(*t)
        out, times = [], []
        for n in (1, 1, 1, 1, 1, 1, 1, 1, 1, 2, 3):
            h.run(n)
            out += [h.download(b) for b in range(3)] + [h.box_info(b)[1] for b in range(3)]
            times.append(h.box_info(1)[1])
        h.close()
        assert times[0] > 0.0 and times[-1] == times[-3] > times[1]     # it ran, and then stood still
        np.testing.assert_array_equal(out[-5], out[-11])
        res.append(out)
    for r in res[1:]:
        for x, y in zip(r, res[0]):
            np.testing.assert_array_equal(x, y)
