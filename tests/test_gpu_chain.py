"""Steps of one-level runs whose workgroups form the time step themselves,
against the launches that have a time-step kernel between the steps (the
queue-fed tuning, and 4^3-cell tiles past the chained range): the same states
and times bit for bit over call lengths that meet every phase of the rotating
slots, the t_end clip and the steps enqueued past it, uploads and a dt query
in between.  FP64 results do not depend on the tuning, so the tolerance is 0.
"""
import dataclasses

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

K4 = (1, 0, 4, 1, 1, 4)
K8 = (1, 0, 4, 1, 8, 8)
K84 = (1, 0, 4, 1, 4, 8)
QUEUE = (1, 1, 8, 1, 1, 4)


@pytest.fixture(scope="module")
def ry():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_14631_amd import ry as R
    R.lib()
    return R


def run(ry, prob, tuning, precision="fp64", timing=False):
    h = ry.Hydro(prob, precision)
    h.set_tuning(*tuning)
    if timing:
        h.set_timing(True)
    out = []
    for n in (1, 2, 3, 7, 4):
        h.advance(n)
        out.append(h.t)
    h.cfl_dt()
    h.advance(1)
    U = h.download(prob.level_min)
    out.append(U)
    h.upload(prob.level_min, U)
    t0, dt = h.t, h.cfl_dt()
    h.advance(9, t_end=t0 + 3.5 * dt)          # ends inside the call: the last steps do nothing
    assert h.t == t0 + 3.5 * dt
    h.advance(3, t_end=t0 + 3.5 * dt)          # nothing left to do
    assert h.t == t0 + 3.5 * dt
    out += [h.download(prob.level_min), h.cfl_dt()]
    h.advance(2)
    out += [h.t, h.download(prob.level_min), h.floors()]
    h.close()
    return out


def same(a, b):
    for x, y in zip(a, b):
        np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("n,bc", [(8, W.BC_PERIODIC), (30, W.BC_OUTFLOW), (84, W.BC_PERIODIC),
                                  (104, W.BC_PERIODIC)])
def test_chained_steps_equal_unchained(ry, n, bc):
    # 104^3: 17,576 4^3-cell tiles, past the chained range
    prob = dataclasses.replace(W.random_smooth(n, seed=5, mach=0.9), bc=(bc,) * 6)
    ref = run(ry, prob, QUEUE)
    for t in (K4, K8, K84):
        same(run(ry, prob, t), ref)
    same(run(ry, prob, K8, timing=True), ref)


def test_chained_scalars_and_mixed(ry):
    prob = W.uniform(16, nscalar=2)
    a = run(ry, prob, K4)
    b = run(ry, prob, (2, 0, 4, 1, 1, 4), timing=True)
    same(a, b)
    prob = W.random_smooth(30, seed=5, mach=0.9)
    ref = run(ry, prob, QUEUE, "mixed")
    for t in (K4, K8, K84):
        same(run(ry, prob, t, "mixed"), ref)


def test_chained_batch(ry):
    boxes = [W.batch_box(60 + i, s, 0.8, 1.2) for i, s in enumerate((6, 16, 18, 24, 10))]
    res = []
    for t in (QUEUE, K4, K8, K84):
        h = ry.BatchHydro(boxes)
        h.set_tuning(*t)
        for n in (1, 2, 3, 5, 4):
            h.run(n)
        if t == K4:                            # a change of launch in the middle
            h.set_tuning(*QUEUE)
            h.run(1)
            h.set_tuning(*K8)
        else:
            h.run(1)
        h.run(2)
        res.append([h.download(b) for b in range(len(boxes))] + [h.box_info(b)[1] for b in range(len(boxes))])
        h.close()
    for r in res[1:]:
        same(r, res[0])


@pytest.mark.parametrize("n,bc", [(30, W.BC_OUTFLOW), (18, W.BC_PERIODIC), (16, W.BC_OUTFLOW), (36, W.BC_PERIODIC)])
def test_floor_census_of_one_level(ry, n, bc):
    """Floors raised into the field's range, so that a good part of all cells
    and face states meet them: the chained kernels' counts (from a thread's
    place in its tile) equal the general census and the oracle's."""
    from oracle.ryo import Oracle
    prob = dataclasses.replace(W.random_smooth(n, seed=11, mach=0.9), bc=(bc,) * 6, rho_floor=0.9, p_floor=0.8)
    o = Oracle(prob)
    o.advance(2)
    counts, states = [], []
    for t in (QUEUE, K4, (1, 0, 4, 1, 2, 4), (1, 0, 4, 1, 4, 4), (4, 0, 4, 1, 1, 4), K8, K84):
        h = ry.Hydro(prob)
        h.set_tuning(*t)
        h.advance(2)
        counts.append(h.floors())
        states.append(h.download(prob.level_min))
        h.close()
    assert counts[0] == o.floors() > n ** 3 // 10
    assert counts == [counts[0]] * len(counts)
    same(states, [states[0]] * len(states))
    m = [ry.Hydro(prob, "mixed") for _ in range(2)]
    m[0].set_tuning(*QUEUE)
    m[1].set_tuning(*K8)
    for h in m:
        h.advance(2)
    assert m[0].floors() == m[1].floors() > 0
