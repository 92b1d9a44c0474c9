"""The Poisson solver on thin grids (an axis of few cells): sweeps of more
workgroups than the chip holds, whose partials are summed by a launch of their
own, and long chunks, against the oracle; the time of an iteration grows with
the problem, not with its square.

Tolerances as in test_gpu_poisson.py: one iteration from a given state differs
by rounding order only (1e-12 of the vector's largest entry); 1e-8 over a
solve, with equal iteration counts.
"""
import time

import numpy as np
import pytest

from oracle import poisson as P
from test_gpu_poisson import VEC, close, ry, smooth_rhs  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,bc,pc", [
    ((1, 260, 1200), P.PERIODIC, P.PC_STENCIL7),       # 1,254 workgroups of one plane
    ((1, 1200, 260), P.DIRICHLET, P.PC_STENCIL7),      # 1,350
    ((2, 259, 1201), P.DIRICHLET, P.PC_NONE),          # 1,254 of two planes
    ((3, 1025, 1024), P.PERIODIC, P.PC_STENCIL7),      # past 5 * 2^18 cells, three planes: 4,128
    ((1, 1, 33000), P.PERIODIC, P.PC_NONE),            # 1,032, one line
    ((1, 8200, 1), P.PERIODIC, P.PC_STENCIL7),         # 1,025
    ((20001, 1, 1), P.PERIODIC, P.PC_STENCIL7),        # long: 1,429 chunks of 14 planes
    ((20001, 3, 2), P.DIRICHLET, P.PC_STENCIL7),
    ((10001, 8, 9), P.PERIODIC, P.PC_STENCIL7),        # long and a quarter full: 1,001 chunks of 10
])
def test_thin_iterations(ry, shape, bc, pc):  # noqa: F811
    b = smooth_rhs(shape, 3, sigma=1.0, mean_free=(bc == P.PERIODIC))
    g = ry.Poisson(shape, bc, pc)
    g.set_rhs(b)
    o = P.PPCG(b, bc, pc)
    vec, a, gm, i = g.state()
    for it in range(4):
        o.set_state(vec, a, gm, i)
        o.step()
        g.iterate(1)
        vec, a, gm, i = g.state()
        assert i == it + 1
        for k in VEC:
            close(vec[k], o.v[k], 1e-12, f"iteration {it + 1}, {k}")
        assert abs(a - o.alpha_prev) <= 1e-12 * abs(o.alpha_prev)
        assert abs(gm - o.gamma_prev) <= 1e-12 * abs(o.gamma_prev)
    g.close()


def test_thin_solve_and_restart(ry):  # noqa: F811
    shape = (1, 300, 1100)
    b = smooth_rhs(shape, 7, sigma=1.5, mean_free=False)
    xo, ho = P.ppcg(b, P.DIRICHLET, P.PC_STENCIL7, eps=1e-3, max_iter=400)
    runs = []
    for mode in ("graph", "eager", "split", "twice"):
        g = ry.Poisson(shape, P.DIRICHLET, P.PC_STENCIL7)
        if mode == "eager":
            g.set_timing(True)
        g.set_rhs(b)
        if mode == "split":
            g.iterate(2)                        # of four
        if mode == "twice":                 # stops at another parity, then goes on from there
            n = g.solve(1e-1, 400)
            assert 0 < n < len(ho) - 1
        assert g.solve(1e-3, 400) == len(ho) - 1
        runs.append((g.download("x"), g.eps_history()))
        g.close()
    np.testing.assert_allclose(runs[0][1], ho, rtol=1e-8)
    close(runs[0][0], xo, 1e-8, "solution")
    for x, h in runs[1:]:
        np.testing.assert_array_equal(x, runs[0][0])
        np.testing.assert_array_equal(h, runs[0][1])


@pytest.mark.parametrize("axis", [0, 1])
def test_thin_time_grows_with_the_size(ry, axis):  # noqa: F811
    """Twice the cells on one line across the tiles: twice the time (four times
    if every workgroup sums every other's partials)."""
    import torch
    times = []
    for n in ((400000, 800000) if axis == 0 else (200000, 400000)):
        shape = (1, 1, n) if axis == 0 else (1, n, 1)
        b = np.zeros(shape)
        b.flat[::2], b.flat[1::2] = 1.0, -1.0
        b += np.random.default_rng(2).standard_normal(shape)
        b -= b.mean()
        g = ry.Poisson(shape)
        g.set_rhs(b)
        best = np.inf
        for _ in range(3):
            g.iterate(15)
            torch.cuda.synchronize()
            t = time.perf_counter()
            g.iterate(63)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        times.append(best)
        g.close()
    assert times[1] < 3.0 * times[0], times
