"""The Poisson solver's two-sweep form (problems of at least 5 * 2^18 cells)
at the sizes where it can go wrong: ragged tiles and chunks, axes of one
cell, both boundary rules and preconditioners, against the oracle.

Tolerances as in test_gpu_poisson.py: one iteration from a given state
differs by rounding order only (the form applies M^-1 and A to x, r, p where
the oracle carries recurrences: a few ulp of the vector's largest entry), so
1e-12 of it; 1e-8 over a whole solve, with equal iteration counts.
"""
import numpy as np
import pytest

from oracle import poisson as P
from test_gpu_poisson import VEC, close, ry, smooth_rhs  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,bc,pc", [
    ((90, 131, 113), P.DIRICHLET, P.PC_STENCIL7),     # 32 x 16 tiles with tails, uneven z chunks
    ((131, 113, 90), P.PERIODIC, P.PC_STENCIL7),
    ((113, 90, 131), P.PERIODIC, P.PC_NONE),
    ((1, 1151, 1140), P.PERIODIC, P.PC_STENCIL7),     # one plane: its own neighbour
    ((1140, 1151, 1), P.DIRICHLET, P.PC_STENCIL7),
    ((1310720, 1, 1), P.PERIODIC, P.PC_STENCIL7),     # the smallest size of the form
    ((3, 2, 218454), P.PERIODIC, P.PC_STENCIL7),      # axes shorter than the halo
])
def test_two_sweep_iterations(ry, shape, bc, pc):  # noqa: F811
    b = smooth_rhs(shape, 3, sigma=1.0, mean_free=(bc == P.PERIODIC))
    g = ry.Poisson(shape, bc, pc)
    g.set_rhs(b)
    o = P.PPCG(b, bc, pc)
    vec, a, gm, i = g.state()
    assert i == 0
    for k in ("x", "r", "u", "w"):
        close(vec[k], o.v[k], 1e-13, f"initial {k}")
    for it in range(3):
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


def test_two_sweep_solve_and_restart(ry):  # noqa: F811
    shape = (97, 120, 115)
    b = smooth_rhs(shape, 7, sigma=1.5, mean_free=False)
    xo, ho = P.ppcg(b, P.DIRICHLET, P.PC_STENCIL7, eps=1e-3, max_iter=200)
    runs = []
    for mode in ("graph", "eager", "split"):
        g = ry.Poisson(shape, P.DIRICHLET, P.PC_STENCIL7)
        if mode == "eager":
            g.set_timing(True)
        g.set_rhs(b)
        if mode == "split":
            g.iterate(5)
        assert g.solve(1e-3, 200) == len(ho) - 1
        runs.append((g.download("x"), g.eps_history()))
        g.close()
    np.testing.assert_allclose(runs[0][1], ho, rtol=1e-8)
    close(runs[0][0], xo, 1e-8, "solution")
    for x, h in runs[1:]:
        np.testing.assert_array_equal(x, runs[0][0])
        np.testing.assert_array_equal(h, runs[0][1])


def test_two_sweep_initial_guess(ry):  # noqa: F811
    shape = (110, 110, 112)
    b = smooth_rhs(shape, 9, sigma=1.0)
    x0 = smooth_rhs(shape, 10, sigma=2.0)
    g = ry.Poisson(shape, P.PERIODIC, P.PC_STENCIL7)
    g.set_rhs(b, x0)
    close(g.download("r"), b - P.apply_A(x0, P.PERIODIC), 1e-13, "r0")
    g.iterate(4)
    close(g.download("r"), b - P.apply_A(g.download("x"), P.PERIODIC), 1e-12, "recursive residual")
    g.close()
