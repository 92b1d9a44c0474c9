"""Chained steps with passive scalars against steps that form no time step on
the device: a loop of ry_cfl_dt and ry_hydro_step over the same mesh (the
unchained kernels, dt from the host), bit for bit, with an end inside the call
and steps enqueued past it.
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


def problem(dims, bc, ns):
    nx, ny, nz = dims
    rng = np.random.default_rng(nx + 10 * ny + 100 * nz + ns)
    rho = np.exp(0.3 * rng.standard_normal((nz, ny, nx)))
    v = 0.4 * rng.standard_normal((3, nz, ny, nx))
    p = np.exp(0.3 * rng.standard_normal((nz, ny, nx)))
    s = rng.random((ns, nz, ny, nx))
    U = np.concatenate([W.conserved(rho, v[0], v[1], v[2], p, 1.4), rho[None] * s], axis=0)
    lvl = int(np.ceil(np.log2(max(dims))))
    return W.Problem("box", lvl, lvl, dims, 1.4, U, bc=(bc,) * 6, nscalar=ns)


def host_steps(h, n, t_end=np.inf):
    """n steps of the CFL rule, clipped to t_end, from the host."""
    for _ in range(n):
        dt = h.cfl_dt()
        last = dt >= t_end - h.t
        if last:
            dt = t_end - h.t
        if not dt > 0.0:
            break
        h.hydro_step(h.prob.level_min, dt)
        h.t = t_end if last else h.t + dt


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("tuning", [None, (1, 0, 4, 1, 1, 4), (2, 0, 4, 1, 1, 4)])
@pytest.mark.parametrize("dims,bc,ns", [((16, 16, 16), W.BC_PERIODIC, 2), ((18, 10, 14), W.BC_OUTFLOW, 1),
                                        ((22, 6, 30), W.BC_PERIODIC, 4)])
def test_chained_scalars_equal_host_steps(ry, dims, bc, ns, tuning, precision):
    prob = problem(dims, bc, ns)
    h, ref = ry.Hydro(prob, precision), ry.Hydro(prob, precision)
    if tuning:
        for x in (h, ref):
            try:
                x.set_tuning(*tuning)
            except ry.RyError:
                pytest.skip("no kernel with passive scalars for this launch")
    lv = prob.level_min
    for n in (1, 3, 6):
        h.advance(n)
        host_steps(ref, n)
        assert h.t == ref.t
        np.testing.assert_array_equal(h.download(lv), ref.download(lv))
    te = h.t + 2.5 * ref.cfl_dt()
    h.advance(7, t_end=te)
    host_steps(ref, 7, t_end=te)
    assert h.t == ref.t == te
    np.testing.assert_array_equal(h.download(lv), ref.download(lv))
    h.advance(2)
    host_steps(ref, 2)
    np.testing.assert_array_equal(h.download(lv), ref.download(lv))
    assert h.cfl_dt() == ref.cfl_dt()
    h.close()
    ref.close()


def test_chained_tiles_equal_host_steps(ry):
    prob = dataclasses.replace(W.random_smooth(30, seed=5, mach=0.9), bc=(W.BC_OUTFLOW,) * 6)
    lv = prob.level_min
    ref = ry.Hydro(prob)
    ref.set_tuning(1, 1, 8, 1, 1, 4)
    host_steps(ref, 5)
    for t in (None, (1, 0, 4, 1, 1, 4), (1, 0, 4, 1, 4, 4), (1, 0, 4, 1, 8, 8), (1, 0, 4, 1, 4, 8)):
        h = ry.Hydro(prob)
        if t:
            h.set_tuning(*t)
        h.advance(5)
        assert h.t == ref.t
        np.testing.assert_array_equal(h.download(lv), ref.download(lv))
        h.close()
    ref.close()
