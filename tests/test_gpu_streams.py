"""Contexts on the calling thread's own stream (hipStreamPerThread): the same
results bit for bit as on an ordinary stream, downloads of every size behind
the work enqueued before them.  Downloads into pinned and ordinary memory.
"""
import types

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
PER_THREAD = 2          # hipStreamPerThread's handle


@pytest.fixture(scope="module")
def ry():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_14631_amd import ry as R
    R.lib()
    return R


def on_stream(ry, monkeypatch, make, per_thread):
    import torch
    with monkeypatch.context() as m:
        if per_thread:
            m.setattr(torch.cuda, "Stream", lambda device=None: types.SimpleNamespace(cuda_stream=PER_THREAD))
        return make()


@pytest.mark.parametrize("n", [24, 64])      # downloads of 0.5 MB and 10.5 MB
def test_hydro_step_then_download(ry, monkeypatch, n):
    prob = W.random_smooth(n, seed=3, mach=0.9)
    out = []
    for per_thread in (False, True):
        h = on_stream(ry, monkeypatch, lambda: ry.Hydro(prob, torch_memory=False), per_thread)
        dt = h.cfl_dt()
        res = []
        for _ in range(3):
            h.hydro_step(prob.level_min, 0.5 * dt)      # asynchronous
            res.append(h.download(prob.level_min))
        h.close()
        out.append(res)
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("shape", [(20, 24, 36), (110, 110, 112)])    # both forms of the solver
def test_poisson_vectors(ry, monkeypatch, shape):
    b = np.random.default_rng(4).standard_normal(shape)
    b -= b.mean()
    out = []
    for per_thread in (False, True):
        g = on_stream(ry, monkeypatch, lambda: ry.Poisson(shape, torch_memory=False), per_thread)
        g.set_rhs(b)
        g.iterate(5)
        out.append([g.download(v) for v in ry.POISSON_VECTORS])
        g.close()
    for x, y in zip(*out):
        np.testing.assert_array_equal(x, y)


def test_download_into_pinned_memory(ry):
    import torch
    prob = W.random_smooth(64, seed=3, mach=0.9)
    h = ry.Hydro(prob)
    h.advance(2)
    ref = h.download(prob.level_min)
    for off in (0, 1):                        # the allocation's first byte, and inside it
        t = torch.full((ref.size + off,), -1.0, dtype=torch.float64, pin_memory=True)
        assert ry.lib().ry_download(h.ctx, prob.level_min, t.data_ptr() + 8 * off) == ry.RY_OK
        np.testing.assert_array_equal(t.numpy()[off:].reshape(ref.shape), ref)
    h.close()


@pytest.mark.parametrize("shape", [(128, 128, 128), (96, 96, 96)])    # both forms of the solver
def test_poisson_source_in_pinned_memory(ry, shape):
    """The source and the first guess are the caller's again after set_rhs."""
    import torch
    rng = np.random.default_rng(5)
    b, x0 = rng.standard_normal(shape), rng.standard_normal(shape)
    b -= b.mean()
    out = []
    for pinned in (False, True):
        g = ry.Poisson(shape)
        if pinned:
            tb, tx = torch.from_numpy(b.copy()).pin_memory(), torch.from_numpy(x0.copy()).pin_memory()
            assert ry.lib().ry_poisson_set_rhs(g.ctx, tb.data_ptr(), tx.data_ptr()) == ry.RY_OK
            tx.numpy()[::-1] = np.nan
            tb.numpy()[::-1] = np.nan
        else:
            g.set_rhs(b, x0)
        g.iterate(3)
        out.append([g.download("x"), g.download("r")])
        g.close()
    for x, y in zip(*out):
        np.testing.assert_array_equal(x, y)
