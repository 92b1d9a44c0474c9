"""The launch an untuned one-level mesh or batch takes by its size, against the default
4^3-cell tile set explicitly: the same states, times and floor counts (results
do not depend on the tuning, so the tolerance is 0), the reported tuning the
default either way.  Sizes either side of the lines: up to 768 tiles, above
them with 8^3-cell tiles that hold at most a third more cells than the
4^3-cell ones, and with emptier ones.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

DEFAULT = dict(tiles_per_wg=1, persistent=0, waves_per_cu=4, batch=1, waves_per_tile=1, tile_cells=4)


@pytest.fixture(scope="module")
def ry():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_14631_amd import ry as R
    R.lib()
    return R


def box(dims, bc):
    nx, ny, nz = dims
    rng = np.random.default_rng(nx + 100 * ny + 10000 * nz)
    rho = np.exp(0.4 * rng.standard_normal((nz, ny, nx)))
    v = 0.5 * rng.standard_normal((3, nz, ny, nx))
    p = np.exp(0.3 * rng.standard_normal((nz, ny, nx)))
    lvl = max(1, int(np.ceil(np.log2(max(dims)))))
    return W.Problem("box", lvl, lvl, dims, 1.4, W.conserved(rho, v[0], v[1], v[2], p, 1.4), bc=(bc,) * 6)


def run(h, lvl):
    out = [h.tuning() == DEFAULT]
    for n in (1, 2, 5):
        h.advance(n)
    U = h.download(lvl)
    h.upload(lvl, U)
    dt = h.cfl_dt()
    h.advance(3, t_end=h.t + 2.5 * dt)
    out += [U, h.t, h.download(lvl), h.floors(), h.tuning() == DEFAULT]
    h.close()
    return out


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("dims,bc", [
    ((2, 2, 2), W.BC_PERIODIC),          # one tile, cut
    ((48, 32, 32), W.BC_PERIODIC),       # 768 tiles
    ((52, 32, 32), W.BC_PERIODIC),       # 832
    ((42, 42, 42), W.BC_OUTFLOW),        # 1,331, cut in every direction
    ((90, 54, 38), W.BC_OUTFLOW),
    ((96, 64, 10), W.BC_PERIODIC),       # 8^3-cell tiles a third emptier
    ((160, 96, 4), W.BC_PERIODIC),       # half empty: not taken
    ((84, 60, 76), W.BC_PERIODIC),       # 5,985
    ((132, 132, 20), W.BC_PERIODIC),     # 5,445: the mixed form's 8^3-cell tiles too empty
])
def test_untuned_equals_default_tuning(ry, dims, bc, precision):
    prob = box(dims, bc)
    a = run(ry.Hydro(prob, precision), prob.level_min)
    h = ry.Hydro(prob, precision)
    h.set_tuning(**DEFAULT)
    b = run(h, prob.level_min)
    assert a[0] and a[-1]
    for x, y in zip(a, b):
        np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("sides", [(6, 16, 18), (16, 32, 40, 24), (18, 18, 34, 34), (48, 6, 2, 22)])
def test_untuned_batch_equals_default_tuning(ry, sides, precision):
    # 4^3-cell tiles: 197; 1,792 (8^3-cell tiles full); 1,708 (8^3-cell tiles too empty); 1,953
    boxes = [box((s, s, s), W.BC_PERIODIC) for s in sides]
    res = []
    for tune in (False, True):
        h = ry.BatchHydro(boxes, precision)
        if tune:
            h.set_tuning(**DEFAULT)
        assert h.tuning() == DEFAULT
        for n in (1, 4, 3):
            h.run(n)
        res.append([h.download(b) for b in range(len(boxes))] + [h.box_info(b)[1] for b in range(len(boxes))])
        assert h.tuning() == DEFAULT
        h.close()
    for x, y in zip(*res):
        np.testing.assert_array_equal(x, y)


def test_untuned_then_tuned(ry):
    prob = box((52, 32, 32), W.BC_PERIODIC)
    h = ry.Hydro(prob)
    ref = ry.Hydro(prob)
    ref.set_tuning(**DEFAULT)
    for step in (3, 4, 2):
        h.advance(step)
        ref.advance(step)
        dt = h.cfl_dt()
        h.hydro_step(prob.level_min, 0.5 * dt)
        ref.hydro_step(prob.level_min, 0.5 * dt)
        np.testing.assert_array_equal(h.download(prob.level_min), ref.download(prob.level_min))
        h.set_tuning(**dict(DEFAULT, waves_per_tile=2))
    h.close()
    ref.close()


def test_untuned_without_memory_for_tables(ry, monkeypatch):
    """No memory for the 8^3-cell tile's tables: the default launch goes on;
    asked for by name they are still refused."""
    prob = box((52, 32, 32), W.BC_PERIODIC)
    table = 4 * 216 * (7 * 4 * 4)
    seen = []

    class Refusing:
        def __init__(self, torch):
            self.torch = torch

        def __getattr__(self, name):
            return getattr(self.torch, name)

        def empty(self, n, **kw):
            if n == table:
                seen.append(n)
                raise RuntimeError("no memory")
            return self.torch.empty(n, **kw)

    class Memory(ry._TorchMemory):
        def __init__(self, torch, device):
            super().__init__(torch, device)
            self.torch = Refusing(torch)

    ref = ry.Hydro(prob)
    with monkeypatch.context() as m:
        m.setattr(ry, "_TorchMemory", Memory)
        h = ry.Hydro(prob)
    assert seen
    for x in (h, ref):
        x.advance(4)
    np.testing.assert_array_equal(h.download(prob.level_min), ref.download(prob.level_min))
    with pytest.raises(ry.RyError):
        h.set_tuning(**dict(DEFAULT, waves_per_tile=8, tile_cells=8))
    h.close()
    ref.close()
