"""Batched boxes with boundaries of their own (periodic, outflow, and both in one
box) under every launch, the untuned one too: each box equals the same box
run alone, bit for bit (FP64 results do not depend on the tuning), and the
oracle within rounding.
"""
import dataclasses

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
P, O = W.BC_PERIODIC, W.BC_OUTFLOW


@pytest.fixture(scope="module")
def ry():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_14631_amd import ry as R
    R.lib()
    return R


def box(dims, bc, seed):
    nx, ny, nz = dims
    rng = np.random.default_rng(seed)
    rho = np.exp(0.3 * rng.standard_normal((nz, ny, nx)))
    v = 0.4 * rng.standard_normal((3, nz, ny, nx))
    p = np.exp(0.3 * rng.standard_normal((nz, ny, nx)))
    lvl = max(1, int(np.ceil(np.log2(max(dims)))))
    return W.Problem("box", lvl, lvl, dims, 1.4, W.conserved(rho, v[0], v[1], v[2], p, 1.4), bc=bc)


SMALL = [((16, 16, 16), (O,) * 6), ((16, 16, 16), (P,) * 6), ((18, 12, 10), (O, O, P, P, O, O)),
         ((8, 24, 6), (P, P, O, O, P, P)), ((2, 2, 2), (O,) * 6), ((20, 10, 34), (P, P, P, P, O, O))]
LARGE = [((32, 32, 32), (O,) * 6), ((40, 32, 24), (P, P, O, O, O, O)), ((32, 16, 32), (P,) * 6)]   # untuned: 8^3-cell tile


@pytest.mark.parametrize("boxes,tuning", [(SMALL, t) for t in
                                          (None, (1, 0, 4, 1, 1, 4), (1, 0, 4, 1, 4, 4), (4, 0, 4, 1, 1, 4),
                                           (1, 1, 8, 1, 1, 4), (1, 0, 4, 1, 8, 8), (1, 0, 4, 1, 4, 8))] +
                         [(LARGE, None), (LARGE, (1, 0, 4, 1, 8, 8))])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_boxes_with_their_own_boundaries(ry, boxes, tuning, precision):
    probs = [box(d, bc, i) for i, (d, bc) in enumerate(boxes)]
    h = ry.BatchHydro(probs, precision)
    if tuning:
        h.set_tuning(*tuning)
    h.run(3)
    h.run(2)
    for b, p in enumerate(probs):
        a = ry.Hydro(p, precision)
        a.set_tuning(*(tuning if precision == "mixed" and tuning else (1, 0, 4, 1, 1, 4)))
        a.advance(5)
        np.testing.assert_array_equal(h.download(b), a.download(p.level_min))
        assert h.box_info(b)[1] == a.t
        a.close()
    h.close()


def test_outflow_boxes_against_the_oracle(ry):
    from oracle.ryo import Oracle
    probs = [box(d, bc, 20 + i) for i, (d, bc) in enumerate(LARGE[:2])]
    h = ry.BatchHydro(probs)
    h.run(4)
    for b, p in enumerate(probs):
        o = Oracle(p)
        o.advance(4)
        ref, got = o.download(p.level_min), h.download(b)
        scale = np.maximum(np.abs(ref), 1e-3 * np.abs(ref).max(axis=1, keepdims=True))
        assert (np.abs(got - ref) / scale).max() <= 1e-11
    h.close()
