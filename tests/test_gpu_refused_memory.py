"""Refused device memory: the runtime keeps a refused hipMalloc on record, which
later successful calls do not clear; calls that can go on without the memory,
and calls after a refusal that was reported, must not meet it.  The refusals
here are the runtime's own (more memory than any card has, asked for by the
allocation hook), so the record is there as with the default allocator.
"""
import ctypes as C

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


class Memory:
    """hipMalloc, refusing the sizes of `refuse` (by hipMalloc itself)."""

    def __init__(self, ry, refuse=()):
        hip = ry.lib()
        hip.hipMalloc.argtypes = [C.POINTER(C.c_void_p), C.c_size_t]
        hip.hipFree.argtypes = [C.c_void_p]
        self.refuse, self.refused, self.log, size = set(refuse), [], [], {}

        def alloc(n, user):
            p = C.c_void_p()
            bad = n in self.refuse
            if bad:
                self.refused.append(n)
            rc = hip.hipMalloc(C.byref(p), C.c_size_t(1 << 60 if bad else n))
            self.log.append(("alloc", n))
            if rc:
                return None
            size[p.value] = n
            return p.value

        def free(p, user):
            self.log.append(("free", size.pop(p)))
            hip.hipFree(p)

        self.alloc_cb = ry.ALLOC_FN(alloc)
        self.free_cb = ry.FREE_FN(free)


def box(dims):
    rng = np.random.default_rng(sum(dims))
    rho = np.exp(0.3 * rng.standard_normal(dims[::-1]))
    v = 0.4 * rng.standard_normal((3,) + dims[::-1])
    return W.Problem("box", 6, 6, dims, 1.4, W.conserved(rho, v[0], v[1], v[2], rho, 1.4),
                     bc=(W.BC_PERIODIC,) * 6)


def tables(dims):
    return 4 * 216 * int(np.prod([-(-n // 8) for n in dims]))


def test_untuned_mesh_goes_on(ry):
    dims = (52, 32, 32)                       # untuned, takes the 8^3-cell tile where its tables fit
    prob = box(dims)
    mem = Memory(ry, [tables(dims)])
    h, ref = ry.Hydro(prob, memory=mem), ry.Hydro(prob)
    assert mem.refused
    for x in (h, ref):
        x.advance(4)
    np.testing.assert_array_equal(h.download(6), ref.download(6))
    h.close()
    ref.close()


def test_refused_tuning_leaves_a_working_mesh(ry):
    dims = (16, 16, 16)
    prob = box(dims)
    mem = Memory(ry, [tables(dims)])
    h, ref = ry.Hydro(prob, memory=mem), ry.Hydro(prob)
    with pytest.raises(ry.RyError) as e:
        h.set_tuning(1, 0, 4, 1, 8, 8)
    assert e.value.code == ry.RY_ENOMEM and mem.refused
    h.set_tuning()
    ref.set_tuning()
    for x in (h, ref):
        x.advance(3)
    np.testing.assert_array_equal(h.download(6), ref.download(6))
    h.close()
    ref.close()


def test_poisson_after_a_refused_one(ry, monkeypatch):
    shape = (12, 10, 14)
    mem = Memory(ry, [8 * 12 * 10 * 14])
    with monkeypatch.context() as m:
        m.setattr(ry, "_TorchMemory", lambda torch, device: mem)
        with pytest.raises(ry.RyError) as e:
            ry.Poisson(shape)
    assert e.value.code == ry.RY_ENOMEM and mem.refused
    b = np.random.default_rng(1).standard_normal(shape)
    g = ry.Poisson(shape, bc=ry.RY_PBC_DIRICHLET, torch_memory=False)
    g.set_rhs(b)
    assert g.solve(1e-6, 200) > 0
    g.close()


def test_regrid_takes_what_it_needs(ry):
    """A growing mesh asks for an eighth more CFL partials than it needs;
    refused, for what it needs."""
    import cases
    prob = cases.amr_blob(level_min=4, level_max=6)
    runs, part = [], None
    for refuse in (False, True):
        mem = Memory(ry)
        h = ry.Hydro(prob, memory=mem)
        # the partials follow the levels' maxima and their slots
        sizes = [n for what, n in mem.log if what == "alloc"]
        i = next(i for i in range(len(sizes) - 1) if sizes[i] == 8 * 3 and sizes[i + 1] % (8 * 3 * 64) == 0)
        old = sizes[i + 2]
        h.set_refine_param(0.25 * prob.refine_param)
        del mem.log[:]
        if refuse:
            mem.refuse.add(part)
        h.regrid()
        if not refuse:
            part = next(b[1] for a, b in zip(mem.log, mem.log[1:]) if a == ("free", old) and b[0] == "alloc")
            assert part > old
        else:
            assert mem.refused == [part]
            k = mem.log.index(("alloc", part))
            need = mem.log[k + 1][1] // 8
            assert need + need // 8 == part // 8
            mem.refuse.clear()
        h.advance(3)
        h.regrid()
        h.advance(2)
        runs.append([h.download(lv) for lv in h.levels])
        h.close()
    for a, b in zip(*runs):
        np.testing.assert_array_equal(a, b)
