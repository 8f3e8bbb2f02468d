"""Results do not depend on how a run's elements are split over blocks: a run's step is the same bit for bit
for every tile of the hydro stage kernel that a batch can be tuned to, and equal to the plain step's.  On the
CPU emulation of the kernel sources and on the GPU."""
import ctypes

import numpy as np
import pytest

from paper_2609_10849_amd import workloads as W
from tests.test_hipemu_kernels import context, emu, ptr  # noqa: F401


def rough_elements(nx, ny, p, m):
    """A nearly constant state whose element K // 3 holds values far beyond each other's size (blocks, waves and
    faces of both kinds)."""
    L, U, Bx, By, Bz = W.random_state(nx, ny, p, m, seed=5, domain=(0, 1.5, 0, 1.0), amp=0.02)
    far = W.random_state(nx, ny, p, m, seed=6, domain=(0, 1.5, 0, 1.0), amp=0.7)[1]
    U[:, L.K // 3] = far[:, L.K // 3]
    return L, [U, Bx, By, Bz]


STEP = 1e-4


@pytest.mark.parametrize("p,m", [(2, 1), (4, 3), (5, 5)])
def test_emulated_step_is_the_same_for_every_tile(emu, p, m):  # noqa: F811
    lib, pk = emu
    L, st = rough_elements(8, 4, p, m)
    opts = pk.Options.full()
    one = [np.ascontiguousarray(a.copy()) for a in st]
    h = context(lib, pk, L, opts)
    assert lib.mhd25_strang_step(h, *[ptr(a) for a in one], STEP, None) == 0
    lib.mhd25_destroy(h)
    desc = (pk.MeshDesc * 1)(pk.MeshDesc(L.nx, L.ny, L.x0, L.x1, L.y0, L.y1, L.p, L.m, L.gamma))
    b = ctypes.c_void_p()
    assert lib.mhd25_batch_create(desc, 1, ctypes.byref(opts), None, ctypes.byref(b)) == 0
    for bs in (128, 256):
        assert lib.mhd25_batch_set_tuning(b, 0, 0, bs) == 0
        got = [np.ascontiguousarray(a.copy()) for a in st]
        arr = [(ctypes.c_void_p * 1)(a.ctypes.data) for a in got]
        assert lib.mhd25_batch_strang_step(b, *arr, (ctypes.c_double * 1)(STEP), None) == 0
        for a, r in zip(got, one):
            assert (a == r).all(), (bs, np.abs(a - r).max())
    lib.mhd25_batch_destroy(b)


@pytest.mark.gpu
@pytest.mark.parametrize("nx,ny", [(20, 12), (90, 61)])
@pytest.mark.parametrize("p,m", [(1, 1), (2, 1), (3, 3), (4, 3), (5, 5), (6, 5)])
def test_gpu_step_is_the_same_for_every_tile(p, m, nx, ny):
    import paper_2609_10849_amd as pk
    from tests._gpu import announce, dev, host
    announce("every tile p=%d m=%d %dx%d" % (p, m, nx, ny))
    L, st = rough_elements(nx, ny, p, m)
    opts = pk.Options.full()
    one = [dev(a) for a in st]
    S = pk.Solver.from_layout(L, opts)
    assert S.strang_step(*one, STEP)[0] == 0
    B = pk.Batch([L], opts)
    for bs in (128, 256):
        B.set_tuning(hydro_bs=bs)
        got = [dev(a) for a in st]
        assert B.strang_step(*[[a] for a in got], [STEP])[0] == 0
        for a, r in zip(got, one):
            assert (host(a) == host(r)).all(), bs
    B.close()
    S.close()
