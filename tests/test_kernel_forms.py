"""What a kernel's tiles may not change.  Results do not depend on how a run's elements are split over blocks: a run's step is the same bit for bit
for every tile of the hydro stage kernel that a batch can be tuned to, and equal to the plain step's.  On the
CPU emulation of the kernel sources and on the GPU.  An element without resistivity is not touched by J, whether or
not its tile holds a resistive one."""
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


@pytest.mark.parametrize("p,m", [(2, 1), (3, 3), (4, 3)])
@pytest.mark.parametrize("r2", [0, 1])
def test_emulated_E_without_resistivity_ignores_J(emu, p, m, r2):  # noqa: F811
    """E on a 6 x 6 mesh whose element (4, 4) alone is resistive, a value of B_x near (1, 1) not a number: every node
    that element (4, 4) does not share holds what it holds without any resistivity, NaN where that is NaN."""
    lib, pk = emu
    L, U, Bx, By, Bz = W.random_state(6, 6, p, m, seed=3, domain=(0, 1.5, 0, 1.0), amp=0.3)
    u = np.ascontiguousarray(U[1:4] / U[0])
    if r2:
        u[2], Bz[:] = 0.0, 0.0
    B = m + 1
    grids = lambda a: a.reshape(6 * B, 6 * B)  # noqa: E731
    grids(Bx)[B, B] = np.nan
    eta = np.zeros(L.K)
    eta[4 * 6 + 4] = 0.02
    out = []
    for et in (None, eta):
        h = context(lib, pk, L, pk.Options.make(reduced_2d2v=r2))
        d = [np.zeros_like(a) for a in (U[0], u, Bx, By, Bz)]
        assert lib.mhd25_rhs_magnetic(h, *[ptr(np.ascontiguousarray(a)) for a in (U[0], u, Bx, By, Bz)],
                                      None if et is None else ptr(et), *[ptr(a) for a in d]) == 0
        lib.mhd25_destroy(h)
        out.append(d)
    far = np.ones((6 * B, 6 * B), bool)
    far[3 * B:, 3 * B:] = False  # rows and columns that read E at a node of element (4, 4)
    assert any(np.isnan(a).any() for a in out[0])
    for k in (2, 3, 4):  # dB_x, dB_y, dB_z
        a, b = grids(out[0][k])[far], grids(out[1][k])[far]
        assert np.array_equal(a, b, equal_nan=True), k
