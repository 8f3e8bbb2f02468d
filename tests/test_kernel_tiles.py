"""Each kernel family at the edges of its block and tile sizes, against the oracle: every degree, meshes
of one element, meshes whose last block is partly filled, and meshes wider than a block's element
range.  The same checks run on the CPU emulation of the kernel sources (small meshes) and on the GPU.

Tolerance: 1e-12 of the largest value of each output, the parity bar of the other tests (the outputs
are sums of a few hundred terms of the size of the inputs, each within a few 2^-53 of its value)."""
import ctypes

import numpy as np
import pytest

import oracle as O
from paper_2609_10849_amd import workloads as W
from tests.test_hipemu_kernels import context, emu, omesh, ptr  # noqa: F401

PM = [(1, 0), (2, 2), (3, 2), (4, 3), (4, 4), (5, 5), (6, 5)]
SMALL = [(1, 1), (3, 2), (5, 4)]
LARGE = [(67, 31), (9, 130)]


def state(p, m, nx, ny, amp=0.3):
    L, U, Bx, By, Bz = W.random_state(nx, ny, p, m, seed=11 * p + m, domain=(0, 1.5, 0, 1.0), amp=amp)
    M = omesh(L)
    return (L, M) + tuple(O.to_primitive(M, U)) + (U, Bx, By, Bz)


def close(got, want, what, terms=0.0):
    """terms: the size of the terms that the output sums, for outputs that may cancel to nothing (the
    EC interface flux of a one-element mesh with itself)."""
    scale = max(np.abs(want).max(), terms)
    assert np.abs(got - want).max() <= 1e-12 * scale, "%s: %.2e of %.2e" % (what, np.abs(got - want).max(), scale)


def run_emulated(emu, L, opts, name, args):  # noqa: F811
    """Call an entry point of the emulated library on copies of numpy arguments; returns the copies."""
    lib, pk = emu
    h = context(lib, pk, L, opts)
    args = [np.ascontiguousarray(a).copy() if isinstance(a, np.ndarray) else a for a in args]
    r = getattr(lib, name)(h, *[ptr(a) if isinstance(a, np.ndarray) else a for a in args])
    lib.mhd25_destroy(h)
    assert r == 0, (name, r)
    return args


def run_gpu(L, opts, name, args):
    from tests._gpu import dev, host
    import paper_2609_10849_amd as pk
    S = pk.Solver.from_layout(L, opts)
    args = [dev(a) if isinstance(a, np.ndarray) else a for a in args]
    r = getattr(S.lib, name)(S.h, *[ctypes.c_void_p(a.data_ptr()) if hasattr(a, "data_ptr") else a for a in args])
    out = [host(a) if hasattr(a, "data_ptr") else a for a in args]
    S.close()
    assert r == 0, (name, r)
    return out


def check_velocity_oe(run, p, m, nx, ny):
    """The full system, and the 2D2V system (u_z = 0, B_z = 0)."""
    import paper_2609_10849_amd as pk
    L, M, rho, e, u, _, Bx, By, Bz = state(p, m, nx, ny)
    tau = 0.05  # damping factors well away from 0 and 1
    plane = u.copy()
    plane[2] = 0.0
    for r2, v, bz in ((0, u, Bz), (1, plane, np.zeros_like(Bz))):
        ru, re, _ = O.velocity_oe(M, O.Options.full(), tau, rho, v, e, Bx, By, bz)
        out = run(L, pk.Options.full(reduced_2d2v=r2), "mhd25_velocity_oe", [tau, rho, v, e, Bx, By, bz])
        close(out[2], ru, "u, 2d2v %d" % r2)
        close(out[3], re, "e, 2d2v %d" % r2)


def check_rhs_hydro(run, p, m, nx, ny):
    """Values within the series range of the logarithmic mean, values beyond it everywhere, and values
    beyond it in one element only (blocks of both kinds, and a face between them)."""
    import paper_2609_10849_amd as pk
    far = state(p, m, nx, ny, amp=0.7)
    near = state(p, m, nx, ny, amp=0.02)
    one = near[5].copy()
    one[:, near[0].K // 2] = far[5][:, near[0].K // 2]
    for U in (near[5], far[5], one):
        for iface in (0, 1):
            want = O.rhs_hydro(near[1], U, iface)
            out = run(near[0], pk.Options.make(iface_flux=iface), "mhd25_rhs_hydro", [U, np.zeros_like(U)])
            for c in range(5):
                close(out[1][c], want[c], "component %d, interface flux %d" % (c, iface),
                      np.abs(U).max() / max(near[1].hx, near[1].hy))


def check_hydro_substep(run, p, m, nx, ny):
    """The combine, statistics and reject word of the stage kernel over the three stages."""
    import paper_2609_10849_amd as pk
    L, M, _, _, _, U = state(p, m, nx, ny)[:6]
    tau = 0.02 * min(M.hx, M.hy) / (2 * p + 1)
    want = O.hydro_substep(M, O.Options.full(), U, tau)[0]
    out = run(L, pk.Options.full(), "mhd25_hydro_substep", [U, tau, None])
    for c in range(5):
        close(out[0][c], want[c], "component %d" % c)


def check_stage_map(run, p, m, nx, ny):
    """The OE sensor's tiles and the map's blocks, with OE alone, PP alone, both and neither, on states whose
    limiter acts (decisions bit for bit)."""
    import paper_2609_10849_amd as pk
    from tests.test_gpu_hydro import stressed_state
    L, U = stressed_state(nx, ny, p, seed=30 + p)
    L.m = m  # (stressed_state's own choice is of no use here)
    L.M1 = m + 1
    M = omesh(L)
    for oe, pp in ((1, 0), (0, 1), (1, 1), (0, 0)):
        tau = 0.013 if not oe else 1e-7
        want, flags, _, _ = O.hydro_stage_map(M, O.Options(oe_hydro=oe, pp=pp), U, tau)
        out = run(L, pk.Options.make(oe_hydro=oe, pp=pp), "mhd25_hydro_stage_map", [U, tau, np.zeros(L.K, np.uint8)])
        assert (out[2] == flags).all()
        for c in range(5):
            close(out[0][c], want[c], "component %d, oe %d, pp %d" % (c, oe, pp))


def check_reconstruction(run, p, m, nx, ny):
    """J and E without resistivity, with it everywhere, and with it in one element (tiles of both kinds)."""
    import paper_2609_10849_amd as pk
    L, M, rho, e, u, _, Bx, By, Bz = state(p, m, nx, ny)
    eta = np.random.default_rng(5).uniform(0.01, 0.05, M.K)
    one = np.where(np.arange(M.K) == M.K // 2, eta, 0.0)
    for et in (None, eta, one):
        want = O.reconstruct_JE(M, u, Bx, By, Bz, et)
        out = run(L, pk.Options.make(), "mhd25_reconstruct_JE", [u, Bx, By, Bz, et, np.zeros((6,) + Bx.shape)])
        for k in range(6):
            # a one-element mesh's derivatives cancel across its own faces
            close(out[5][k], want[k], "grid %d" % k, np.abs(Bx).max() / max(M.hx, M.hy))


def check_adjoint(run, p, m, nx, ny):
    """Both VJPs against the oracle's JVP (dot products of random directions and cotangents, relative to the
    sum of the terms' sizes, at least that of one derivative of B: a one-element mesh's cancel across its
    own faces), the magnetic one without resistivity, with it, and with it in one element."""
    import paper_2609_10849_amd as pk
    L, M, rho, e, u, U, Bx, By, Bz = state(p, m, nx, ny)
    rng = np.random.default_rng(7)

    def dot_test(grads, dirs, cots, outs):
        lhs = [(g * v).sum() for g, v in zip(grads, dirs)]
        rhs = [(c * o).sum() for c, o in zip(cots, outs)]
        size = max(sum(np.abs(g * v).sum() for g, v in zip(grads, dirs)), np.abs(Bx).max() / max(M.hx, M.hy))
        assert abs(sum(lhs) - sum(rhs)) <= 1e-12 * size, (sum(lhs), sum(rhs), size)

    eta = np.random.default_rng(5).uniform(0.01, 0.05, M.K)
    for et in (None, eta, np.where(np.arange(M.K) == M.K // 2, eta, 0.0)):
        ins = [u, Bx, By, Bz]
        cots = [rng.standard_normal(a.shape) for a in [e] + ins]
        dirs = [rng.standard_normal(a.shape) for a in ins]
        out = run(L, pk.Options.make(), "mhd25_rhs_magnetic_vjp",
                  [rho, u, Bx, By, Bz, et] + cots + [np.zeros_like(a) for a in ins])
        dot_test(out[-4:], dirs, cots, O.rhs_magnetic_jvp(M, rho, u, Bx, By, Bz, et, *dirs))
    for iface in (0, 1):
        cot, V = rng.standard_normal(U.shape), rng.standard_normal(U.shape)
        out = run(L, pk.Options.make(iface_flux=iface), "mhd25_rhs_hydro_vjp", [U, cot, np.zeros_like(U)])
        dot_test([out[2]], [V], [cot], [O.rhs_hydro_jvp(M, U, V, iface)])


CHECKS = [check_velocity_oe, check_rhs_hydro, check_hydro_substep, check_stage_map, check_reconstruction, check_adjoint]


@pytest.mark.parametrize("nx,ny", SMALL)
@pytest.mark.parametrize("p,m", PM)
@pytest.mark.parametrize("check", CHECKS)
def test_emulated(emu, check, p, m, nx, ny):  # noqa: F811
    check(lambda *a: run_emulated(emu, *a), p, m, nx, ny)


@pytest.mark.gpu
@pytest.mark.parametrize("nx,ny", SMALL + LARGE)
@pytest.mark.parametrize("p,m", PM)
@pytest.mark.parametrize("check", CHECKS)
def test_gpu(check, p, m, nx, ny):
    from tests._gpu import announce
    announce("%s p=%d m=%d %dx%d" % (check.__name__, p, m, nx, ny))
    check(run_gpu, p, m, nx, ny)
