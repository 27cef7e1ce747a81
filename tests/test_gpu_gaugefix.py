"""GPU: temporal gauge fixing. The library's rotation Omega is checked
independently (unitarity; the oracle-side transform of the links gives unit
t-links on all but the last slice), and the dslash that skips the unit links
matches the FP64 oracle applied to the transformed links and, by covariance,
Omega times the oracle on the original links."""
import ctypes

import numpy as np
import pytest

import lattice_synth as ls
import oracle as orc

pytestmark = pytest.mark.gpu
BC = (1, 1, 1, -1)
DIMS = (4, 6, 4, 8)


def transform(U, Om):
    out = np.empty_like(U)
    for mu in range(4):
        ax = {0: 3, 1: 2, 2: 1, 3: 0}[mu]
        out[mu] = Om @ U[mu] @ np.conj(np.swapaxes(np.roll(Om, -1, axis=ax), -1, -2))
    return out


@pytest.fixture(scope="module")
def fixed():
    from paper_0810_5365_amd import wdirac as w
    ctx = w.Context(0)
    U = ls.gauge_field(DIMS, 0.5, 77)
    X, Y, Z, T = DIMS
    out = {}
    for recon in (12, 18):
        g = w.Gauge(ctx, DIMS, BC, recon)
        g.upload(U)
        Om = np.empty((T, Z, Y, X, 3, 3), dtype=np.complex128)
        w.wd_gauge_fix_temporal(g.handle, Om.ctypes.data)
        out[recon] = (g, Om)
    yield w, ctx, U, out
    for g, _ in out.values():
        g.close()
    ctx.close()


def test_rotation_is_su3_and_fixes_time_links(fixed):
    w, ctx, U, out = fixed
    g, Om = out[12]
    eye = np.eye(3)
    assert np.abs(Om @ np.conj(np.swapaxes(Om, -1, -2)) - eye).max() < 1e-13
    assert np.abs(np.linalg.det(Om) - 1).max() < 1e-13
    Up = transform(U, Om)
    assert np.abs(Up[3][:-1] - eye).max() < 1e-13          # t = 0 .. T-2
    assert np.abs(Up[3][-1] - eye).max() > 0.1              # the last slice keeps the Polyakov-line product


@pytest.mark.parametrize("recon", [12, 18])
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_fixed_gauge_dslash_matches_oracle(fixed, recon, prec):
    w, ctx, U, out = fixed
    g, Om = out[recon]
    p = w.PREC_BY_NAME[prec]
    tol = 1e-5 if p == w.F32 else 1e-12
    Up = transform(U, Om)
    X, Y, Z, T = DIMS
    lat = w.lattice(DIMS, BC)
    psi = ls.gaussian_complex((X * Y * Z * T // 2, 4, 3), 5, ls.STREAM_SPINOR)
    for out_sub, in_sub, ref in ((w.EVEN, w.ODD, orc.d_eo), (w.ODD, w.EVEN, orc.d_oe)):
        for dag in (0, 1):
            fin = w.pack(ctx, lat, in_sub, p, psi)
            fo = w.new_field(lat, out_sub, p)
            w.wd_dslash(g.handle, out_sub, dag, p, 1, fin.data_ptr(), fo.data_ptr())
            got = w.unpack(ctx, lat, out_sub, p, fo, psi.shape)
            assert orc.rel_l2(got, ref(Up, psi, BC, bool(dag))) < tol


def test_covariance_of_the_fixed_operator(fixed):
    """M[U'] (Omega psi) = Omega M[U] psi with M from the fixed-gauge GPU kernels."""
    w, ctx, U, out = fixed
    g, Om = out[12]
    lat = w.lattice(DIMS, BC)
    kappa = 0.124
    psi = ls.gaussian_spinor(DIMS, 9)
    rot = lambda f: np.einsum("tzyxab,tzyxsb->tzyxsa", Om, f)
    fin = w.pack(ctx, lat, w.FULL, w.F64, rot(psi))
    fo = w.new_field(lat, w.FULL, w.F64)
    w.wd_apply_M(g.handle, kappa, w.FULL, 0, w.F64, 1, fin.data_ptr(), fo.data_ptr())
    got = w.unpack(ctx, lat, w.FULL, w.F64, fo, psi.shape)
    assert orc.rel_l2(got, rot(orc.apply_m(U, psi, kappa, BC))) < 1e-12


def test_solve_in_fixed_gauge(fixed):
    import torch
    w, ctx, U, out = fixed
    g, Om = out[12]
    lat = w.lattice(DIMS, BC)
    kappa, tol = 0.124, 1e-10
    b = ls.gaussian_spinor(DIMS, 10)
    rot = lambda f: np.einsum("tzyxab,tzyxsb->tzyxsa", Om, f)
    fb = w.pack(ctx, lat, w.FULL, w.F64, rot(b))
    fx = torch.zeros_like(fb)
    prm = w.solver_params(tol=tol, maxiter=1000, sloppy=w.F32)
    info = w.WdSolverInfo()
    w.wd_wilson_solve(g.handle, kappa, ctypes.byref(prm), fb.data_ptr(), fx.data_ptr(), ctypes.byref(info))
    xp = w.unpack(ctx, lat, w.FULL, w.F64, fx, b.shape)
    x = np.einsum("tzyxba,tzyxsb->tzyxsa", np.conj(Om), xp)       # back to the original gauge
    assert orc.rel_residual(lambda v: orc.apply_m(U, v, kappa, BC), x, b) <= 1.05 * tol


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (6, 2, 4, 2), (2, 8, 6, 14), (10, 4, 6, 4)])
def test_rotation_at_the_edges_of_its_launches(dims):
    """Extents of two (every hop wraps), site counts that fill no workgroup of either kernel, and a
    second upload in between: Omega against the product of the links in numpy (T - 1 products of
    unitary matrices: below 1e-13), the float64 dslash against the oracle on the rotated links."""
    from paper_0810_5365_amd import wdirac as w
    ctx = w.Context(0)
    X, Y, Z, T = dims
    lat = w.lattice(dims, BC)
    g = w.Gauge(ctx, dims, BC, 18)
    psi = ls.gaussian_complex((X * Y * Z * T // 2, 4, 3), 6, ls.STREAM_SPINOR)
    for seed in (78, 79):
        U = ls.gauge_field(dims, 0.6, seed)
        g.upload(U)
        g.prepare(w.F64)
        Om = np.full((T, Z, Y, X, 3, 3), np.nan, dtype=np.complex128)
        w.wd_gauge_fix_temporal(g.handle, Om.ctypes.data)
        ref = [np.broadcast_to(np.eye(3, dtype=complex), U[3][0].shape)]
        for t in range(T - 1):
            ref.append(ref[t] @ U[3][t])
        assert np.abs(Om - np.stack(ref)).max() < 1e-13
        fin = w.pack(ctx, lat, w.ODD, w.F64, psi)
        fo = w.new_field(lat, w.EVEN, w.F64)
        w.wd_dslash(g.handle, w.EVEN, 0, w.F64, 1, fin.data_ptr(), fo.data_ptr())
        got = w.unpack(ctx, lat, w.EVEN, w.F64, fo, psi.shape)
        assert orc.rel_l2(got, orc.d_eo(transform(U, Om), psi, BC)) < 1e-12
    g.close()
    ctx.close()


def test_fixing_a_large_lattice_takes_no_device_memory():
    """Past 64 MB of Omega the rotation is made in the links' own place: what the card has free is the same before
    and after (a first field of the same size has loaded the kernels and what the runtime keeps for copies), Omega
    is the product of the t-links and the float64 dslash that of the rotated ones (links constant over space, random
    along t: Omega(t) is the same at every site of a slice, and the spatial links are rotated into another constant)."""
    import torch
    from paper_0810_5365_amd import wdirac as w
    dims = (32, 32, 32, 16)   # 71 MB of Omega
    X, Y, Z, T = dims
    small = ls.gauge_field((2, 2, 2, T), 0.6, 80)[:, :, 0, 0, 0]   # (4, T, 3, 3)
    U = np.ascontiguousarray(np.broadcast_to(small[:, :, None, None, None], (4, T, Z, Y, X, 3, 3)))
    om = [np.eye(3, dtype=complex)]
    for t in range(T - 1):
        om.append(om[t] @ small[3, t])
    om = np.stack(om)
    Om = np.empty((T, Z, Y, X, 3, 3), dtype=np.complex128)
    free = []
    for _ in range(2):
        ctx = w.Context(0)
        g = w.Gauge(ctx, dims, BC, 18)
        g.upload(U)
        g.prepare(w.F64)
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        w.wd_gauge_fix_temporal(g.handle, Om.ctypes.data)
        free.append((before, torch.cuda.mem_get_info()[0]))
        assert np.abs(Om - om[:, None, None, None]).max() < 1e-13
        # a spinor constant over space, hopped onto the even sites: the same lattice two sites wide gives its values
        col = ls.gaussian_complex((T, 4, 3), 81, ls.STREAM_SPINOR)
        lat = w.lattice(dims, BC)
        psi = np.broadcast_to(col[:, None, None, None], (T, Z, Y, X, 4, 3))
        fin = w.pack(ctx, lat, w.ODD, w.F64, orc.eo_split(psi, dims, 1))
        fo = w.new_field(lat, w.EVEN, w.F64)
        w.wd_dslash(g.handle, w.EVEN, 0, w.F64, 1, fin.data_ptr(), fo.data_ptr())
        got = w.unpack(ctx, lat, w.EVEN, w.F64, fo, (X * Y * Z * T // 2, 4, 3))
        d2 = (2, 2, 2, T)
        U2 = np.ascontiguousarray(np.broadcast_to(small[:, :, None, None, None], (4, T, 2, 2, 2, 3, 3)))
        Om2 = np.ascontiguousarray(np.broadcast_to(om[:, None, None, None], (T, 2, 2, 2, 3, 3)))
        psi2 = np.ascontiguousarray(np.broadcast_to(col[:, None, None, None], (T, 2, 2, 2, 4, 3)))
        ref = orc.d_eo(transform(U2, Om2), orc.eo_split(psi2, d2, 1), BC).reshape(T, -1, 4, 3)
        assert np.abs(ref - ref[:, :1]).max() < 1e-12      # constant over space, as it should be
        assert np.abs(got.reshape(T, -1, 4, 3) - ref[:, :1]).max() < 1e-12
        g.close()
        ctx.close()
    assert free[1][1] >= free[1][0]
