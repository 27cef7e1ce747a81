"""GPU: flexible GMRES with and without the network preconditioner reaches the
requested residual (recomputed by the FP64 oracle), the fallback to the plain
solver fires on a broken network, training lowers the loss, and the committed
trained network cuts the iterations on fields it was not trained on."""
import ctypes

import numpy as np
import pytest

import lattice_synth as ls
import oracle as orc

pytestmark = pytest.mark.gpu
BC = (1, 1, 1, -1)


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_0810_5365_amd import wdirac as w
    ctx = w.Context(0)
    dims = (8, 8, 8, 16)
    U = ls.gauge_field(dims, 0.7, 5001)
    g = w.Gauge(ctx, dims, BC, 12)
    g.upload(U)
    yield w, ctx, dims, U, g
    g.close()
    ctx.close()


def _solve(w, ctx, g, dims, kappa, net_ws=None, widths=None, wprec=0, restart=16, tol=1e-10, delta=1e-4):
    import torch
    lat = w.lattice(dims, BC)
    X, Y, Z, T = dims
    b = ls.gaussian_complex((T, Z, Y, X, 4, 3), 9, ls.STREAM_SPINOR)
    fb = w.pack(ctx, lat, w.FULL, w.F64, b)
    fx = torch.zeros_like(fb)
    prm = w.solver_params(tol=tol, maxiter=3000, sloppy=w.F32, delta=delta)
    info = w.WdSolverInfo()
    if net_ws is None:
        w.wd_fgmres_solve(g.handle, kappa, ctypes.byref(prm), restart, 0, None, None, w.F32, fb.data_ptr(),
                          fx.data_ptr(), ctypes.byref(info))
    else:
        wid = (ctypes.c_int * len(widths))(*widths)
        ptrs = (ctypes.c_void_p * len(net_ws))(*[t.data_ptr() for t in net_ws])
        w.wd_fgmres_solve(g.handle, kappa, ctypes.byref(prm), restart, len(net_ws), wid, ptrs, wprec, fb.data_ptr(),
                          fx.data_ptr(), ctypes.byref(info))
    x = w.unpack(ctx, lat, w.FULL, w.F64, fx, b.shape)
    return info, orc.rel_residual(lambda v: orc.apply_m(orc_links(dims), v, kappa, BC), x, b)


_LINKS = {}


def orc_links(dims):
    return _LINKS[dims]


# delta -1: the library's default cycle reduction (1e-5)
@pytest.mark.parametrize("delta", [1e-4, -1.0])
def test_fgmres_unpreconditioned(env, delta):
    w, ctx, dims, U, g = env
    _LINKS[dims] = U
    info, res = _solve(w, ctx, g, dims, 0.1248, delta=delta)
    assert info.status == w.WD_OK and info.fell_back == 0
    assert res <= 1.05e-10, (res, info.as_dict())
    assert abs(res - info.true_resid_M) < 1e-12


def test_fgmres_long_cycle(env):
    """One cycle past 16 Krylov vectors (restart 40, cycle reduction 1e-9): the Gram-Schmidt
    passes beyond the fused two-pass kernel's range, in several vector groups per sweep."""
    w, ctx, dims, U, g = env
    _LINKS[dims] = U
    info, res = _solve(w, ctx, g, dims, 0.1248, restart=40, delta=1e-9)
    assert info.status == w.WD_OK and info.fell_back == 0
    assert res <= 1.05e-10, (res, info.as_dict())
    assert info.iters > 16 and info.cycles <= 3, info.as_dict()


@pytest.mark.parametrize("wprec,delta", [("f32", 1e-4), ("bf16", 1e-4), ("bf16", -1.0)])
def test_fgmres_with_network(env, wprec, delta):
    import torch
    from paper_0810_5365_amd import ptconv as pt
    w, ctx, dims, U, g = env
    _LINKS[dims] = U
    net = pt.PTNet((4, 8, 8, 4), w.PREC_BY_NAME[wprec])
    net.init_identity(hop=0.02)
    info, res = _solve(w, ctx, g, dims, 0.1248, net.storage(), net.widths, net.wprec, delta=delta)
    assert info.status == w.WD_OK
    assert res <= 1.05e-10, (res, info.as_dict())


def test_fgmres_long_cycles(env):
    """A cycle longer than 16 iterations takes the unfused second Gram-Schmidt pass: with a
    cycle target it cannot reach in float32 and an iteration cap of 17 the first cycle runs
    exactly 17 iterations; its update must still be the least-squares one (residual checked
    by the FP64 oracle), and a full solve with long cycles reaches the tolerance."""
    import torch
    w, ctx, dims, U, g = env
    _LINKS[dims] = U
    lat = w.lattice(dims, BC)
    X, Y, Z, T = dims
    b = ls.gaussian_complex((T, Z, Y, X, 4, 3), 11, ls.STREAM_SPINOR)
    fb = w.pack(ctx, lat, w.FULL, w.F64, b)
    for maxiter, delta in ((17, 1e-12), (3000, 1e-9)):
        fx = torch.zeros_like(fb)
        prm = w.solver_params(tol=1e-10, maxiter=maxiter, sloppy=w.F32, delta=delta)
        info = w.WdSolverInfo()
        w.wd_fgmres_solve(g.handle, 0.1248, ctypes.byref(prm), 40, 0, None, None, w.F32, fb.data_ptr(), fx.data_ptr(),
                          ctypes.byref(info), ok=(w.WD_OK, w.WD_ENOCONV))
        x = w.unpack(ctx, lat, w.FULL, w.F64, fx, b.shape)
        res = orc.rel_residual(lambda v: orc.apply_m(U, v, 0.1248, BC), x, b)
        assert info.fell_back == 0 and abs(res - info.true_resid_M) < 1e-12, info.as_dict()
        if maxiter == 17:
            assert info.iters == 17 and info.cycles == 1 and res < 1e-6, (res, info.as_dict())
        else:
            assert info.status == w.WD_OK and res <= 1.05e-10, (res, info.as_dict())


def test_fgmres_parity_skips_change_nothing(env, monkeypatch):
    """The network's first layer skips paths that read the zero odd half of (v_e, 0), the last
    computes only even sites; with bf16 weights on the matrix cores the skipped terms are exact
    zeros, so the whole solve is bit-identical to computing every path and site (both with
    float32 hidden features: the skip-free route has no bf16 ones).  With bf16 hidden features
    (the default) the solve reaches the same tolerance."""
    import torch
    from paper_0810_5365_amd import ptconv as pt, learn
    w, ctx, dims, U, g = env
    net = learn.load_net(learn.DEFAULT_WEIGHTS, w.BF16)
    lat = w.lattice(dims, BC)
    X, Y, Z, T = dims
    fb = w.pack(ctx, lat, w.FULL, w.F64, ls.gaussian_complex((T, Z, Y, X, 4, 3), 10, ls.STREAM_SPINOR))
    ws = net.storage()
    wid = (ctypes.c_int * len(net.widths))(*net.widths)
    ptrs = (ctypes.c_void_p * len(ws))(*[t.data_ptr() for t in ws])
    out = []
    for skip, f32 in (("1", "1"), ("0", "0"), ("1", "0")):
        monkeypatch.setenv("WD_PTCONV_PARITY_SKIP", skip)
        monkeypatch.setenv("WD_PTNET_F32_FEATURES", f32)
        fx = torch.zeros_like(fb)
        prm = w.solver_params(tol=1e-10, maxiter=500, sloppy=w.F32, delta=1e-4)
        info = w.WdSolverInfo()
        w.wd_fgmres_solve(g.handle, 0.1248, ctypes.byref(prm), 16, len(ws), wid, ptrs, net.wprec, fb.data_ptr(),
                          fx.data_ptr(), ctypes.byref(info))
        out.append((fx.clone(), info.iters, info.true_resid_M, info.fell_back))
    assert out[0][1] == out[1][1] and out[0][2] == out[1][2]
    assert torch.equal(out[0][0], out[1][0])
    # bf16 hidden features: a different preconditioner by rounding, the same bar
    assert out[2][3] == 0 and out[2][2] <= 1e-10 and abs(out[2][1] - out[0][1]) <= 1


def test_fgmres_falls_back_on_a_broken_network(env):
    import torch
    from paper_0810_5365_amd import ptconv as pt
    w, ctx, dims, U, g = env
    _LINKS[dims] = U
    net = pt.PTNet((4, 4), w.F32)
    with torch.no_grad():
        net.weights[0].fill_(float("nan"))
    info, res = _solve(w, ctx, g, dims, 0.1248, net.storage(), net.widths, net.wprec)
    assert info.fell_back == 1 and info.status == w.WD_OK
    assert res <= 1.05e-10


def test_training_lowers_the_loss():
    import torch
    from paper_0810_5365_amd import wdirac as w, ptconv as pt, learn
    ctx = w.Context(0)
    kappa = 0.1248
    fields = [learn.Field(ctx, (4, 4, 4, 8), 0.7, s) for s in (11, 12)]
    net = pt.PTNet((4, 8, 8, 4), w.F32)
    net.init_identity()
    before = learn.evaluate_loss(net, fields, kappa, n=4)
    hist = learn.train(net, fields, kappa, pairs_per_field=64, batch=4, epochs=2, lr=3e-3, n_null=4)
    after = learn.evaluate_loss(net, fields, kappa, n=4)
    assert np.all(np.isfinite(hist["loss"]))
    assert after < 0.7 * before, (before, after)
    for f in fields:
        f.close()
    ctx.close()



def test_trained_network_cuts_iterations_on_unseen_fields():
    """The committed network (trained on fields 5001-5008 at 16^3 x 32) on two test fields it
    has not seen: flexible GMRES with it needs at most three quarters of the iterations it
    needs without (18 -> 11 when measured), and both solves reach the FP64-checked 1e-10."""
    import torch
    from paper_0810_5365_amd import wdirac as w, learn
    ctx = w.Context(0)
    net = learn.load_net(learn.DEFAULT_WEIGHTS, w.BF16)
    dims, kappa = (16, 16, 16, 32), 0.1248
    X, Y, Z, T = dims
    lat = w.lattice(dims, BC)
    for seed in (6001, 6003):
        U = ls.gauge_field(dims, 0.7, seed)
        g = w.Gauge(ctx, dims, BC, 12)
        g.upload(U)
        b = ls.gaussian_complex((T, Z, Y, X, 4, 3), 4242, ls.STREAM_SPINOR)
        fb = w.pack(ctx, lat, w.FULL, w.F64, b)
        its = {}
        for name in ("plain", "net"):
            fx = torch.zeros_like(fb)
            prm = w.solver_params(tol=1e-10, maxiter=2000, sloppy=w.F32, delta=1e-4)
            info = w.WdSolverInfo()
            if name == "plain":
                w.wd_fgmres_solve(g.handle, kappa, ctypes.byref(prm), 16, 0, None, None, w.F32, fb.data_ptr(),
                                  fx.data_ptr(), ctypes.byref(info))
            else:
                ws = net.storage()
                wid = (ctypes.c_int * len(net.widths))(*net.widths)
                ptrs = (ctypes.c_void_p * len(ws))(*[t.data_ptr() for t in ws])
                w.wd_fgmres_solve(g.handle, kappa, ctypes.byref(prm), 16, len(ws), wid, ptrs, net.wprec,
                                  fb.data_ptr(), fx.data_ptr(), ctypes.byref(info))
            x = w.unpack(ctx, lat, w.FULL, w.F64, fx, b.shape)
            res = orc.rel_residual(lambda v: orc.apply_m(U, v, kappa, BC), x, b)
            assert info.status == w.WD_OK and info.fell_back == 0 and res <= 1.05e-10, (name, res, info.as_dict())
            its[name] = info.iters
        assert its["net"] <= 0.75 * its["plain"], its
        g.close()
    ctx.close()

@pytest.mark.parametrize("restart", [3, 4, 5, 8, 9, 20])
def test_gram_schmidt_kernel_widths(restart):
    """Flexible GMRES with cycles ending at the edges of its fused Gram-Schmidt kernels (4, 8 and 16
    vectors, and past 16 the separate passes): the oracle's residual meets the tolerance, and with a
    loose cycle reduction every width up to the restart length is used."""
    import ctypes
    import torch
    from paper_0810_5365_amd import wdirac as w
    dims, kappa, tol = (4, 6, 4, 10), 0.1248, 1e-10
    X, Y, Z, T = dims
    ctx = w.Context(0)
    U = ls.gauge_field(dims, 0.7, 7101)
    g = w.Gauge(ctx, dims, (1, 1, 1, -1), 12)
    g.upload(U)
    lat = w.lattice(dims, (1, 1, 1, -1))
    b = ls.gaussian_complex((T, Z, Y, X, 4, 3), 7102, ls.STREAM_SPINOR)
    fb = w.pack(ctx, lat, w.FULL, w.F64, b)
    fx = torch.zeros_like(fb)
    prm = w.solver_params(tol=tol, maxiter=400, sloppy=w.F32, delta=1e-8)
    info = w.WdSolverInfo()
    w.wd_fgmres_solve(g.handle, kappa, ctypes.byref(prm), restart, 0, None, None, w.F32, fb.data_ptr(), fx.data_ptr(),
                      ctypes.byref(info))
    x = w.unpack(ctx, lat, w.FULL, w.F64, fx, b.shape)
    assert orc.rel_residual(lambda v: orc.apply_m(U, v, kappa, (1, 1, 1, -1)), x, b) <= 1.05 * tol
    g.close()
    ctx.close()


def _gmres64(A, rhs, bb, tol, restart, delta):
    """Restarted GMRES in float64 by the solver's own stopping rules: per cycle the vectors it took, the residual
    over the one it began with, and how near (as a ratio) any of its estimates came to the cycle's bound."""
    r = rhs.copy()
    x = np.zeros_like(rhs)
    cycles = []
    while np.linalg.norm(r) > tol * np.sqrt(bb):
        beta = np.linalg.norm(r)
        bound = max(delta, 0.5 * tol * np.sqrt(bb) / beta)
        V, H, near = [r / beta], np.zeros((restart + 1, restart), complex), np.inf
        for j in range(restart):
            v = A(V[j])
            for _ in range(2):
                for i in range(j + 1):
                    h = np.vdot(V[i], v)
                    H[i, j] += h
                    v = v - h * V[i]
            H[j + 1, j] = np.linalg.norm(v)
            V.append(v / H[j + 1, j])
            e = np.zeros(j + 2, complex)
            e[0] = beta
            y = np.linalg.lstsq(H[:j + 2, :j + 1], e, rcond=None)[0]
            est = np.linalg.norm(e - H[:j + 2, :j + 1] @ y) / beta
            near = min(near, max(est / bound, bound / est))
            if est <= bound:
                break
        x = x + sum(c * v for c, v in zip(y, V))
        r = rhs - A(x)
        cycles.append((len(y), np.linalg.norm(r) / beta, near))
    return cycles


@pytest.mark.parametrize("restart,kappa,widest", [(3, 0.1248, 3), (4, 0.1248, 4), (5, 0.1248, 5), (8, 0.1248, 8), (9, 0.1248, 9),
                                                  (17, 0.19, 17), (20, 0.18, 20), (20, 0.2, 20)])
def test_gram_schmidt_widths_against_float64_gmres(restart, kappa, widest):
    """The float32 cycles take the iterations that float64 GMRES takes, cycle for cycle, and leave its residual: with
    up to 4, 8, 9, 16 and more than 16 vectors, never the plain solver in their place.  A float32 basis of m vectors
    is orthonormal to about m 2^-23, so the first cycle's reduction is off by at most a few of these (4e-6 allowed
    for 20), and an estimate further than 10% from the bound (checked) falls on the same side of it."""
    import ctypes
    import torch
    from paper_0810_5365_amd import wdirac as w
    dims, tol, delta, bc = (4, 6, 4, 10), 1e-10, 1e-5, (1, 1, 1, -1)
    X, Y, Z, T = dims
    U = ls.gauge_field(dims, 0.7, 7101)
    b = ls.gaussian_complex((T, Z, Y, X, 4, 3), 7102, ls.STREAM_SPINOR)
    bb = np.vdot(b, b).real
    rhs = orc.schur_source(U, b, kappa, bc).reshape(-1)
    ref = _gmres64(lambda v: orc.mhat(U, v.reshape(-1, 4, 3), kappa, bc).reshape(-1), rhs, bb, tol, restart, delta)
    assert max(n for n, _, _ in ref) == widest and min(near for _, _, near in ref) > 1.1
    ctx = w.Context(0)
    g = w.Gauge(ctx, dims, bc, 12)
    g.upload(U)
    lat = w.lattice(dims, bc)
    fb = w.pack(ctx, lat, w.FULL, w.F64, b)
    for maxiter, cycles, iters in ((ref[0][0], 1, ref[0][0]), (400, len(ref), sum(n for n, _, _ in ref))):
        fx = torch.zeros_like(fb)
        prm = w.solver_params(tol=tol, maxiter=maxiter, sloppy=w.F32, delta=delta)
        info = w.WdSolverInfo()
        w.wd_fgmres_solve(g.handle, kappa, ctypes.byref(prm), restart, 0, None, None, w.F32, fb.data_ptr(), fx.data_ptr(),
                          ctypes.byref(info), ok=(w.WD_OK, w.WD_ENOCONV))
        assert (info.fell_back, info.cycles, info.iters) == (0, cycles, iters), info.as_dict()
        if cycles == 1:
            assert abs(info.true_resid * np.sqrt(bb) / np.linalg.norm(rhs) - ref[0][1]) < 4e-6
    x = w.unpack(ctx, lat, w.FULL, w.F64, fx, b.shape)
    assert orc.rel_residual(lambda v: orc.apply_m(U, v, kappa, bc), x, b) <= 1.05 * tol
    g.close()
    ctx.close()
