// Temporal gauge fixing (paper Sections 4 and 7): a gauge rotation Omega with
// Omega(x, 0) = 1 and Omega(x, t + 1) = Omega(x, t) U_t(x, t) makes every
// time-direction link the identity except those leaving the last time slice:
//     U'_mu(x) = Omega(x) U_mu(x) Omega(x + mu)^dagger,
//     U'_t(x, t) = 1 for t < T - 1,  U'_t(x, T - 1) = Omega(x, T - 1) U_t(x, T - 1).
// The Wilson operator is gauge covariant, M[U'] (Omega psi) = Omega M[U] psi, so
// solves in the fixed gauge return Omega x.  The dslash then skips the unit
// t-links (576 -> 480 algorithmic bytes per site in FP32 with 12-real links).
// Both steps run on the device in float64 on the canonical links; only Omega goes to the host, if
// it is asked for.  16^3 x 32: 21 us for Omega, 36 us for the rotation (190 MB, 5.3 TB/s); with the
// links' upload from the host and Omega's way back 3.8 ms, against 38.9 ms when the host made the
// rotation (0.2 GB over the host link and 131 072 sites of serial 3 x 3 products).
#include "wd_core.h"

namespace wd {

// Omega along t, one work-item per (spatial site, row): row i of Omega(t + 1) is row i of Omega(t)
// times U_t(t).  The product is serial in t, so the next step's link is loaded before the present
// one is multiplied; three work-items share a link's cache lines.
// Bound by that chain (0.65 us a slice).
__global__ void __launch_bounds__(64) omega_kernel(const double* __restrict__ Ut, double* __restrict__ Om, long long S, int T)
{
    const long long i = (long long)blockIdx.x * 64 + threadIdx.x;
    if (i >= 3 * S) return;
    const long long s = i / 3;
    const int row = (int)(i - 3 * s);
    double o[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int j = 0; j < 3; ++j) o[2 * j] = j == row ? 1.0 : 0.0;
    double2 u[9], un[9];
    auto load = [&](int t, double2* v) {
        const double2* p = (const double2*)(Ut + 18 * (s + S * t));
#pragma unroll
        for (int k = 0; k < 9; ++k) v[k] = p[k];
    };
    auto store = [&](int t) {
        double2* p = (double2*)(Om + 18 * (s + S * t) + 6 * row);
#pragma unroll
        for (int j = 0; j < 3; ++j) p[j] = make_double2(o[2 * j], o[2 * j + 1]);
    };
    store(0);
    load(0, u);
    for (int t = 0; t + 1 < T; ++t) {
        if (t + 2 < T) load(t + 1, un);
        double n[6];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            double re = 0.0, im = 0.0;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const double2 y = u[3 * k + j];
                re += o[2 * k] * y.x - o[2 * k + 1] * y.y;
                im += o[2 * k] * y.y + o[2 * k + 1] * y.x;
            }
            n[2 * j] = re;
            n[2 * j + 1] = im;
        }
#pragma unroll
        for (int j = 0; j < 6; ++j) o[j] = n[j];
        store(t + 1);
#pragma unroll
        for (int k = 0; k < 9; ++k) u[k] = un[k];
    }
}

// U'_mu(x) = Omega(x) U_mu(x) Omega(x + mu)^dagger in place, one work-item per (mu, x, row); the
// t-links below the last slice become exactly the identity.
__global__ void __launch_bounds__(192) rotate_kernel(double* __restrict__ U, const double* __restrict__ Om, int X, int Y, int Z,
                                                     int T)
{
    const long long S = (long long)X * Y * Z, V = S * T;
    const int row = (int)threadIdx.x % 3;
    const long long x = (long long)blockIdx.x * 64 + threadIdx.x / 3;
    const int mu = blockIdx.y;
    const bool live = x < V;
    double n[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    double* u = U + 18 * ((long long)mu * V + (live ? x : 0));
    if (live) {
        const int t = (int)(x / S);
        long long r = x - S * t;
        if (mu == 3 && t + 1 < T) {
#pragma unroll
            for (int j = 0; j < 3; ++j) n[2 * j] = j == row ? 1.0 : 0.0;
        } else {
            const int z = (int)(r / (X * Y));
            r -= (long long)z * X * Y;
            const int y = (int)(r / X), c0 = (int)(r - (long long)y * X);
            long long xf;
            switch (mu) {
            case 0: xf = c0 + 1 == X ? x - (X - 1) : x + 1; break;
            case 1: xf = y + 1 == Y ? x - (long long)X * (Y - 1) : x + X; break;
            case 2: xf = z + 1 == Z ? x - (long long)X * Y * (Z - 1) : x + (long long)X * Y; break;
            default: xf = t + 1 == T ? x - S * (T - 1) : x + S; break;
            }
            const double2* o = (const double2*)(Om + 18 * x + 6 * row);
            const double2* f = (const double2*)(Om + 18 * xf);
            const double2* v = (const double2*)u;
            double a[6];
#pragma unroll
            for (int j = 0; j < 3; ++j) {   // row of Omega(x) U
                double re = 0.0, im = 0.0;
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const double2 p = o[k], q = v[3 * k + j];
                    re += p.x * q.x - p.y * q.y;
                    im += p.x * q.y + p.y * q.x;
                }
                a[2 * j] = re;
                a[2 * j + 1] = im;
            }
#pragma unroll
            for (int j = 0; j < 3; ++j) {   // times Omega(x + mu)^dagger
                double re = 0.0, im = 0.0;
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const double2 q = f[3 * j + k];
                    re += a[2 * k] * q.x + a[2 * k + 1] * q.y;
                    im += a[2 * k + 1] * q.x - a[2 * k] * q.y;
                }
                n[2 * j] = re;
                n[2 * j + 1] = im;
            }
        }
    }
    __syncthreads();   // the three rows of a link have read it before any of them is replaced
    if (live) {
        double2* p = (double2*)u + 3 * row;
#pragma unroll
        for (int j = 0; j < 3; ++j) p[j] = make_double2(n[2 * j], n[2 * j + 1]);
    }
}

} // namespace wd

using namespace wd;

extern "C" wd_status wd_gauge_fix_temporal(wd_gauge g, double* omega_out)
{
    if (!g) {
        set_error("wd_gauge_fix_temporal: gauge is NULL");
        return WD_EINVAL;
    }
    if (!g->uploaded) {
        set_error("gauge field has not been uploaded");
        return WD_EINVAL;
    }
    const int X = g->geom.L[0], Y = g->geom.L[1], Z = g->geom.L[2], T = g->geom.L[3];
    const long long S = (long long)X * Y * Z, V = S * T;
    const size_t obytes = (size_t)V * 18 * sizeof(double);
    wd_context ctx = g->ctx;
    WD_HIP(hipSetDevice(ctx->device));
    void* om;
    WD_TRY(ws_get(ctx, "gaugefix.omega", obytes, &om));
    hipLaunchKernelGGL(omega_kernel, dim3((unsigned)((3 * S + 63) / 64)), dim3(64), 0, ctx->stream,
                       (const double*)g->canon + 18 * 3 * V, (double*)om, S, T);
    WD_LAUNCHED();
    hipLaunchKernelGGL(rotate_kernel, dim3((unsigned)((V + 63) / 64), 4), dim3(192), 0, ctx->stream, (double*)g->canon,
                       (const double*)om, X, Y, Z, T);
    WD_LAUNCHED();
    for (int p = 0; p < 4; ++p)
        if (g->packed[p]) WD_TRY(launch_pack_gauge(ctx, g->geom, p, g->recon, g->canon, g->packed[p]));
    if (omega_out) WD_HIP(hipMemcpyAsync(omega_out, om, obytes, hipMemcpyDeviceToHost, ctx->stream));
    WD_HIP(hipStreamSynchronize(ctx->stream));
    g->gf = true;
    return WD_OK;
}
