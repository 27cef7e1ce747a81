// Temporal gauge fixing (paper Sections 4 and 7): a gauge rotation Omega with
// Omega(x, 0) = 1 and Omega(x, t + 1) = Omega(x, t) U_t(x, t) makes every
// time-direction link the identity except those leaving the last time slice:
//     U'_mu(x) = Omega(x) U_mu(x) Omega(x + mu)^dagger,
//     U'_t(x, t) = 1 for t < T - 1,  U'_t(x, T - 1) = Omega(x, T - 1) U_t(x, T - 1).
// The Wilson operator is gauge covariant, M[U'] (Omega psi) = Omega M[U] psi, so
// solves in the fixed gauge return Omega x.  The dslash then skips the unit
// t-links (576 -> 480 algorithmic bytes per site in FP32 with 12-real links).
// Both steps run on the device in float64 on the canonical links; only Omega goes to the host, if it is
// asked for.  Omega up to OMEGA_KEPT bytes has a workspace of the context's.  A larger one, or one that
// the card has no room for, takes the place of the t-links themselves: Omega(t + 1) that of U_t(t), which
// only its own product reads and which ends as the identity.  So a lattice whose links fit the card can
// be fixed without a byte beside them.  16^3 x 32: 21 us for Omega, 42 us for the rotation (190 MB, 4.5
// TB/s); in place 24, 40 and 12 us for the identities.  With the links' upload from the host and Omega's way
// back 3.7 ms, against 38.9 ms when the host made the rotation (0.2 GB over the host link and 131 072 sites of
// serial 3 x 3 products).
#include "wd_core.h"

namespace wd {

// Omega along t, one work-item per (spatial site, row): row i of Omega(t + 1) is row i of Omega(t)
// times U_t(t).  Ut: the t-links, S per slice; Om: Omega(1), Omega(2), .., or Ut.  The product is serial
// in t, so the next step's link is loaded before the present one is multiplied; a wave holds the three
// rows of 21 sites, which share their links' cache lines.  Bound by that chain (0.65 us a slice).
constexpr int OMEGA_SITES = 21;
constexpr size_t OMEGA_KEPT = (size_t)64 << 20;

__global__ void __launch_bounds__(64) omega_kernel(const double* Ut, double* Om, long long S, int T)
{
    const int at = (int)threadIdx.x / 3, row = (int)threadIdx.x % 3;
    const long long s0 = (long long)blockIdx.x * OMEGA_SITES;
    const bool live = at < OMEGA_SITES && s0 + at < S;
    const long long s = s0 + (live ? at : 0);   // (work-items past the end follow the wave's first site)
    double o[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int j = 0; j < 3; ++j) o[2 * j] = j == row ? 1.0 : 0.0;
    double2 u[9], un[9];
    auto load = [&](int t, double2* v) {
        const double2* p = (const double2*)(Ut + 18 * (s + S * t));
#pragma unroll
        for (int k = 0; k < 9; ++k) v[k] = p[k];
    };
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
        __syncthreads();   // the rows of a link have read it before any of them is replaced
        if (live) {
            double2* p = (double2*)(Om + 18 * (s + S * t) + 6 * row);
#pragma unroll
            for (int j = 0; j < 3; ++j) p[j] = make_double2(o[2 * j], o[2 * j + 1]);
        }
#pragma unroll
        for (int k = 0; k < 9; ++k) u[k] = un[k];
    }
}

// U'_mu(x) = Omega(x) U_mu(x) Omega(x + mu)^dagger in place, one work-item per (mu, x, row).  The t-links
// below the last slice become exactly the identity, by unit_kernel afterwards if Omega lies in their place.
__global__ void __launch_bounds__(192) rotate_kernel(double* U, const double* Om, int X, int Y, int Z, int T)
{
    const long long S = (long long)X * Y * Z, V = S * T;
    const int row = (int)threadIdx.x % 3;
    const long long x = (long long)blockIdx.x * 64 + threadIdx.x / 3;
    const int mu = blockIdx.y;
    const int t = (int)(x / S);
    const bool unit = mu == 3 && t + 1 < T;
    const bool live = x < V && !(unit && Om == U + 18 * 3 * V);
    auto omega = [&](long long site, int i, int k) {
        if (site < S) return make_double2(i == k ? 1.0 : 0.0, 0.0);
        return *(const double2*)(Om + 18 * (site - S) + 6 * i + 2 * k);
    };
    double n[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    double* u = U + 18 * ((long long)mu * V + (live ? x : 0));
    if (live && unit) {
#pragma unroll
        for (int j = 0; j < 3; ++j) n[2 * j] = j == row ? 1.0 : 0.0;
    } else if (live) {
        long long r = x - S * t;
        const int z = (int)(r / (X * Y));
        r -= (long long)z * X * Y;
        const int y = (int)(r / X), c0 = (int)(r - (long long)y * X);
        long long xf;
        switch (mu) {
        case 0: xf = c0 + 1 == X ? x - (X - 1) : x + 1; break;
        case 1: xf = y + 1 == Y ? x - (long long)X * (Y - 1) : x + X; break;
        case 2: xf = z + 1 == Z ? x - (long long)X * Y * (Z - 1) : x + (long long)X * Y; break;
        default: xf = x - S * (T - 1); break;   // from the last slice
        }
        const double2* v = (const double2*)u;
        double a[6];
#pragma unroll
        for (int j = 0; j < 3; ++j) {   // row of Omega(x) U
            double re = 0.0, im = 0.0;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const double2 p = omega(x, row, k), q = v[3 * k + j];
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
                const double2 q = omega(xf, j, k);
                re += a[2 * k] * q.x + a[2 * k + 1] * q.y;
                im += a[2 * k + 1] * q.x - a[2 * k] * q.y;
            }
            n[2 * j] = re;
            n[2 * j + 1] = im;
        }
    }
    __syncthreads();   // the three rows of a link have read it before any of them is replaced
    if (live) {
        double2* p = (double2*)u + 3 * row;
#pragma unroll
        for (int j = 0; j < 3; ++j) p[j] = make_double2(n[2 * j], n[2 * j + 1]);
    }
}

// n complex entries of 3 x 3 identities.
__global__ void __launch_bounds__(256) unit_kernel(double2* Ut, long long n)
{
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i < n) Ut[i] = make_double2(i % 9 % 4 == 0 ? 1.0 : 0.0, 0.0);
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
    wd_context ctx = g->ctx;
    WD_HIP(hipSetDevice(ctx->device));
    double* ut = g->canon + 18 * 3 * V;
    const long long nu = S * (T - 1) * 9;   // complex entries of Omega past its first slice, the identity
    const size_t obytes = (size_t)nu * sizeof(double2);
    double* om = ut;
    void* ws;
    if (obytes <= OMEGA_KEPT && ws_get(ctx, "gaugefix.omega", obytes, &ws) == WD_OK) om = (double*)ws;
    if (om == ut) {   // (an allocation that failed is no error here)
        (void)hipGetLastError();
        clear_error();
    }
    hipLaunchKernelGGL(omega_kernel, dim3((unsigned)((S + OMEGA_SITES - 1) / OMEGA_SITES)), dim3(64), 0, ctx->stream,
                       (const double*)ut, om, S, T);
    WD_LAUNCHED();
    hipLaunchKernelGGL(rotate_kernel, dim3((unsigned)((V + 63) / 64), 4), dim3(192), 0, ctx->stream, g->canon,
                       (const double*)om, X, Y, Z, T);
    WD_LAUNCHED();
    hipError_t copied = hipSuccess;   // reported at the end: the links are left whole either way
    auto copy_out = [&] {
        if (!omega_out) return;
        for (long long i = 0; i < 18 * S; ++i) omega_out[i] = i % 18 % 8 == 0 ? 1.0 : 0.0;
        copied = hipMemcpyAsync(omega_out + 18 * S, om, obytes, hipMemcpyDeviceToHost, ctx->stream);
    };
    if (om == ut) {
        copy_out();
        hipLaunchKernelGGL(unit_kernel, dim3((unsigned)((nu + 255) / 256)), dim3(256), 0, ctx->stream, (double2*)ut, nu);
        WD_LAUNCHED();
    }
    for (int p = 0; p < 4; ++p)
        if (g->packed[p]) WD_TRY(launch_pack_gauge(ctx, g->geom, p, g->recon, g->canon, g->packed[p]));
    if (om != ut) copy_out();
    WD_HIP(hipStreamSynchronize(ctx->stream));
    WD_HIP(copied);
    g->gf = true;
    return WD_OK;
}
