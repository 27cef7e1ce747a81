// The per-site body of the Wilson hopping term on one parity (paper
// Section 4: one work-item per site of the even or odd sub-lattice), shared
// by the plain launch (dslash.hip) and the persistent batch (batch.hip).
//
// Per output site x of parity par and each of the 8 directions:
//   1. fetch the neighbour spinor psi(x +- mu) (24 reals, structure-of-arrays),
//   2. project it to a half spinor with (1 -+ gamma_mu)  (12 reals, 12 flops),
//   3. fetch the link U_mu(x) or U_mu(x - mu) (12 reals + row-2 rebuild, or 18),
//   4. multiply both colour triplets by U or U^dagger  (132 flops),
//   5. expand to 4 spin rows and accumulate  (24 flops; 7 of 8 counted),
// then store, optionally fused with out = a x + b D in.  1320 flops per site.
#pragma once

#include "wd_core.h"

namespace wd {

// Keeps each direction's loads behind the previous direction's arithmetic.
// Without it the compiler hoists all 72 loads of the 8 directions to the top
// of the kernel, needs > 256 VGPRs and runs one wave per SIMD; with it the
// kernel fits in < 100 VGPRs and latency is hidden by occupancy instead.
template <typename T> __device__ __forceinline__ void order_fence(T* a)
{
#pragma unroll
    for (int k = 0; k < 24; k += 8)
        asm volatile("" : "+v"(a[k]), "+v"(a[k + 1]), "+v"(a[k + 2]), "+v"(a[k + 3]), "+v"(a[k + 4]), "+v"(a[k + 5]),
                     "+v"(a[k + 6]), "+v"(a[k + 7])::"memory");
}

struct DslashArgs {
    const char* gauge;
    const char* in;
    char* out;
    const char* x;
    long long in_stride, out_stride, x_stride;
    double a, b;
    Geom g;
    int par;
    int remap;
    int rhs_inner;   // > 1: that many rhs interleaved with the site tiles on grid x
    int zb;          // > 0: z-blocked site traversal with this block depth (divides Z)
    int gf;          // links in temporal gauge: U_t = 1 except on the last time slice
    FastDiv dzb, dt; // division by zb and by T for the blocked traversal
    FastDiv drhs;    // division by the number of rhs for the interleaved order
    double* red;     // per-workgroup partial sums of a fused reduction (dslash_red.hip)
    const char* y;   // the other operand of the fused <y, out>
    const double* coef;   // RED_CGR: the step length alpha, in device memory
    int xnt;              // fused update: load x non-temporally
};

// Kernel arguments for a launch of the hopping term with launch shape tp (dslash.hip).
wd_status dslash_setup(const Geom& g, const DslashCall& c, const TuneParam& tp, DslashArgs* A);
// The launch shape with what it leaves to the rules (link loads, waves per group) settled for this call.
TuneParam dslash_shape(const Geom& g, const DslashCall& c, const TuneParam& tp);

// v <- the values that storing v at 16-bit precision and loading it back gives (the store's
// scale and rounding, repeated).
template <int P> __device__ __forceinline__ void quant_roundtrip(float* v)
{
    float s = 0.0f;
#pragma unroll
    for (int k = 0; k < 24; ++k) s = fmaxf(s, fabsf(v[k]));
    const float inv = s > 0.0f ? 1.0f / s : 0.0f;
#pragma unroll
    for (int k = 0; k < 24; ++k) v[k] = h2f<P>(f2h<P>(v[k] * inv)) * s;
}

// Reductions a fused-update launch (out = a x + b D in) can sum in its epilogue, per site in
// float64 from the stored values:
//   RED_NORM  |out|^2                        -> r[0]
//   RED_XDOT  <out, x>, |out|^2              -> r[0] + i r[1], r[2]
//   RED_YDOT  <y, out> (y = A.y), |out|^2    -> r[0] + i r[1], r[2]
//   RED_RESID out = y - (a x + b D in), |out|^2 -> r[0]   (a residual, stored instead)
//   RED_YDIFF |y - out|^2                    -> r[0]
//   RED_RESLO as RED_RESID, the residual stored in float32 -> r[0]
//   RED_CGR   r -= alpha out (r = A.out at the accumulation precision), |r|^2 -> r[0]
template <typename T>
__device__ __forceinline__ void site_dot_norm(const T* a, const T* b, const T* o, double* r)
{
    double re = 0.0, im = 0.0, nn = 0.0;
#pragma unroll
    for (int i = 0; i < 12; ++i) {
        const double ar = a[2 * i], ai = a[2 * i + 1], br = b[2 * i], bi = b[2 * i + 1];
        re += ar * br + ai * bi;
        im += ar * bi - ai * br;
    }
#pragma unroll
    for (int k = 0; k < 24; ++k) nn += (double)o[k] * (double)o[k];
    r[0] = re;
    r[1] = im;
    r[2] = nn;
}

// Site order index i -> checkerboard index and coordinates of the z-blocked
// traversal: i = xh + Xh (y + Y (zi + zb (t + T b))), z = b zb + zi.  Sites of
// one z-block are walked through all t before the next block, so the slices
// t - 1, t, t + 1 of a block that the stencil reads stay close in time.
__device__ __forceinline__ uint32_t zblock_site(const DslashArgs& A, uint32_t i, int c[4])
{
    const Geom& g = A.g;
    const uint32_t q1 = fdiv(i, g.dxh);
    const uint32_t xh = i - q1 * (uint32_t)g.Xh;
    const uint32_t q2 = fdiv(q1, g.dy);
    const uint32_t y = q1 - q2 * (uint32_t)g.L[1];
    const uint32_t q3 = fdiv(q2, A.dzb);
    const uint32_t zi = q2 - q3 * (uint32_t)A.zb;
    const uint32_t b = fdiv(q3, A.dt);
    const uint32_t t = q3 - b * (uint32_t)g.L[3];
    const uint32_t z = b * (uint32_t)A.zb + zi;
    c[1] = (int)y;
    c[2] = (int)z;
    c[3] = (int)t;
    c[0] = (int)(2 * xh + ((A.par + y + z + t) & 1));
    return xh + (uint32_t)g.Xh * (y + (uint32_t)g.L[1] * (z + (uint32_t)g.L[2] * t));
}

// In temporal gauge the t-link of a hop is the identity unless the hop leaves
// the last time slice (forward from t = T - 1, backward into t = 0), so it is
// neither loaded nor multiplied (paper Sections 4 and 7: the gauge-fixing trick).
template <int MU, bool FWD>
__device__ __forceinline__ bool unit_link(const DslashArgs& A, const int c[4])
{
    if constexpr (MU != 3) return false;
    else return A.gf && (FWD ? c[3] != A.g.L[3] - 1 : c[3] != 0);
}

// Loads of direction D: the link (U_mu(x) forward, U_mu(x - mu) backward)
// and the neighbour spinor.
template <int D, bool NT, typename X>
__device__ __forceinline__ void hop_load(const DslashArgs& A, uint32_t cb, const int c[4], const char* in, size_t gbytes,
                                         X& x)
{
    constexpr int MU = D >> 1;
    constexpr bool FWD = (D & 1) == 0;
    const uint32_t nb = neighbour<MU, FWD>(A.g, cb, c);
    const int lpar = FWD ? A.par : 1 - A.par;
    const uint32_t lcb = FWD ? cb : nb;
    if (!unit_link<MU, FWD>(A, c)) x.template load_link<NT>(A.gauge + (size_t)(2 * MU + lpar) * gbytes, A.g.ps, lcb);
    x.load_spinor(in, A.g.ps, nb);
}

// Direction D's half spinor: project, boundary sign, colour multiply.
template <int D, bool DAG, typename X, typename T>
__device__ __forceinline__ void hop_half_spinor(const DslashArgs& A, const int c[4], const X& x, T* w)
{
    constexpr int MU = D >> 1;
    constexpr bool FWD = (D & 1) == 0;
    // D: (1 - gamma) on the forward hop, (1 + gamma) on the backward hop; D^dagger swaps them
    constexpr int S = (FWD != DAG) ? -1 : 1;
    T h[12], psi[24];
    x.spinor(psi);
    project<MU, S>(psi, h);
    T sg;
    if constexpr (sizeof(T) == 8) sg = on_boundary<MU, FWD>(A.g, c) ? A.g.bcd[MU] : 1.0;
    else sg = on_boundary<MU, FWD>(A.g, c) ? A.g.bcf[MU] : 1.0f;
#pragma unroll
    for (int k = 0; k < 12; ++k) h[k] *= sg;
    if (unit_link<MU, FWD>(A, c)) {
#pragma unroll
        for (int k = 0; k < 12; ++k) w[k] = h[k];
    } else {
        T u[18];
        x.link(u);
        su3_mul<!FWD>(u, h, w);
    }
}

template <int D, bool DAG, typename T> __device__ __forceinline__ void hop_accumulate(T* acc, const T* w)
{
    constexpr int S = (((D & 1) == 0) != DAG) ? -1 : 1;
    accumulate<(D >> 1), S>(acc, w);
}

template <int D, bool DAG, typename X, typename T>
__device__ __forceinline__ void hop_compute(const DslashArgs& A, const int c[4], const X& x, T* acc)
{
    T w[12];
    hop_half_spinor<D, DAG>(A, c, x, w);
    hop_accumulate<D, DAG>(acc, w);
}

// One direction at a time: its loads, then its arithmetic, then a fence.
template <int D, typename X, bool DAG, bool NT, typename T>
__device__ __forceinline__ void hop(const DslashArgs& A, uint32_t cb, const int c[4], const char* in, size_t gbytes,
                                    T* acc)
{
    X x;
    hop_load<D, NT>(A, cb, c, in, gbytes, x);
    hop_compute<D, DAG>(A, c, x, acc);
    order_fence(acc);
}

// Software-pipelined: the loads of direction D + 1 are issued before the
// arithmetic of direction D, so each wave keeps two directions in flight.
template <int D, bool DAG, bool NT, typename X, typename T>
__device__ __forceinline__ void hop_pipelined(const DslashArgs& A, uint32_t cb, const int c[4], const char* in,
                                              size_t gbytes, T* acc, X& cur, X& nxt)
{
    if constexpr (D + 1 < 8) hop_load<D + 1, NT>(A, cb, c, in, gbytes, nxt);
    asm volatile("" ::: "memory");
    hop_compute<D, DAG>(A, c, cur, acc);
    order_fence(acc);
}

// What follows the sum over directions: out = a x + b D in, stored.  RED > 0 (with XPAY): the site's
// values of that fused reduction go to red[0 .. 3).  The output is stored first, so the reduction
// adds no registers to the store.  XPRE: x has been loaded already.
template <int P, bool XPAY, int RED, bool XPRE, typename T>
__device__ __forceinline__ void dslash_finish(const DslashArgs& A, uint32_t cb, int rhs, T* acc, double* red,
                                              const T* xpre = nullptr)
{
    const T b = (T)A.b;
    T xv[24];
    if constexpr (XPAY) {
        if constexpr (XPRE) {
#pragma unroll
            for (int k = 0; k < 24; ++k) xv[k] = xpre[k];
        } else {
            // x is read once, at the site written: a non-temporal load leaves the last-level cache
            // to the fields the next launch reads (measured: 0.75% on the Mhat^dag Mhat step)
            if (A.xnt) SpinorIO<P>::load_nt(A.x + rhs * A.x_stride, A.g.ps, cb, xv);
            else SpinorIO<P>::load(A.x + rhs * A.x_stride, A.g.ps, cb, xv);
        }
        const T a = (T)A.a;
        // (spelt out: left to the compiler, which product is fused depends on where x was loaded)
#pragma unroll
        for (int k = 0; k < 24; ++k) acc[k] = fma(b, acc[k], a * xv[k]);
    } else {
#pragma unroll
        for (int k = 0; k < 24; ++k) acc[k] *= b;
    }
    if constexpr (RED == RED_CGR) {
        // r -= alpha (a x + b D in) at the accumulation precision; the operator's own result
        // is never stored
        constexpr int PA = P == P_F64 ? P_F64 : P_F32;
        using TA = typename RealOf<PA>::T;
        char* rp = A.out + rhs * A.out_stride;
        TA rv[24];
        SpinorIO<PA>::load(rp, A.g.ps, cb, rv);
        const TA al = (TA)A.coef[0];
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < 24; ++k) {
            rv[k] -= al * (TA)acc[k];
            s += (double)rv[k] * (double)rv[k];
        }
        SpinorIO<PA>::store(rp, A.g.ps, cb, rv);
        red[0] = s;
        return;
    }
    if constexpr (RED == RED_RESLO) {
        // the float64 residual y - (a x + b D in), its norm taken before it is stored in float32
        T yv[24];
        float lo[24];
        SpinorIO<P>::load(A.y + rhs * A.out_stride, A.g.ps, cb, yv);
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < 24; ++k) {
            const double d = (double)yv[k] - (double)acc[k];
            s += d * d;
            lo[k] = (float)d;
        }
        SpinorIO<P_F32>::store(A.out + rhs * A.out_stride, A.g.ps, cb, lo);
        red[0] = s;
        return;
    }
    if constexpr (RED == 4) {   // the residual y - (a x + b D in) is what is stored
        T yv[24];
        SpinorIO<P>::load(A.y + rhs * A.out_stride, A.g.ps, cb, yv);
#pragma unroll
        for (int k = 0; k < 24; ++k) acc[k] = yv[k] - acc[k];
    }
    SpinorIO<P>::store(A.out + rhs * A.out_stride, A.g.ps, cb, acc);
    if constexpr (RED > 0) {
        // the reduction sees the values a later load returns (16-bit: the codes times the scale)
        if constexpr (P == P_F16 || P == P_BF16) quant_roundtrip<P>(acc);
        if constexpr (RED == 1 || RED == 4) {
            double s = 0.0;
#pragma unroll
            for (int k = 0; k < 24; ++k) s += (double)acc[k] * (double)acc[k];
            red[0] = s;
        } else if constexpr (RED == 2) {
            site_dot_norm(acc, xv, acc, red);
        } else if constexpr (RED == 3) {
            T yv[24];
            SpinorIO<P>::load(A.y + rhs * A.out_stride, A.g.ps, cb, yv);
            site_dot_norm(yv, acc, acc, red);
        } else {
            T yv[24];
            SpinorIO<P>::load(A.y + rhs * A.out_stride, A.g.ps, cb, yv);
            double s = 0.0;
#pragma unroll
            for (int k = 0; k < 24; ++k) {
                const double d = (double)yv[k] - (double)acc[k];
                s += d * d;
            }
            red[0] = s;
        }
    }
}

template <int P, int R, bool DAG, bool XPAY, bool NT, bool PF, int RED = 0, typename X = HopRaw<P, R>>
__device__ __forceinline__ void dslash_site(const DslashArgs& A, uint32_t cb, const int c[4], int rhs,
                                            double* red = nullptr)
{
    using T = typename RealOf<P>::T;
    const size_t gbytes = link_site_bytes(P, R) * (size_t)A.g.ps;
    const char* in = A.in + rhs * A.in_stride;
    T acc[24];
#pragma unroll
    for (int k = 0; k < 24; ++k) acc[k] = 0;
    if constexpr (PF) {
        X ra, rb;
        hop_load<0, NT>(A, cb, c, in, gbytes, ra);
        hop_pipelined<0, DAG, NT>(A, cb, c, in, gbytes, acc, ra, rb);
        hop_pipelined<1, DAG, NT>(A, cb, c, in, gbytes, acc, rb, ra);
        hop_pipelined<2, DAG, NT>(A, cb, c, in, gbytes, acc, ra, rb);
        hop_pipelined<3, DAG, NT>(A, cb, c, in, gbytes, acc, rb, ra);
        hop_pipelined<4, DAG, NT>(A, cb, c, in, gbytes, acc, ra, rb);
        hop_pipelined<5, DAG, NT>(A, cb, c, in, gbytes, acc, rb, ra);
        hop_pipelined<6, DAG, NT>(A, cb, c, in, gbytes, acc, ra, rb);
        hop_pipelined<7, DAG, NT>(A, cb, c, in, gbytes, acc, rb, ra);
    } else {
        hop<0, X, DAG, NT>(A, cb, c, in, gbytes, acc);
        hop<1, X, DAG, NT>(A, cb, c, in, gbytes, acc);
        hop<2, X, DAG, NT>(A, cb, c, in, gbytes, acc);
        hop<3, X, DAG, NT>(A, cb, c, in, gbytes, acc);
        hop<4, X, DAG, NT>(A, cb, c, in, gbytes, acc);
        hop<5, X, DAG, NT>(A, cb, c, in, gbytes, acc);
        hop<6, X, DAG, NT>(A, cb, c, in, gbytes, acc);
        hop<7, X, DAG, NT>(A, cb, c, in, gbytes, acc);
    }
    dslash_finish<P, XPAY, RED, false>(A, cb, rhs, acc, red);
}

template <int P, int R, bool DAG, bool XPAY, bool NT, bool PF, int RED = 0, typename X = HopRaw<P, R>>
__device__ __forceinline__ void dslash_site(const DslashArgs& A, uint32_t cb, int rhs, double* red = nullptr)
{
    int c[4];
    cb_coords(A.g, cb, A.par, c);
    dslash_site<P, R, DAG, XPAY, NT, PF, RED, X>(A, cb, c, rhs, red);
}

// The i-th output site in the launch's site order.  The 16-bit kernels join the two orders before
// the body (90 -> 80 registers in F16); the wide ones keep a body for each (joined, they measured 0.5%
// slower on the 32^3 x 64 F32 step).
template <int P, int R, bool DAG, bool XPAY, bool NT, bool PF, int RED = 0>
__device__ __forceinline__ void dslash_at(const DslashArgs& A, uint32_t i, int rhs, double* red = nullptr)
{
    int c[4];
    if constexpr (P == P_F16 || P == P_BF16) {
        uint32_t cb = i;
        if (A.zb > 0) cb = zblock_site(A, i, c);
        else cb_coords(A.g, i, A.par, c);
        dslash_site<P, R, DAG, XPAY, NT, PF, RED>(A, cb, c, rhs, red);
    } else if (A.zb > 0) {
        const uint32_t cb = zblock_site(A, i, c);
        dslash_site<P, R, DAG, XPAY, NT, PF, RED>(A, cb, c, rhs, red);
    } else {
        dslash_site<P, R, DAG, XPAY, NT, PF, RED>(A, i, rhs, red);
    }
}

// A workgroup of four waves covers 64 output sites, wave mu taking the two hops along mu: all of a
// site's loads are in flight at once instead of two directions of eight, and a lattice of N groups
// of 64 sites runs 4 N waves.  The half spinors go through LDS and the first wave sums them in the
// order of dslash_site, so the results are the same bit for bit.  Only the first wave returns true
// (for sites on the lattice), with the site finished.
constexpr size_t dslash_split_lds(int P) { return 8 * 12 * 64 * (P == P_F64 ? sizeof(double) : sizeof(float)); }

template <int MU, int P, int R, bool DAG, bool NT>
__device__ __forceinline__ void split_hops(const DslashArgs& A, uint32_t cb, const int c[4], const char* in,
                                           float4* lds, int lane)
{
    using T = typename RealOf<P>::T;
    constexpr int NV = 12 * sizeof(T) / 16;   // 16-byte words of a half spinor
    const size_t gbytes = link_site_bytes(P, R) * (size_t)A.g.ps;
    HopRaw<P, R> f, b;
    hop_load<2 * MU, NT>(A, cb, c, in, gbytes, f);
    hop_load<2 * MU + 1, NT>(A, cb, c, in, gbytes, b);
    T w[12];
    float4 q[NV];
    hop_half_spinor<2 * MU, DAG>(A, c, f, w);
    __builtin_memcpy(q, w, sizeof(w));
#pragma unroll
    for (int k = 0; k < NV; ++k) lds[(2 * MU * NV + k) * 64 + lane] = q[k];
    hop_half_spinor<2 * MU + 1, DAG>(A, c, b, w);
    __builtin_memcpy(q, w, sizeof(w));
#pragma unroll
    for (int k = 0; k < NV; ++k) lds[((2 * MU + 1) * NV + k) * 64 + lane] = q[k];
}

template <int D, int P, bool DAG, typename T>
__device__ __forceinline__ void split_sum(const float4* lds, int lane, T* acc)
{
    constexpr int NV = 12 * sizeof(T) / 16;
    float4 q[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) q[k] = lds[(D * NV + k) * 64 + lane];
    T w[12];
    __builtin_memcpy(w, q, sizeof(w));
    hop_accumulate<D, DAG>(acc, w);
    if constexpr (D + 1 < 8) split_sum<D + 1, P, DAG>(lds, lane, acc);
}

template <int P, int R, bool DAG, bool XPAY, bool NT, int RED = 0>
__device__ __forceinline__ bool dslash_split(const DslashArgs& A, uint32_t group, int rhs, float4* lds,
                                             double* red = nullptr)
{
    using T = typename RealOf<P>::T;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const uint32_t i = group * 64 + lane;
    const bool valid = i < (uint32_t)A.g.Vh;
    const uint32_t cb = valid ? i : 0;   // lanes past the last site work on site 0 and store nothing
    int c[4];
    cb_coords(A.g, cb, A.par, c);
    const char* in = A.in + rhs * A.in_stride;
    T xv[24];
    if (XPAY && wave == 0) SpinorIO<P>::load(A.x + rhs * A.x_stride, A.g.ps, cb, xv);
    if (wave == 0) split_hops<0, P, R, DAG, NT>(A, cb, c, in, lds, lane);
    else if (wave == 1) split_hops<1, P, R, DAG, NT>(A, cb, c, in, lds, lane);
    else if (wave == 2) split_hops<2, P, R, DAG, NT>(A, cb, c, in, lds, lane);
    else split_hops<3, P, R, DAG, NT>(A, cb, c, in, lds, lane);
    __syncthreads();
    if (wave != 0 || !valid) return false;
    T acc[24];
#pragma unroll
    for (int k = 0; k < 24; ++k) acc[k] = 0;
    split_sum<0, P, DAG>(lds, lane, acc);
    dslash_finish<P, XPAY, RED, XPAY>(A, cb, rhs, acc, red, xv);
    return true;
}

} // namespace wd
